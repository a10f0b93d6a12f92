// The cell list's grid (collide.hip): its size and the numbering of its cells.
#ifndef SGP_GRID_H
#define SGP_GRID_H

#include <algorithm>
#include <cmath>
#include <cstdint>

struct Grid {
    double lo[3];
    double inv_h;
    int32_t dim[3];
    int64_t ncell;   // cell numbers per cluster
    // Cell numbering: row by row, or (bricks) in cubes of 2^bits cells per
    // axis, so that consecutive cells fill a cube: the product's tiles of a few
    // hundred cells then have about as many outside neighbours as cells (2.5
    // times as many in rows: 738 against 291 for 256 cells at 1e6)
    int32_t bits[3], nb[3];
    bool bricks;
};

// cell numbers of all clusters at most (keys are 32 bits)
constexpr double GRID_MAX_CELLS = 4.0e9;

// The grid over the box [lo, hi] of n cells in n_inst clusters of radius rmax
// at most: cubes of side 2 rmax or, where that makes more than four cells a
// vertex (or GRID_MAX_CELLS in all), larger ones, which is a correct cell list too.
// bricks: number them in bricks, unless their padding (4 times the cells of
// 5 x 5 x 5 in every one of many clusters) leaves the range of the keys.
inline Grid size_grid(const double *lo, const double *hi, double rmax, int64_t n, int64_t n_inst, bool bricks)
{
    Grid g = {};
    double h = 2.0 * rmax * (1.0 + 0x1p-20);
    if (!(h > 0.0)) h = 1.0;
    const double budget = (double)std::max<int64_t>(4 * n / std::max<int64_t>(n_inst, 1), 64);
    double span[3], ncell;
    // (counted in doubles: a cell far from the others makes more cubes than
    // integers hold before they are enlarged)
    for (;; h *= 1.25) {
        g.inv_h = 1.0 / h;
        ncell = 1.0;
        for (int a = 0; a < 3; a++) {
            g.lo[a] = lo[a];
            span[a] = std::floor((hi[a] - lo[a]) * g.inv_h) + 1.0;
            ncell *= span[a];
        }
        const bool ints = std::max(std::max(span[0], span[1]), span[2]) <= 0x1p30;
        if (ints && ncell <= budget && ncell * (double)n_inst <= GRID_MAX_CELLS) break;
        if (!std::isfinite(h)) {   // a box wider than doubles: one cell
            g.inv_h = 0.0;
            span[0] = span[1] = span[2] = ncell = 1.0;
            break;
        }
    }
    for (int a = 0; a < 3; a++) g.dim[a] = (int32_t)span[a];
    g.ncell = (int64_t)ncell;
    if (bricks) {
        // six bits of brick: two per axis, less along an axis of fewer than
        // four cells (a sheet or a thread), more along the others
        int thin = 0, used = 0;
        for (int a = 0; a < 3; a++) {
            g.bits[a] = -1;
            if (g.dim[a] >= 4) continue;
            g.bits[a] = g.dim[a] > 2 ? 2 : g.dim[a] > 1 ? 1 : 0;
            used += g.bits[a];
            thin++;
        }
        int64_t padded = 1;
        for (int a = 0; a < 3; a++) {
            if (g.bits[a] < 0) g.bits[a] = thin == 0 ? 2 : thin == 1 ? 3 : 6 - used;
            g.nb[a] = (g.dim[a] + (1 << g.bits[a]) - 1) >> g.bits[a];
            padded *= (int64_t)g.nb[a] << g.bits[a];
        }
        g.bricks = (double)padded * n_inst <= GRID_MAX_CELLS;
        if (g.bricks) g.ncell = padded;
    }
    return g;
}

#endif
