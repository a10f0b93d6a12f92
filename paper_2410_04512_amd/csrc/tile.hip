// The product q = Gamma p from the cells themselves (large systems).
//
// A contact's block is a function of its two cells (eq. cell_cell_friction):
// with dx = r_j - r_i, d = |dx| and the contact area w(R_i + R_j - d),
//   q_i = g_med p_i + sum_j w (g_perp e + (g_par - g_perp) (u . e) u),
//   e = p_i - p_j, u = dx / d,
// so a row needs its cell's position and radius (32 B) and its neighbours'
// numbers, not 24 B per entry of stored contact vectors and a diagonal block:
// 1e6 cells, ~10.5 contacts each: 418 MB -> 140 MB of memory traffic a product
// by the counters, 87.1 -> 34.7 us alone (4.0 TB/s), 89.1 -> 35.5 in a solve.  The price, a square root and
// ~45 FP64 operations per entry, keeps the vector units busy for half of that
// time and the LDS for a third; two lanes per contact, each row its own, cost
// less than sums that meet from both sides.  w is bit for bit the collide's
// (same operations, a correctly rounded square root); no value is kept in
// fewer bits than before, and the FP32 product's sums are FP64 too.
//
// Rows are cut into tiles of consecutive cells of the internal order (cubes of
// the cell list's bricks, so a tile's outside neighbours, its halo, number
// about as many as its rows).  A workgroup stages position, radius and p of its
// rows and its halo in LDS, and the entries are 16-bit LDS numbers, [row][W]
// with W the largest row of the graph rounded up to 4, 0xffff past the row's
// end.  Entries keep the row's neighbour order, the sums are in that order
// (TPR lanes per row take every TPR-th group of four, read together: one entry
// at a time behind a branch of its own took 52 us), so a product is bitwise
// reproducible.  A tile whose halo does not fit, or whose distances leave the
// range of the plain square root iteration, is marked and multiplied from the
// columns in global memory (hcnt < 0).
#include "sgp_internal.h"

#include <hip/hip_ext.h>

#include <climits>
#include <type_traits>

constexpr int TILE_HASH = 2048;
constexpr int TILE_HALO_MAX = 474;   // (256 + 474) x 56 B of LDS: four workgroups per CU

// Tile shape by size: 256 rows of one lane where that gives every CU a few
// workgroups, 128 rows of two lanes below.  ms per solve or step with 64 (four
// lanes), 128 and 256 rows: 2e4 cells 15.7, 15.2, 16.3; 5e4 16.1, 15.9, 16.2;
// 2e5 14.1, 13.3, 12.9; 5e5 (FP32) 27.4, 26.1, 25.3; 1e6 61.7, 57.4, 55.6.
// With more than TILE_DENSE contacts a cell in the mean the halos of larger tiles
// do not fit, so 64: us per product (and per iteration with block Jacobi) at 200k
// cells with 256 and with 64 rows: 14 contacts 29.0, 30.6 (34.0, 38.6), 18 contacts
// 36.9, 31.7 (42.1, 39.5), 25 contacts 57.6, 34.0 (63.3, 41.6; stored contacts
// 53.0, 69.1); 20k cells with 128 and with 64: 25 contacts 12.6, 10.6 (17.4, 15.5;
// stored 12.2, 27.5).
constexpr int64_t TILE_DENSE = 16;
static int tile_rows_for(int64_t n, int64_t entries)
{
    return entries > TILE_DENSE * n ? 64 : n >= 150000 ? 256 : 128;
}
// Tiles are cut at the clusters of a batch, so that a product forms p.q per
// cluster, unless that makes more than TILE_CUT times as many (clusters much
// smaller than a tile): then they are cut straight through, and p.q takes a pass
// of its own.  us per product and ms per block Jacobi solve, cut at the clusters
// and straight: 7000 clusters of 30 cells (8.5 times the tiles) 37.1, 19.8 and
// 7.48, 6.04; 3000 of 64 (4) 24.0, 18.3 and 4.64, 4.19; 2000 of 100 (2.6) 23.5,
// 20.7 and 4.20, 4.05; 300 of 64 (2) 9.3, 9.0 and 1.65, 1.74; 1000 of 200 (1.3)
// 21.4, 21.4 and 3.61, 3.94.
constexpr double TILE_CUT = 2.5;
constexpr int tile_halo_cap(int rows) { return rows == 256 ? TILE_HALO_MAX : rows == 128 ? 384 : 512; }

struct TileArgs {
    int64_t n;
    int32_t W, cap;
    const int32_t *row0, *row1, *inst;   // per tile (null: one cluster, tiles of TR rows)
    const int32_t *rowptr, *ecol;        // block CSR rows (the diagonal block counted), columns
    const uint16_t *idx;
    const int32_t *halo, *hcnt;
    const double4 *pos;                  // position and radius, internal order
    double gpar, gperp, gmed;
};

template <int TR>
SGP_DEV void tile_range(const TileArgs &A, int64_t tile, int64_t &r0, int64_t &r1)
{
    if (A.row0) {
        r0 = A.row0[tile];
        r1 = A.row1[tile];
    } else {
        r0 = tile * TR;
        r1 = min(r0 + TR, A.n);
    }
}

// ---------------------------------------------------------------- assembly

// squared distances that the plain square root iteration takes (tile_root)
SGP_DEV bool tile_in_range(double d2) { return d2 > 0x1p-700 && d2 < 0x1p700; }

SGP_DEV uint32_t tile_hash(int32_t j) { return ((uint32_t)j * 2654435761u) >> 21; }

// One workgroup per tile: the columns of its rows (internal numbers), its halo
// (distinct outside columns by a hash table in LDS, then in ascending order)
// and the entries' LDS numbers.  Bound by the chains of gathers of a thread, so
// BUILD_LANES lanes share a row and take eight entries of their TR / 64 rows
// together, the next ones' columns with them: the longest row of a wave counts,
// 40 entries where radii differ by 3.  The rows' positions stay in LDS, so that
// four workgroups fit a CU.  200k cells 50 -> 43 us, radii in [0.3, 1] 86 -> 51,
// 25 contacts a cell 139 -> 82, against one or two lanes a row.
constexpr int BUILD_LANES = 4;
template <int TR>
__global__ __launch_bounds__(256, 4) void k_tile_build(TileArgs A, const int32_t *grow, const int32_t *gcol,
                                                    const int32_t *perm, const int32_t *inv, int32_t *ecol,
                                                    uint16_t *idx, int32_t *halo, int32_t *hcnt)
{
    constexpr int PASS = 256 / BUILD_LANES, RP = TR / PASS, EPR = 8 / RP, STEP = BUILD_LANES * EPR;
    __shared__ int32_t tab[TILE_HASH], where[1024];
    __shared__ alignas(16) int32_t list[1024];
    __shared__ uint16_t val[TILE_HASH];
    __shared__ double own[3][TR];   // the rows' positions
    __shared__ int32_t count, bad, fill, most;
    const int tid = threadIdx.x, sub = tid % BUILD_LANES, lr = tid / BUILD_LANES;
    const int64_t tile = blockIdx.x;
    int64_t r0, r1;
    tile_range<TR>(A, tile, r0, r1);
    // the thread's rows lr, lr + PASS, .. (a row past the tile's end: no entries)
    int32_t u[RP], b[RP], deg[RP], k0[RP], longest = 0;
#pragma unroll
    for (int k = 0; k < RP; k++) {
        const int64_t i = min(r0 + lr + PASS * k, A.n - 1);
        u[k] = perm[i];
        k0[k] = A.rowptr[i] - (int32_t)i;
    }
#pragma unroll
    for (int k = 0; k < RP; k++) {
        b[k] = grow[u[k]];
        deg[k] = grow[u[k] + 1];
    }
    for (int k = tid; k < TILE_HASH; k += 256) tab[k] = -1;
    for (int k = tid; k < 1024; k += 256) list[k] = INT_MAX;   // past the halo: below no cell
    if (tid == 0) count = bad = fill = most = 0;
    if (tid < TR) {
        const double4 me = A.pos[min(r0 + tid, A.n - 1)];
        own[0][tid] = me.x;
        own[1][tid] = me.y;
        own[2][tid] = me.z;
    }
    const int32_t any = u[0];   // (what a row without entries reads)
#pragma unroll
    for (int k = 0; k < RP; k++) {
        deg[k] = r0 + lr + PASS * k < r1 ? deg[k] - b[k] : 0;
        longest = max(longest, deg[k]);
    }
    __syncthreads();
    if (sub == 0 && longest > *(volatile int32_t *)&most) atomicMax(&most, longest);
    // columns of entries c0 + sub + BUILD_LANES m (clamped; of a row without entries: any cell)
    int32_t js[RP][EPR];
    auto columns = [&](int32_t c0) {
#pragma unroll
        for (int k = 0; k < RP; k++)
#pragma unroll
            for (int m = 0; m < EPR; m++)
                js[k][m] = deg[k] > 0 ? gcol[b[k] + min(c0 + sub + BUILD_LANES * m, deg[k] - 1)] : any;
    };
    if (longest > 0) columns(0);
    for (int32_t c0 = 0; c0 < longest; c0 += STEP) {
        int32_t jj[RP][EPR];
        double ox[RP][EPR], oy[RP][EPR], oz[RP][EPR];
#pragma unroll
        for (int k = 0; k < RP; k++)
#pragma unroll
            for (int m = 0; m < EPR; m++) jj[k][m] = inv[js[k][m]];
        columns(c0 + STEP);
#pragma unroll
        for (int k = 0; k < RP; k++)
#pragma unroll
            for (int m = 0; m < EPR; m++) {
                ox[k][m] = A.pos[jj[k][m]].x;
                oy[k][m] = A.pos[jj[k][m]].y;
                oz[k][m] = A.pos[jj[k][m]].z;
            }
        keep_loads_above();
#pragma unroll
        for (int k = 0; k < RP; k++)
#pragma unroll
            for (int m = 0; m < EPR; m++) {
                const int32_t c = c0 + sub + BUILD_LANES * m, j = jj[k][m];
                if (c >= deg[k]) continue;
                ecol[k0[k] + c] = j;
                const int l = lr + PASS * k;
                const double dx = ox[k][m] - own[0][l], dy = oy[k][m] - own[1][l], dz = oz[k][m] - own[2][l];
                const double d2 = (dx * dx + dy * dy) + dz * dz;
                if (!tile_in_range(d2)) bad = 1;
                if (j >= r0 && j < r1) continue;
                // (past the cap the tile is marked and nothing more is inserted: at
                // most 256 threads are beyond this test, so the table never fills)
                if (*(volatile int32_t *)&count > A.cap) continue;
                for (uint32_t h = tile_hash(j);; h = (h + 1) & (TILE_HASH - 1)) {
                    const int32_t old = atomicCAS(&tab[h], -1, j);
                    if (old == -1) atomicAdd(&count, 1);
                    if (old == -1 || old == j) break;
                }
            }
    }
    __syncthreads();
    const int32_t hc = count;
    if (hc > A.cap || bad) {
        if (tid == 0) hcnt[tile] = bad ? -2 : -1;
        return;
    }
    for (int k = tid; k < TILE_HASH; k += 256)
        if (tab[k] >= 0) {
            const int32_t p = atomicAdd(&fill, 1);
            list[p] = tab[k];
            where[p] = k;
        }
    __syncthreads();
    for (int k = tid; k < hc; k += 256) {
        const int32_t j = list[k];
        int32_t rank = 0;
        for (int m = 0; m < hc; m += 4) {
            const int4 o = *(const int4 *)(list + m);
            rank += (o.x < j) + (o.y < j) + (o.z < j) + (o.w < j);
        }
        halo[tile * A.cap + rank] = j;
        val[where[k]] = (uint16_t)(TR + rank);
    }
    if (tid == 0) hcnt[tile] = hc;
    __syncthreads();
    // groups of four entries, as far as the product reads them: the first four,
    // and those up to the tile's longest row and one round of lanes beyond
    constexpr int TPR = 256 / TR;
    const int used = max(4, ((most + 3) / 4 + TPR - 1) / TPR * TPR) + TPR, groups = min(A.W / 4, used);
    for (int g = sub; g < groups; g += BUILD_LANES) {
        int32_t c[RP][4];
#pragma unroll
        for (int k = 0; k < RP; k++)
#pragma unroll
            for (int m = 0; m < 4; m++)   // (stored above by this workgroup)
                c[k][m] = 4 * g + m < deg[k] ? ecol[k0[k] + 4 * g + m] : -1;
#pragma unroll
        for (int k = 0; k < RP; k++) {
            const int64_t i = r0 + lr + PASS * k;
            uint16_t l[4];
#pragma unroll
            for (int m = 0; m < 4; m++) {
                const int32_t j = c[k][m];
                l[m] = 0xffff;
                if (j < 0) continue;
                if (j >= r0 && j < r1) {
                    l[m] = (uint16_t)(j - r0);
                } else {
                    uint32_t h = tile_hash(j);
                    while (tab[h] != j) h = (h + 1) & (TILE_HASH - 1);
                    l[m] = val[h];
                }
            }
            if (i < r1) *(ushort4 *)(idx + i * A.W + 4 * g) = make_ushort4(l[0], l[1], l[2], l[3]);
        }
    }
}

// ---------------------------------------------------------------- the product

constexpr double TILE_PI = 3.14159265358979323846;

SGP_DEV double contact_area(double ri, double rj, double d, bool hertz)
{
    const double s = ri + rj, a = s - d;
    return hertz ? (TILE_PI * ((ri * rj) / s)) * a : a;
}

// d = sqrt(d2) and v = 1 / d, for d2 in the range that the tile build checks.
// The root by Goldschmidt's iteration from the hardware's reciprocal square root
// estimate, with two residual corrections (Markstein), which round correctly in
// that range; v by one Newton step from the same half reciprocal.
SGP_DEV void tile_root(double d2, double &d, double &v)
{
    const double y = __builtin_amdgcn_rsq(d2);
    double g = d2 * y, h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    g = __builtin_fma(__builtin_fma(-g, g, d2), h, g);
    d = __builtin_fma(__builtin_fma(-g, g, d2), h, g);
    v = h + h;
    v = __builtin_fma(__builtin_fma(-d, v, 1.0), v, v);
}

// q += W e of one contact, dx = b - a and radii ra, rb; nothing where !on.
template <bool HERTZ>
SGP_DEV void tile_entry(bool on, double dx, double dy, double dz, double ra, double rb, double e0, double e1, double e2,
                        double gperp, double gdif, double &q0, double &q1, double &q2)
{
    double d2 = (dx * dx + dy * dy) + dz * dz;
    d2 = on ? d2 : 1.0;
    double d, v;
    tile_root(d2, d, v);
    double w = contact_area(ra, rb, d, HERTZ);
    w = on ? w : 0.0;
    const double s = __builtin_fma(dz, e2, __builtin_fma(dy, e1, dx * e0));
    const double cp = w * gperp, cu = ((w * gdif) * (v * v)) * s;
    q0 = __builtin_fma(cp, e0, __builtin_fma(cu, dx, q0));
    q1 = __builtin_fma(cp, e1, __builtin_fma(cu, dy, q1));
    q2 = __builtin_fma(cp, e2, __builtin_fma(cu, dz, q2));
}

// a pair of values, and the LDS of a tile: planes of pairs, so that the lanes
// of a wave, whose s-th neighbours are mostly consecutive cells too, read
// consecutive 16-byte words
template <class T>
struct alignas(2 * sizeof(T)) Pair {
    T a, b;
};

// Partials of p.q per tile (mode 1).  S: the solve's scalars (null: always
// run), inst: the cluster of each tile (null: cluster 0).
template <class T, int TR, bool HERTZ>
__global__ __launch_bounds__(256, 4) void k_spmv_tile(TileArgs A, const T *__restrict__ x, T *__restrict__ y,
                                                   const PcgScalars *S, const int32_t *inst, double *part, int mode)
{
    constexpr int TPR = 256 / TR, CAP = tile_halo_cap(TR), HR = (CAP + 255) / 256, PRE = 4 / TPR > 0 ? 4 / TPR : 1;
    __shared__ Pair<double> lxy[TR + CAP], lzr[TR + CAP];
    __shared__ Pair<T> l01[TR + CAP];
    __shared__ T l2[TR + CAP];
    __shared__ double sh[4];
    const int tid = threadIdx.x, sub = tid % TPR, lr = tid / TPR;
    const int64_t tile = xcd_block(blockIdx.x, gridDim.x);
    int64_t r0, r1;
    tile_range<TR>(A, tile, r0, r1);
    const int32_t dn = S ? S[inst ? inst[tile] : 0].done : 0;
    const int32_t hc = A.hcnt[tile];
    const int64_t i = min(r0 + lr, max(r1 - 1, r0)), ic = min(i, A.n - 1);
    const bool on = r0 + lr < r1;
    // the halo's numbers, the first groups of the row's entries and the rows'
    // own data, then the halo's data (indices clamped; surplus not used)
    int32_t j[HR];
#pragma unroll
    for (int k = 0; k < HR; k++) j[k] = A.halo[tile * CAP + min(tid + 256 * k, CAP - 1)];
    const ushort4 *ip = (const ushort4 *)(A.idx + ic * A.W);
    const int groups = A.W / 4;
    ushort4 iv[PRE];
#pragma unroll
    for (int k = 0; k < PRE; k++) iv[k] = ip[min(sub + TPR * k, groups - 1)];
    const double *pos = (const double *)A.pos;
    const double ax = pos[4 * ic], ay = pos[4 * ic + 1], az = pos[4 * ic + 2], ar = pos[4 * ic + 3];
    const T p0 = x[3 * ic], p1 = x[3 * ic + 1], p2 = x[3 * ic + 2];
    double hp[HR][4];
    T hx[HR][3];
#pragma unroll
    for (int k = 0; k < HR; k++) {
        const int64_t jj = tid + 256 * k < hc ? j[k] : ic;
        for (int t = 0; t < 4; t++) hp[k][t] = pos[4 * jj + t];
        for (int t = 0; t < 3; t++) hx[k][t] = x[3 * jj + t];
    }
    keep_loads_above();
    if (dn) return;
    double q0 = 0.0, q1 = 0.0, q2 = 0.0;
    const double gdif = A.gpar - A.gperp;
    if (hc >= 0) {
        if (sub == 0) {
            lxy[lr] = {ax, ay};
            lzr[lr] = {az, ar};
            l01[lr] = {p0, p1};
            l2[lr] = p2;
        }
#pragma unroll
        for (int k = 0; k < HR; k++) {
            const int l = TR + min(tid + 256 * k, CAP - 1);
            if (tid + 256 * k < hc) {
                lxy[l] = {hp[k][0], hp[k][1]};
                lzr[l] = {hp[k][2], hp[k][3]};
                l01[l] = {hx[k][0], hx[k][1]};
                l2[l] = hx[k][2];
            }
        }
        __syncthreads();
        // four entries at a time, all their reads first; a lane past its
        // row's end reads its own cell and adds nothing
        auto group = [&](const ushort4 &v) {
            const uint16_t l[4] = {v.x, v.y, v.z, v.w};
            Pair<double> xy[4], zr[4];
            Pair<T> pp[4];
            T p3[4];
#pragma unroll
            for (int m = 0; m < 4; m++) {
                const int lm = l[m] == 0xffff ? lr : l[m];
                xy[m] = lxy[lm];
                zr[m] = lzr[lm];
                pp[m] = l01[lm];
                p3[m] = l2[lm];
            }
#pragma unroll
            for (int m = 0; m < 4; m++)
                tile_entry<HERTZ>(l[m] != 0xffff, xy[m].a - ax, xy[m].b - ay, zr[m].a - az, ar, zr[m].b,
                                  (double)p0 - (double)pp[m].a, (double)p1 - (double)pp[m].b,
                                  (double)p2 - (double)p3[m], A.gperp, gdif, q0, q1, q2);
        };
#pragma unroll
        for (int k = 0; k < PRE; k++) {
            if (!on || sub + TPR * k >= groups) iv[k].x = iv[k].y = iv[k].z = iv[k].w = 0xffff;
            if (__any(iv[k].x != 0xffff)) group(iv[k]);
        }
        for (int g = TPR * PRE; g < groups; g += TPR) {
            ushort4 v = ip[min(g + sub, groups - 1)];
            if (!on || g + sub >= groups) v.x = v.y = v.z = v.w = 0xffff;
            if (!__any(v.x != 0xffff)) break;
            group(v);
        }
    } else if (on) {
        // marked tiles (hc -1: the halo does not fit, -2: distances): columns and
        // cells from global memory
        const int32_t b = A.rowptr[i] - (int32_t)i, e = A.rowptr[i + 1] - (int32_t)(i + 1);
        if (hc == -1) {
            // the gathers of two entries together: 116 registers, so that the path
            // costs no tile a workgroup per CU (four together: 150, 25.2 -> 26.3 us
            // for 32 clusters with halos; one behind the other, with the library's
            // root and divisions: radii in [0.2, 1], 200k cells, 35.3 us instead of
            // 31.0, stored contacts 31.7)
            for (int32_t g = b + 4 * sub; g < e; g += 4 * TPR) {
                int32_t nx[4];
#pragma unroll
                for (int m = 0; m < 4; m++) nx[m] = A.ecol[min(g + m, e - 1)];
#pragma unroll
                for (int h = 0; h < 4; h += 2) {
                    double o[2][4];
                    T px[2][3];
#pragma unroll
                    for (int m = 0; m < 2; m++) {
                        const int64_t jj = nx[h + m];
                        for (int t = 0; t < 4; t++) o[m][t] = pos[4 * jj + t];
                        for (int t = 0; t < 3; t++) px[m][t] = x[3 * jj + t];
                    }
                    keep_loads_above();
#pragma unroll
                    for (int m = 0; m < 2; m++) {
                        __builtin_amdgcn_sched_barrier(0);
                        tile_entry<HERTZ>(g + h + m < e, o[m][0] - ax, o[m][1] - ay, o[m][2] - az, ar, o[m][3],
                                          (double)p0 - (double)px[m][0], (double)p1 - (double)px[m][1],
                                          (double)p2 - (double)px[m][2], A.gperp, gdif, q0, q1, q2);
                    }
                }
            }
        } else {
            for (int32_t g = b + 4 * sub; g < e; g += 4 * TPR)
                for (int32_t k = g; k < min(g + 4, e); k++) {
                    const int64_t jj = A.ecol[k];
                    const double4 o = A.pos[jj];
                    const double dx = o.x - ax, dy = o.y - ay, dz = o.z - az;
                    const double d = sqrt((dx * dx + dy * dy) + dz * dz);
                    const double w = contact_area(ar, o.w, d, HERTZ), u0 = dx / d, u1 = dy / d, u2 = dz / d;
                    const double e0 = (double)p0 - (double)x[3 * jj], e1 = (double)p1 - (double)x[3 * jj + 1],
                                 e2 = (double)p2 - (double)x[3 * jj + 2];
                    const double cu = (w * gdif) * ((u0 * e0 + u1 * e1) + u2 * e2), cp = w * A.gperp;
                    q0 += cp * e0 + cu * u0;
                    q1 += cp * e1 + cu * u1;
                    q2 += cp * e2 + cu * u2;
                }
        }
    }
#pragma unroll
    for (int o = 1; o < TPR; o <<= 1) {
        q0 = q0 + __shfl_xor(q0, o, 64);
        q1 = q1 + __shfl_xor(q1, o, 64);
        q2 = q2 + __shfl_xor(q2, o, 64);
    }
    double d = 0.0;
    if (on && sub == 0) {
        const T y0 = (T)__builtin_fma(A.gmed, (double)p0, q0), y1 = (T)__builtin_fma(A.gmed, (double)p1, q1),
                y2 = (T)__builtin_fma(A.gmed, (double)p2, q2);
        y[3 * i] = y0;
        y[3 * i + 1] = y1;
        y[3 * i + 2] = y2;
        d = ((double)p0 * (double)y0 + (double)p1 * (double)y1) + (double)p2 * (double)y2;
    }
    if (mode) {
        d = wave_sum(d);
        if ((tid & 63) == 0) sh[tid >> 6] = d;
        __syncthreads();
        if (tid == 0) part[tile] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
    }
}

// Gamma's diagonal blocks (64-row groups of 6 planes), summed over the row's
// contacts in neighbour order: the assembly's sums, with u to the last place.
// Bound by the FP64 operations and a row's chain of gathers: four entries at a
// time and no library root or division.
template <bool HERTZ>
__global__ void k_tile_diag(TileArgs A, double *dg)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    const double4 me = A.pos[i];
    double D[9];
    for (int t = 0; t < 9; t++) D[t] = t % 4 == 0 ? A.gmed : 0.0;
    const int64_t b = (int64_t)A.rowptr[i] - i, e = (int64_t)A.rowptr[i + 1] - (i + 1);
    constexpr int BATCH = 4;
    int32_t nx[BATCH];
#pragma unroll
    for (int m = 0; m < BATCH; m++) nx[m] = b < e ? A.ecol[min(b + m, e - 1)] : (int32_t)i;
    for (int64_t k0 = b; k0 < e; k0 += BATCH) {
        double4 o[BATCH];
#pragma unroll
        for (int m = 0; m < BATCH; m++) o[m] = A.pos[nx[m]];
#pragma unroll
        for (int m = 0; m < BATCH; m++) nx[m] = A.ecol[min(k0 + BATCH + m, e - 1)];
        keep_loads_above();
#pragma unroll
        for (int m = 0; m < BATCH; m++) {
            if (k0 + m >= e) break;
            const double dx = o[m].x - me.x, dy = o[m].y - me.y, dz = o[m].z - me.z;
            const double d2 = (dx * dx + dy * dy) + dz * dz;
            double d, v, u[3] = {dx, dy, dz};
            if (tile_in_range(d2)) {
                tile_root(d2, d, v);
                for (int a = 0; a < 3; a++) {   // u / d with one residual correction
                    const double t = u[a] * v;
                    u[a] = __builtin_fma(__builtin_fma(-t, d, u[a]), v, t);
                }
            } else {
                d = sqrt(d2);
                for (int a = 0; a < 3; a++) u[a] = u[a] / d;
            }
            const double w = contact_area(me.w, o[m].w, d, HERTZ);
            for (int a = 0; a < 3; a++)
                for (int c = a; c < 3; c++) {
                    const double uu = u[a] * u[c], id = a == c ? 1.0 : 0.0;
                    D[3 * a + c] = D[3 * a + c] + w * (A.gpar * uu + A.gperp * (id - uu));
                }
        }
    }
    double *g = dg + (i >> 6) * 384 + (i & 63);
    g[0] = D[0];
    g[64] = D[1];
    g[128] = D[2];
    g[192] = D[4];
    g[256] = D[5];
    g[320] = D[8];
}

static TileArgs tile_args(sgp_bsr A)
{
    TileArgs t = {};
    t.n = A->n;
    t.W = A->tile_w;
    t.cap = tile_halo_cap(A->tile_rows);
    if (A->tile_off.size() > 2) {
        const int32_t *d = (const int32_t *)A->tile_tab.p;
        t.row0 = d;
        t.row1 = d + A->n_tiles;
        t.inst = d + 2 * (size_t)A->n_tiles;
    }
    t.rowptr = (const int32_t *)A->rowptr.p;
    t.ecol = (const int32_t *)A->ecol.p;
    t.idx = (const uint16_t *)A->tile_idx.p;
    t.halo = (const int32_t *)A->tile_halo.p;
    t.hcnt = t.halo + (size_t)A->n_tiles * t.cap;
    t.pos = (const double4 *)A->tile_pos.p;
    t.gpar = A->gpar;
    t.gperp = A->gperp;
    t.gmed = A->gmed;
    return t;
}

// the tile form of A (rowptr built, ecol allocated) from graph g
int tile_assemble(sgp_ctx ctx, sgp_graph g, sgp_bsr A)
{
    hipStream_t st = ctx->stream;
    const int64_t n = A->n;
    A->tile_rows = tile_rows_for(n, 2 * g->m);
    A->tile_w = (std::max(g->max_deg, 1) + 3) / 4 * 4;
    A->tile_hertz = g->hertz;
    const std::vector<int64_t> &off = g->h_inst_off;
    const double most = TILE_CUT * (double)((n + A->tile_rows - 1) / A->tile_rows);
    int64_t tiles = 0;
    for (int64_t k = 0; k < g->n_inst && (double)tiles <= most; k++)
        tiles += std::max<int64_t>((off[k + 1] - off[k] + A->tile_rows - 1) / A->tile_rows, 1);
    if ((double)tiles > most)
        A->tile_off = {0, n};
    else
        A->tile_off = off;
    if (A->tile_off.size() > 2) {
        std::vector<int32_t> buf;
        build_tab(A->tile_off, A->tile_rows, buf, A->n_tiles);
        int32_t *d;
        SGP_TRY(ensure_t(ctx, A->tile_tab, buf.size(), &d));
        SGP_TRY(upload(ctx, d, buf.data(), buf.size() * 4));
    } else {
        A->n_tiles = (int32_t)((n + A->tile_rows - 1) / A->tile_rows);
    }
    const int cap = tile_halo_cap(A->tile_rows);
    uint16_t *idx;
    int32_t *halo;
    double4 *pos;
    SGP_TRY(ensure_t(ctx, A->tile_idx, (size_t)n * A->tile_w, &idx));
    SGP_TRY(ensure_t(ctx, A->tile_halo, (size_t)A->n_tiles * (cap + 1), &halo));
    SGP_TRY(ensure_t(ctx, A->tile_pos, n, &pos));
    const int32_t *perm = (const int32_t *)g->perm.p, *inv = (const int32_t *)g->inv.p;
    HIP_TRY(ctx, hipMemcpyAsync(pos, g->cell.p, n * sizeof(double4), hipMemcpyDeviceToDevice, st));
    const TileArgs t = tile_args(A);
    int32_t *hcnt = halo + (size_t)A->n_tiles * cap;
    const int32_t *gr = (const int32_t *)g->rowptr.p, *gc = (const int32_t *)g->col.p;
    int32_t *ecol = (int32_t *)A->ecol.p;
    if (A->tile_rows == 256)
        k_tile_build<256><<<A->n_tiles, 256, 0, st>>>(t, gr, gc, perm, inv, ecol, idx, halo, hcnt);
    else if (A->tile_rows == 128)
        k_tile_build<128><<<A->n_tiles, 256, 0, st>>>(t, gr, gc, perm, inv, ecol, idx, halo, hcnt);
    else
        k_tile_build<64><<<A->n_tiles, 256, 0, st>>>(t, gr, gc, perm, inv, ecol, idx, halo, hcnt);
    LAUNCH_CHECK(ctx);
    return SGP_OK;
}

int tile_diag(sgp_ctx ctx, sgp_bsr A)
{
    double *dg;
    SGP_TRY(ensure_t(ctx, A->dg, sym_group_size(A->n) + 8, &dg));
    const TileArgs t = tile_args(A);
    if (A->tile_hertz)
        k_tile_diag<true><<<grid_for(A->n, 256), 256, 0, ctx->stream>>>(t, dg);
    else
        k_tile_diag<false><<<grid_for(A->n, 256), 256, 0, ctx->stream>>>(t, dg);
    LAUNCH_CHECK(ctx);
    return SGP_OK;
}

template <class T, int TR, bool HERTZ>
static void tile_launch(sgp_ctx ctx, sgp_bsr A, const T *x, T *y, const PcgScalars *S, const int32_t *inst,
                        double *part, int mode)
{
    const TileArgs t = tile_args(A);
    const auto kernel = k_spmv_tile<T, TR, HERTZ>;
    if (ctx->kt_start) {   // a timed launch carries the kernel timer's events (ktimer_begin)
        hipExtLaunchKernelGGL(kernel, dim3(A->n_tiles), dim3(256), 0, ctx->stream, ctx->kt_start, ctx->kt_stop, 0, t,
                              x, y, S, inst, part, mode);
        ctx->kt_used = true;
    } else {
        kernel<<<A->n_tiles, 256, 0, ctx->stream>>>(t, x, y, S, inst, part, mode);
    }
}

template <class T>
int spmv_tile(sgp_ctx ctx, sgp_bsr A, const T *x, T *y, const PcgScalars *S, bool per_inst, double *part, int mode)
{
    const int32_t *inst = per_inst ? tile_args(A).inst : nullptr;
    auto rows = [&](auto hertz) {
        constexpr bool H = decltype(hertz)::value;
        if (A->tile_rows == 256) tile_launch<T, 256, H>(ctx, A, x, y, S, inst, part, mode);
        else if (A->tile_rows == 128) tile_launch<T, 128, H>(ctx, A, x, y, S, inst, part, mode);
        else tile_launch<T, 64, H>(ctx, A, x, y, S, inst, part, mode);
    };
    if (A->tile_hertz) rows(std::true_type{});
    else rows(std::false_type{});
    LAUNCH_CHECK(ctx);
    return SGP_OK;
}
template int spmv_tile<double>(sgp_ctx, sgp_bsr, const double *, double *, const PcgScalars *, bool, double *, int);
template int spmv_tile<float>(sgp_ctx, sgp_bsr, const float *, float *, const PcgScalars *, bool, double *, int);
