"""The cell list's grid sizes (csrc/grid.h, host code): over boxes of every
shape, numbers of cells and of clusters, all cell numbers, the padding of the
bricks among them, fit the 32-bit keys, and each cell has a number of its own."""
import itertools
import os
import random
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_04512_amd", "csrc")
PROGRAM = """
#include "grid.h"
#include <cstdio>
int main()
{
    double lo[3] = {0, 0, 0}, hi[3], r;
    long long n, inst;
    int bricks;
    while (std::scanf("%lf %lf %lf %lf %lld %lld %d", hi, hi + 1, hi + 2, &r, &n, &inst, &bricks) == 7) {
        Grid g = size_grid(lo, hi, r, n, inst, bricks != 0);
        std::printf("%d %d %d %lld %d %d %d %d %d %d %d %.17g\\n", g.dim[0], g.dim[1], g.dim[2], (long long)g.ncell,
                    (int)g.bricks, g.bits[0], g.bits[1], g.bits[2], g.nb[0], g.nb[1], g.nb[2], g.inv_h);
    }
}
"""


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("grid")
    (d / "grid.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(d / "grid.cpp"), "-o", str(d / "grid")], check=True)

    def run(cases):
        text = "\n".join("%.17g %.17g %.17g %.17g %d %d %d" % c for c in cases)
        out = subprocess.run([str(d / "grid")], input=text, capture_output=True, text=True, check=True).stdout
        rows = []
        for line in out.splitlines():
            v = line.split()
            rows.append({"dim": [int(x) for x in v[:3]], "ncell": int(v[3]), "bricks": v[4] == "1",
                         "bits": [int(x) for x in v[5:8]], "nb": [int(x) for x in v[8:11]], "inv_h": float(v[11])})
        assert len(rows) == len(cases)
        return rows

    return run


def _number(g, c):
    if not g["bricks"]:
        return (c[2] * g["dim"][1] + c[1]) * g["dim"][0] + c[0]
    hi = [x >> b for x, b in zip(c, g["bits"])]
    lo = [x & ((1 << b) - 1) for x, b in zip(c, g["bits"])]
    k = (hi[2] * g["nb"][1] + hi[1]) * g["nb"][0] + hi[0]
    for a in (2, 1, 0):
        k = (k << g["bits"][a]) | lo[a]
    return k


def test_numbers_fit_their_keys(sizes):
    rng = random.Random(1)
    cases = []
    for _ in range(4000):
        n = int(10 ** rng.uniform(4, 9.02))
        inst = int(n ** rng.uniform(0, 1)) if rng.random() < 0.7 else 1
        side = (n / inst) ** (1 / 3) * 10 ** rng.uniform(-0.5, 1.5)
        cases.append(tuple(max(1e-3, side * 10 ** rng.uniform(-1, 1)) for _ in range(3)) + (0.5, n, inst, 1))
    # cubes of 5 grid cells in many clusters, a thread and a slab at the largest size
    cases += [(4.5, 4.5, 1.5, 0.5, 10 ** 9, 40_000_000, 1), (4.5, 4.5, 4.5, 0.5, 10 ** 9, 30_000_000, 1),
              (4.5, 4.5, 1.5e8, 0.5, 10 ** 9, 1, 1), (4.5, 3.5e4, 2.5e4, 0.5, 10 ** 9, 1, 1)]
    for c, g in zip(cases, sizes(cases)):
        assert g["ncell"] * c[5] <= 2 ** 32, (c, g)
        last = [d - 1 for d in g["dim"]]
        assert _number(g, last) < g["ncell"], (c, g)
        for a in range(3):
            assert last[a] >= int((c[a]) * g["inv_h"]), (c, g)   # the box is covered


@pytest.mark.parametrize("far", [1e7, 1e11, 1e15, 1e300])
def test_far_cells(sizes, far):
    """A cell far from the others: more cubes along an axis than 32 bits count."""
    cases = [(far, 9.0, 9.0, 0.5, 20_000, 1, 1), (far, far, far, 0.5, 1_000_000, 1, 1), (5.0, far, far, 0.5, 100, 7, 0),
             (far, 0.5, 0.5, 0.5, 2 ** 30 - 1, 1, 1)]
    for c, g in zip(cases, sizes(cases)):
        assert 1 <= min(g["dim"]) and max(g["dim"]) < 2 ** 31 and 0 < g["ncell"] < 2 ** 32, (c, g)
        assert g["dim"][0] * g["dim"][1] * g["dim"][2] <= max(4 * c[4] // c[5], 64), (c, g)


@pytest.mark.parametrize("bricks", [0, 1])
def test_every_cell_has_its_own_number(sizes, bricks):
    boxes = [(a, b, c) for a, b, c in itertools.product((0.5, 1.5, 2.5, 4.5, 6.5), repeat=3)]
    cases = [(a, b, c, 0.5, 10_000, 1, bricks) for a, b, c in boxes]
    for g in sizes(cases):
        cells = list(itertools.product(*(range(d) for d in g["dim"])))
        numbers = {_number(g, c) for c in cells}
        assert len(numbers) == len(cells) and max(numbers) < g["ncell"]
