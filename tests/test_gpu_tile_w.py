"""The product from the cells forms each contact's w again; it is the collide's,
bit for bit.  With equal frictions and none against the medium, the row of a cell
next to exactly one cell that moves by 1 along x is -w of that contact: cells
three contacts apart or more move, and every contact they have is compared."""
import numpy as np
import pytest
import torch

from workloads import sphere_cluster
from workloads.paper import hcp_sites

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import host, to_dev  # noqa: E402


def _cells(kind, n):
    rng = np.random.default_rng(n)
    if kind == "fcc":
        c = sphere_cluster(n, 73)
        return c["pos"], c["radius"]
    if kind == "hcp":
        return hcp_sites(n) + rng.normal(0, 0.15, (n, 3)), np.full(n, 0.5)
    if kind == "dense":
        return rng.uniform(0, (n / 6.0) ** (1 / 3), (n, 3)), np.full(n, 0.5)
    return rng.uniform(0, (n / 1.22) ** (1 / 3), (n, 3)), rng.uniform(0.2, 1.0, n)   # about 10 contacts a cell


@pytest.mark.parametrize("kind,n,scale,hertz", [
    ("fcc", 9001, 1.0, False), ("fcc", 150_001, 1.0, True), ("hcp", 20_011, 1e3, True), ("dense", 9001, 1.0, True),
    ("mixed", 160_003, 1.0, True), ("mixed", 9001, 1e-4, False), ("fcc", 9000, 1e-110, False)])
def test_w_is_the_collides(kind, n, scale, hertz):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pos, R = _cells(kind, n)
    ctx = P.Context()
    ctx.set_contact_model("hertz" if hertz else "overlap")
    g = ctx.collide(to_dev(scale * pos), to_dev(scale * R), 64)
    e = ctx.graph_export(g)
    ei, ej, w = (host(e[k]) for k in ("ei", "ej", "w"))
    rowptr, col = host(e["rowptr"]), host(e["col"])
    A = ctx.assemble_gamma(g, g_par=1.0, g_perp=1.0, g_med=0.0)
    order = np.random.default_rng(1).permutation(n)
    near = np.zeros(n, bool)   # within two contacts of a moved cell
    moved = np.zeros(n, bool)
    for i in order[:20_000]:
        row = col[rowptr[i]:rowptr[i + 1]]
        if near[i] or near[row].any():
            continue
        moved[i] = True
        near[i] = True
        near[row] = True
    x = np.zeros((n, 3))
    x[moved, 0] = 1.0
    y = host(ctx.spmv(A, to_dev(x)))
    assert np.array_equal(y[:, 1:], np.zeros((n, 2)))
    a, b = np.where(moved[ei])[0], np.where(moved[ej])[0]
    assert len(a) + len(b) > 1000 and not np.intersect1d(a, b).size
    assert np.array_equal(y[ej[a], 0], -w[a]) and np.array_equal(y[ei[b], 0], -w[b])
    ctx.close()
