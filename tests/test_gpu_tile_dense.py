"""The product from the cells with more than 16 contacts a cell (tiles of 64
rows): both sides of that rule, rows of up to 64 contacts, FP32, a batch whose
product forms p.q per cluster, and one cut straight through its clusters."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import host, to_dev  # noqa: E402


@pytest.fixture()
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = P.Context()
    yield c
    c.close()


def _cloud(n, contacts, seed):
    """Random points of equal radius with about that many contacts a cell."""
    rng = np.random.default_rng(seed)
    return rng.uniform(0, (n * 4 / 3 * np.pi / contacts) ** (1 / 3), (n, 3)), np.full(n, 0.5)


@pytest.mark.parametrize("n,contacts", [(8193, 16.6), (8193, 18.0), (20_000, 25.0), (9001, 36.0), (150_001, 25.0)])
def test_dense_product_matches_oracle(ctx, n, contacts):
    pos, R = _cloud(n, contacts, n)
    g = ctx.collide(to_dev(pos), to_dev(R), 64)
    A = ctx.assemble_gamma(g)
    oa = O.assemble(O.collide(pos, R))
    x = np.random.default_rng(3).normal(size=(n, 3))
    ref = O.spmv(oa, x)
    y = ctx.spmv(A, to_dev(x))
    assert np.linalg.norm(host(y) - ref) <= 1e-14 * np.linalg.norm(ref)
    assert torch.equal(y, ctx.spmv(A, to_dev(x)))
    J = ctx.make_jacobi(A)
    for precision in ("f64", "f32ir"):
        _, info = ctx.pcg_solve(A, J, to_dev(x), precision=precision, inner_rtol=1e-4)
        assert info["status"] == 0 and info["relres_true"] <= 1.0001e-8


@pytest.mark.parametrize("sizes", [[6000, 63, 64, 65, 5000], [400] * 25, [25] * 400])
def test_dense_batches(ctx, sizes):
    parts = [_cloud(s, 30.0, k) for k, s in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pos, R = (np.concatenate([p[k] for p in parts]) for k in (0, 1))
    g = ctx.collide_batched(off, to_dev(pos), to_dev(R), 64)
    A = ctx.assemble_gamma(g)
    x = np.random.default_rng(4).normal(size=(int(off[-1]), 3))
    y = host(ctx.spmv(A, to_dev(x)))
    M = ctx.factor_tree(g, ctx.build_tree(g))
    v, infos = ctx.pcg_solve_batched(A, M, off, to_dev(x))
    assert all(i["status"] == 0 and i["relres_true"] <= 1.0001e-8 for i in infos)
    for k in range(0, len(sizes), max(1, len(sizes) // 8)):
        s = slice(off[k], off[k + 1])
        ref = O.spmv(O.assemble(O.collide(*parts[k])), x[s])
        assert np.linalg.norm(y[s] - ref) <= 1e-14 * np.linalg.norm(ref), k
