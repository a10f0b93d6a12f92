"""The product from the cells on batches: clusters much smaller than a tile (cut
straight through, p.q in a pass of its own), of about its size and larger (cut
at the clusters), with empty clusters between; product and block Jacobi against
the oracle's Gamma, solves against each cluster's own."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from workloads import batched_instance

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


@pytest.mark.parametrize("sizes", [[10] * 900, [3] * 2800, [51] * 180, [52] * 180, [60] * 160, [20] * 120 + [7000],
                                   [129, 128, 127] * 25, [0, 9000, 0, 500, 0]])
def test_batched_product_and_solves(ctx, sizes):
    parts = [batched_instance(k + 7, n_override=s) if s else None for k, s in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pos, R, F = (np.concatenate([p[k] for p in parts if p]) for k in ("pos", "radius", "force"))
    n = int(off[-1])
    assert n > 8192
    g = ctx.collide_batched(off, to_dev(pos), to_dev(R))
    A = ctx.assemble_gamma(g)
    M, J = ctx.factor_tree(g, ctx.build_tree(g)), ctx.make_jacobi(A)
    x = np.random.default_rng(2).normal(size=(n, 3))
    y, z = host(ctx.spmv(A, to_dev(x))), host(ctx.prec_apply(J, to_dev(x)))
    sols = [ctx.pcg_solve_batched(A, m, off, to_dev(F)) for m in (M, J)]
    again = ctx.pcg_solve_batched(A, M, off, to_dev(F))
    assert torch.equal(again[0], sols[0][0]) and again[1] == sols[0][1]
    for k in range(0, len(sizes), max(1, len(sizes) // 12)):
        if not sizes[k]:
            continue
        s = slice(off[k], off[k + 1])
        oa = O.assemble(O.collide(parts[k]["pos"], parts[k]["radius"]))
        ref = O.spmv(oa, x[s])
        assert np.linalg.norm(y[s] - ref) <= 1e-14 * np.linalg.norm(ref), k
        diag = np.stack([oa.val[oa.rowptr[i] + np.searchsorted(oa.bcol[oa.rowptr[i]:oa.rowptr[i + 1]], i)]
                         for i in range(sizes[k])])
        zo = np.linalg.solve(diag, x[s][:, :, None])[:, :, 0]
        assert np.linalg.norm(z[s] - zo) <= 1e-12 * np.linalg.norm(zo), k
        if sizes[k] <= 500:   # relres 1e-8 bounds the velocity by the condition number, below 1e5 here
            vo = np.linalg.solve(_dense(oa), F[s].ravel()).reshape(-1, 3)
            for v, _ in sols:
                assert np.linalg.norm(host(v)[s] - vo) <= 1e-3 * np.linalg.norm(vo), k
    for _, infos in sols:
        assert all(i["status"] == 0 and i["relres_true"] <= 1.0001e-8 for i in infos)


def _dense(a):
    d = np.zeros((a.n, 3, a.n, 3))
    for i in range(a.n):
        for k in range(a.rowptr[i], a.rowptr[i + 1]):
            d[i, :, a.bcol[k]] = np.asarray(a.val[k]).reshape(3, 3)
    return d.reshape(3 * a.n, 3 * a.n)
