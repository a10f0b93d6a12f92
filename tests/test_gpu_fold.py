"""The CG scalars formed by every block of the pass that uses them (up to 2048
partials a cluster) or by a launch of their own, and block Jacobi applied in
the pass that forms r: a few iterations against NumPy's CG on the library's own
product and apply.  Tolerance: a dot product of 3n terms carries at most
(8 + log2 of the partials) roundings of 2^-53 on either side, under 1e-14, and
five iterations multiply an error of alpha or beta by at most ten each (the
residual falls by less than that): 1e-9."""
import numpy as np
import pytest
import torch

from workloads import batched_instance, sphere_cluster

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import host, to_dev  # noqa: E402

ITS = 5


def _cg(product, apply, F):
    x, r = np.zeros_like(F), F.copy()
    z = apply(r)
    p, rho = z, np.sum(r * z)
    for _ in range(ITS):
        q = product(p)
        a = rho / np.sum(p * q)
        x, r = x + a * p, r - a * q
        z = apply(r)
        beta, rho = np.sum(r * z) / rho, np.sum(r * z)
        p = z + beta * p
    return x, np.linalg.norm(r) / np.linalg.norm(F)


@pytest.mark.parametrize("prec", ["none", "jacobi", "tree"])
@pytest.mark.parametrize("n", [8193, 65537, 262144, 262145, 524289])   # 33, 257, 1024, 1025 and 2049 blocks of rows
def test_first_iterations(n, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context()
    c = sphere_cluster(n, 5)
    g = ctx.collide(to_dev(c["pos"]), to_dev(c["radius"]))
    A = ctx.assemble_gamma(g)
    M = {"none": lambda: None, "jacobi": lambda: ctx.make_jacobi(A),
         "tree": lambda: ctx.factor_tree(g, ctx.build_tree(g))}[prec]()
    apply = (lambda r: host(ctx.prec_apply(M, to_dev(r)))) if M is not None else (lambda r: r)
    x, res = _cg(lambda p: host(ctx.spmv(A, to_dev(p))), apply, c["force"])
    v, info = ctx.pcg_solve(A, M, to_dev(c["force"]), fixed_iters=ITS)
    assert info["iters"] == ITS
    assert np.linalg.norm(host(v) - x) <= 1e-9 * np.linalg.norm(x)
    assert abs(info["relres_rec"] - res) <= 1e-9 * res
    ctx.close()


def test_first_iterations_batched():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context()
    sizes = [8500, 1, 257, 256, 4000]
    parts = [batched_instance(k + 17, n_override=s) for k, s in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pos, R, F = (np.concatenate([p[k] for p in parts]) for k in ("pos", "radius", "force"))
    g = ctx.collide_batched(off, to_dev(pos), to_dev(R))
    A = ctx.assemble_gamma(g)
    J = ctx.make_jacobi(A)
    v, infos = ctx.pcg_solve_batched(A, J, off, to_dev(F), fixed_iters=ITS)
    for k in range(len(sizes)):
        a, b = off[k], off[k + 1]
        if sizes[k] == 1:   # (exact after one iteration: nothing left to compare)
            continue

        def padded(f):
            def g(w):
                full = np.zeros_like(F)
                full[a:b] = w
                return host(f(to_dev(full)))[a:b]
            return g
        x, res = _cg(padded(lambda t: ctx.spmv(A, t)), padded(lambda t: ctx.prec_apply(J, t)), F[a:b])
        assert infos[k]["iters"] == ITS
        assert np.linalg.norm(host(v)[a:b] - x) <= 1e-9 * np.linalg.norm(x)
        assert abs(infos[k]["relres_rec"] - res) <= 1e-9 * res
    ctx.close()
