"""The network's weight gradients are sums over all rows and entries.  The energy
loss's derivative at a row is 2 sV (Gamma v_hat - F) / (v . F): v enters it only
through v . F, so k copies of one cluster (a batch: same cells, no contacts
between copies) have, row by row, the derivative of one copy whose v is k times
as large, and k times its gradient.  (The mean squared error's has 1 / (3 n k) in
it before the rounding to BF16, which moves roundings unless k is a power of
two, so its gradients of 1 and k copies differ by more than their sums' order.)
At row counts around the 16-row blocks, the workgroups' shares and the partials'
runs; tolerance 10 sqrt(rows) 2^-24 of a block's norm (FP32 sums in another
order), and the column sums of the output layer against the forward pass."""
import numpy as np
import pytest
import torch

from oracle import mpnn as N
from workloads import sphere_cluster

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import host, to_dev  # noqa: E402


@pytest.mark.parametrize("n,k", [(1, 2), (15, 3), (17, 61), (16, 64), (65, 253), (130, 400)])
def test_gradient_of_copies(n, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context()
    c = sphere_cluster(n, 91)
    rng = np.random.default_rng(n)
    vp, v = rng.normal(size=(2, n, 3))
    M = P.Mpnn(ctx)
    M.set_params(N.init_params(4) + 0.02 * rng.normal(size=N.param_count()), 1.0, 1.0, 0.1)
    got = []
    for copies in (1, k):
        off = n * np.arange(copies + 1)
        t = [to_dev(np.tile(a, (copies, 1))) for a in (c["pos"], c["force"], vp, v)]
        g = ctx.collide_batched(off, t[0], to_dev(np.tile(c["radius"], copies)))
        out = host(M.forward(g, t[1], t[2]))
        assert np.array_equal(out, np.tile(out[:n], (copies, 1)))
        mse, gr = M.grad(g, t[1], t[2], t[3])
        gb = [(2.0 * (out - host(t[3])) / out.size).sum(0)]
        bo = [N.unpack(host(gr).astype(np.float64))["b_out"].ravel()]
        A = ctx.assemble_gamma(g)
        vk = to_dev(host(t[3]) * (k // copies))   # k v for the one copy, v for the k copies
        _, gr = M.grad(g, t[1], t[2], vk, A)
        blocks = N.unpack(host(gr).astype(np.float64) * (k // copies))
        F = host(t[1])
        gb.append((2.0 * (host(ctx.spmv(A, to_dev(out))) - F) / np.sum(host(vk) * F)).sum(0) * (k // copies))
        bo.append(blocks["b_out"].ravel())
        got.append((mse, blocks, bo, gb))
    tol = 10.0 * np.sqrt(n * k) * 2.0 ** -24
    assert abs(got[0][0] - got[1][0]) <= tol * got[0][0]
    for name, _ in N.LAYOUT:
        a, b = got[0][1][name].ravel(), got[1][1][name].ravel()
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(a), name
    for _, _, bo, gb in got:
        for a, b in zip(bo, gb):
            assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b)
    ctx.close()
