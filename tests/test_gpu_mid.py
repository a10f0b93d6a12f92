"""The mid steps' packed words in every shape of the LDS sweeps (groups up to
128, 256, 512, 1024 and 1536 vertices by the knob light_cap) and beyond the
packed words' limit: bit for bit the generic workgroup sweeps, FP64, and inside
an FP32 solve."""
import pytest
import torch

from workloads import sphere_cluster

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import to_dev  # noqa: E402


@pytest.mark.parametrize("n,cap", [(2201, 1), (20011, 64), (120011, 64), (120011, 200), (300007, 512), (300007, 1),
                                   (300007, 1300)])
def test_packed_mid_sweeps_match_generic(n, cap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context()
    ctx.tune("light_cap", cap)
    c = sphere_cluster(n, 33)
    F = to_dev(c["force"])
    g = ctx.collide(to_dev(c["pos"]), to_dev(c["radius"]))
    A = ctx.assemble_gamma(g)
    M = ctx.factor_tree(g, ctx.build_tree(g))
    out = []
    for on in (1, 0):
        ctx.tune("mid_lds", on)
        z = ctx.prec_apply(M, F)
        v, info = ctx.pcg_solve(A, M, F, precision="f32ir", rtol=1e-6, inner_rtol=1e-3)
        out.append((z, v, info["iters"]))
    assert torch.equal(out[0][0], out[1][0])
    assert out[0][2] == out[1][2] and torch.equal(out[0][1], out[1][1])
    ctx.close()
