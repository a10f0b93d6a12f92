"""The autotuner times a factor once where tail_max does not change it: beyond
2200 cells a contraction factor ends in the dense block whatever tail_max is, and
three timings of the same factor would be chosen among by noise."""
import pytest
import torch

from workloads import sphere_cluster

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from paper_2410_04512_amd import autotune  # noqa: E402
from tests.gpu_util import to_dev  # noqa: E402


@pytest.mark.parametrize("n,alike", [(6000, True), (2100, False)])
def test_equal_factors_are_timed_once(n, alike):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context()
    ctx.tune("small_solve", 0)
    c = sphere_cluster(n, 8)
    g = ctx.collide(to_dev(c["pos"]), to_dev(c["radius"]))
    A, T = ctx.assemble_gamma(g), ctx.build_tree(g)
    res = autotune.tune(ctx, g, T, A, to_dev(c["force"]), fixed_iters=4, repeats=1)
    t = [res["table"][f"schedule=contract,light_height=0,tail_max={tm}"] for tm in autotune.TAIL_MAX]
    assert (len(set(t)) == 1) == alike
    assert len(res["table"]) == len(autotune.TAIL_MAX) * (len(autotune.LIGHT_HEIGHT) + 1) + len(autotune.SPMV_WAVES) \
        + len(autotune.GRAPH) * len(autotune.CHECK_EVERY)
    v, info = ctx.pcg_solve(A, res["prec"], to_dev(c["force"]))
    assert info["status"] == 0
    ctx.close()
