"""The one-workgroup tail where the sweeps have one: level schedules, light
subtrees, and small contraction factors solved outside the one-workgroup solve.
Where the tail begins (tail_max) changes no bit as long as the first elimination
step stays outside it.  A factor has a tail if the step it begins
at follows tail_max; the dense block of larger contraction factors does not."""
import pytest
import torch

from workloads import sphere_cluster

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import to_dev  # noqa: E402

# cells, schedule, light_height, the tail_max values (none reaching the first step)
KINDS = [(9000, "level", 0, (2200, 300, 0)), (20011, "contract", 8, (2200, 500, 0)), (2100, "contract", 0, (900, 200, 0))]


@pytest.fixture()
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = P.Context()
    c.tune("small_solve", 0)
    yield c
    c.close()


def _system(ctx, n, seed):
    c = sphere_cluster(n, seed)
    g = ctx.collide(to_dev(c["pos"]), to_dev(c["radius"]))
    return g, ctx.assemble_gamma(g), ctx.build_tree(g), to_dev(c["force"])


def _factor(ctx, g, T, schedule, light, tail):
    ctx.tune("light_height", light)
    ctx.tune("tail_max", tail)
    M = ctx.factor_tree(g, T, schedule=schedule)
    info = M.info()
    assert 0 < info["tail_step"] <= info["steps"] and sum(info["step_sizes"][info["tail_step"]:]) <= tail
    return M, info["tail_step"]


def _same(a, b):
    for (va, ia), (vb, ib) in zip(a, b):
        assert ia == ib and torch.equal(va, vb)


@pytest.mark.parametrize("n,schedule,light,tails", KINDS)
def test_tail_max_changes_no_bit(ctx, n, schedule, light, tails):
    g, A, T, F = _system(ctx, n, 61)
    b = torch.randn_like(F)
    runs, starts = [], []
    for tail in tails:
        M, start = _factor(ctx, g, T, schedule, light, tail)
        starts.append(start)
        runs.append((ctx.prec_apply(M, b), [ctx.pcg_solve(A, M, F, check_every=4),
                                            ctx.pcg_solve(A, M, F, precision="f32ir", inner_rtol=1e-4)]))
    assert starts == sorted(set(starts))   # three different tails
    for z, r in runs[1:]:
        assert torch.equal(z, runs[0][0])
        _same(r, runs[0][1])
