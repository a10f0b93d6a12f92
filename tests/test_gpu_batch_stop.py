"""Clusters of a batch that stop at different iterations (no force, a start that
is the solution, sizes far apart): the others' bits do not depend on them, a
second solve on the same handles repeats the first, and a recorded batch replays
with the same bits."""
import numpy as np
import pytest
import torch

from workloads import batched_instance

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import to_dev  # noqa: E402

SIZES = [9000, 30, 700, 2500, 5, 9000, 260]


@pytest.fixture()
def batch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context()
    parts = [batched_instance(k + 71, n_override=s) for k, s in enumerate(SIZES)]
    off = np.concatenate([[0], np.cumsum(SIZES)]).astype(np.int64)
    pos, R, F = (to_dev(np.concatenate([p[k] for p in parts])) for k in ("pos", "radius", "force"))
    g = ctx.collide_batched(off, pos, R)
    A = ctx.assemble_gamma(g)
    yield ctx, off, pos, R, F, A, {"tree": ctx.factor_tree(g, ctx.build_tree(g)), "jacobi": ctx.make_jacobi(A),
                                   "none": None}
    ctx.close()


@pytest.mark.parametrize("prec", ["tree", "jacobi", "none"])
def test_stopped_clusters_change_nothing(batch, prec):
    ctx, off, _, _, F, A, M = batch
    ref, iref = ctx.pcg_solve_batched(A, M[prec], off, F)
    assert len({i["iters"] for i in iref}) > 3 and all(i["status"] == 0 for i in iref)
    Fz = F.clone()
    Fz[off[0]:off[1]] = 0
    Fz[off[3]:off[4]] = 0
    x0 = torch.zeros_like(F)
    x0[off[2]:off[3]] = ref[off[2]:off[3]]
    for _ in range(2):
        v, info = ctx.pcg_solve_batched(A, M[prec], off, Fz, x0.clone(), use_x0=True)
        for k, i in enumerate(info):
            s = slice(off[k], off[k + 1])
            if k in (0, 3):
                assert i["iters"] == 0 and not v[s].any()
            elif k == 2:
                assert i["iters"] == 0 and torch.equal(v[s], ref[s])
            else:   # (from a start of zeros the first residual is F - Gamma 0: the same bits)
                assert i["iters"] == iref[k]["iters"] and torch.equal(v[s], ref[s]), k


def test_recorded_batch_replays(batch):
    ctx, off, pos, R, F, A, M = batch
    Fz = F.clone()
    Fz[off[0]:off[1]] = 0
    ref, _ = ctx.pcg_solve_batched(A, M["tree"], off, Fz)
    step, v = P.Step(ctx), torch.zeros_like(F)
    step.record_batched(off, pos, R, Fz, v)
    for _ in range(4):
        v.fill_(7.0)
        torch.cuda.synchronize()
        step.replay()
        assert torch.equal(v, ref)
        ctx.pcg_solve_batched(A, M["jacobi"], off, F)   # eager work between the replays
