"""Clusters of a batch are independent: one with a force or a start that is not
finite is reported as such and leaves the others' bits alone.  The factor's
last vertices of all clusters share one dense block (more than 2200 cells)."""
import numpy as np
import pytest
import torch

from workloads import batched_instance

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import to_dev  # noqa: E402

SIZES = [[3000, 500, 2500, 40], [9000, 700, 1, 2500]]   # the edge and the tile product


@pytest.fixture()
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = P.Context()
    yield c
    c.close()


def _batch(ctx, sizes):
    parts = [batched_instance(k + 91, n_override=s) for k, s in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pos, R, F = (to_dev(np.concatenate([p[k] for p in parts])) for k in ("pos", "radius", "force"))
    g = ctx.collide_batched(off, pos, R)
    A = ctx.assemble_gamma(g)
    M = ctx.factor_tree(g, ctx.build_tree(g))
    info = M.info()
    assert info["tail_step"] < info["steps"] and int(off[-1]) > 2200   # the dense block is there
    return off, A, M, F


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("what", ["force", "start"])
def test_bad_cluster_leaves_the_others_alone(ctx, sizes, bad, what):
    off, A, M, F = _batch(ctx, sizes)
    x0 = 1e-3 * torch.randn_like(F)
    ref, ir = ctx.pcg_solve_batched(A, M, off, F, x0.clone(), use_x0=True)
    Fb, xb = F.clone(), x0.clone()
    (Fb if what == "force" else xb)[off[1] + 3, 1] = bad
    v, info = ctx.pcg_solve_batched(A, M, off, Fb, xb, use_x0=True, check=False)
    assert info[1]["status"] == P.ENONFINITE
    for k in (0, 2, 3):
        assert info[k]["status"] == 0 and info[k]["iters"] == ir[k]["iters"], k
        assert torch.equal(v[off[k]:off[k + 1]], ref[off[k]:off[k + 1]]), k


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("bad", [float("nan"), float("-inf")])
def test_apply_keeps_trees_apart(ctx, sizes, bad):
    off, A, M, F = _batch(ctx, sizes)
    z = ctx.prec_apply(M, F)
    Fb = F.clone()
    Fb[off[3] - 1] = bad   # the last cell of cluster 2
    zb = ctx.prec_apply(M, Fb)
    assert not torch.isfinite(zb[off[2]:off[3]]).all()
    for k in (0, 1, 3):
        assert torch.equal(zb[off[k]:off[k + 1]], z[off[k]:off[k + 1]]), k
