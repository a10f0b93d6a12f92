"""The tree apply's last steps as one dense block (more cells than the
one-workgroup tail holds) and the mid steps' ranges below it, against the
oracle's tree solve: the smallest system that has the block, ordinary ones
with one and with two mid ranges, a batch whose block spans several trees, and
one with more trees ending in the last step than the block holds."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from workloads import sphere_cluster, batched_instance

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


@pytest.mark.parametrize("n", [2201, 7001, 120_011, 300_007])
def test_top_block_matches_oracle(ctx, n):
    c = sphere_cluster(n, 51)
    g = ctx.collide(to_dev(c["pos"]), to_dev(c["radius"]))
    M = ctx.factor_tree(g, ctx.build_tree(g))
    info = M.info()
    assert 0 < info["tail_step"] < info["steps"] and sum(info["step_sizes"][info["tail_step"]:]) <= 512
    b = np.random.default_rng(n).normal(size=(n, 3))
    og = O.collide(c["pos"], c["radius"])
    zo = O.tree_solve(O.tree_factor(og, O.build_tree(og)), b)
    z = ctx.prec_apply(M, to_dev(b))
    assert np.linalg.norm(host(z) - zo) <= 1e-10 * np.linalg.norm(zo)
    assert torch.equal(z, ctx.prec_apply(M, to_dev(b)))   # fixed summation order
    A = ctx.assemble_gamma(g)
    v, i32 = ctx.pcg_solve(A, M, to_dev(c["force"]), precision="f32ir", inner_rtol=1e-4)
    assert i32["status"] == 0 and i32["relres_true"] <= 1.0001e-8


@pytest.mark.parametrize("sizes", [[3000, 9, 500, 2500, 1], [6] * 700])
def test_top_block_over_several_trees(ctx, sizes):
    parts = [batched_instance(k + 61, n_override=s) for k, s in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pos, R = (np.concatenate([p[k] for p in parts]) for k in ("pos", "radius"))
    g = ctx.collide_batched(off, to_dev(pos), to_dev(R))
    M = ctx.factor_tree(g, ctx.build_tree(g))
    b = np.random.default_rng(5).normal(size=(int(off[-1]), 3))
    z = host(ctx.prec_apply(M, to_dev(b)))
    for k, p in enumerate(parts):
        og = O.collide(p["pos"], p["radius"])
        zo = O.tree_solve(O.tree_factor(og, O.build_tree(og)), b[off[k]:off[k + 1]])
        assert np.linalg.norm(z[off[k]:off[k + 1]] - zo) <= 1e-10 * np.linalg.norm(zo), k
