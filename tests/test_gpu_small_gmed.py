"""The tree preconditioner with a friction against the medium that is tiny
beside the friction between cells: the pivot of a tree's root is then tiny too,
and the dense block over the last vertices keeps the roots apart from the rest.
The solve takes the iterations of the oracle's (two correct FP64 runs differ by
about 1 % in these counts, 5 % is allowed), FP32 refinement converges, and the
apply of a batch, whose block mixes the trees' vertices, is each tree's own."""
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


@pytest.mark.parametrize("n,g_med", [(3000, 1e-11), (3000, 1e-13), (9000, 1e-9), (9000, 1e-11)])
def test_iterations_at_small_medium_friction(ctx, n, g_med):
    c = sphere_cluster(n, 4)
    F = c["force"] - c["force"].mean(0)   # no net force: the velocities stay of order 1
    g = ctx.collide(to_dev(c["pos"]), to_dev(c["radius"]))
    A, T = ctx.assemble_gamma(g, g_med=g_med), ctx.build_tree(g)
    M = ctx.factor_tree(g, T, g_med=g_med)
    _, info = ctx.pcg_solve(A, M, to_dev(F))
    og = O.collide(c["pos"], c["radius"])
    _, io = O.pcg(O.assemble(og, g_med=g_med), F, "tree", O.tree_factor(og, O.build_tree(og), g_med=g_med))
    assert info["status"] == 0 and abs(info["iters"] - io.iters) <= 0.05 * io.iters, (info["iters"], io.iters)


def test_f32_refinement_at_small_medium_friction(ctx):
    c = sphere_cluster(3000, 4)
    F = to_dev(c["force"] - c["force"].mean(0))
    g = ctx.collide(to_dev(c["pos"]), to_dev(c["radius"]))
    A, T = ctx.assemble_gamma(g, g_med=1e-11), ctx.build_tree(g)
    M = ctx.factor_tree(g, T, g_med=1e-11)
    _, info = ctx.pcg_solve(A, M, F, precision="f32ir", inner_rtol=1e-4, check=False)
    assert info["status"] == 0 and info["relres_true"] <= 1.0001e-8


@pytest.mark.parametrize("sizes", [[2300], [3000, 9, 500, 2500, 1], [40] * 60])
@pytest.mark.parametrize("g_med", [1e-3, 1e-6])
def test_apply_with_the_roots_apart(ctx, sizes, g_med):
    """A root's pivot carries a relative error of about 1e-16 times the ratio
    of the frictions over the tree's cells: at most 1e5 here, and a few such
    roundings."""
    parts = [batched_instance(k + 31, n_override=s) for k, s in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pos, R = (np.concatenate([p[k] for p in parts]) for k in ("pos", "radius"))
    g = ctx.collide_batched(off, to_dev(pos), to_dev(R))
    M = ctx.factor_tree(g, ctx.build_tree(g), g_med=g_med)
    b = np.random.default_rng(7).normal(size=(int(off[-1]), 3))
    zt = ctx.prec_apply(M, to_dev(b))
    assert torch.equal(zt, ctx.prec_apply(M, to_dev(b)))
    z = host(zt)
    for k, p in enumerate(parts):
        og = O.collide(p["pos"], p["radius"])
        zo = O.tree_solve(O.tree_factor(og, O.build_tree(og), g_med=g_med), b[off[k]:off[k + 1]])
        assert np.linalg.norm(z[off[k]:off[k + 1]] - zo) <= 1e-9 * np.linalg.norm(zo), k
