"""The product from the cells themselves (more than 8192 cells) and the brick
order it needs, against the oracle's assembled Gamma: both sides of the size
rule and of the tile shapes, rows longer than a few groups of entries, tiles
whose halo does not fit or whose distances leave the square root iteration's
range (both multiplied from global memory), sheets and threads of cells, and a
batch whose solve forms p.q per cluster in the product."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from workloads import sphere_cluster, batched_instance
from workloads.paper import hcp_sites

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


def _system(kind, n):
    rng = np.random.default_rng(n)
    if kind == "fcc":
        c = sphere_cluster(n, 71)
        return c["pos"], c["radius"]
    if kind == "hcp":
        return hcp_sites(n) + rng.normal(0, 0.15, (n, 3)), np.full(n, 0.5)
    if kind == "dense":   # ~25 contacts a cell, up to 64
        return rng.uniform(0, (n / 6.0) ** (1 / 3), (n, 3)), np.full(n, 0.5)
    if kind == "mixed":   # small cells among few large ones: halos of any size
        R = np.where(rng.random(n) < 0.01, 0.7, 0.05)
        return rng.uniform(0, (n / 8.0) ** (1 / 3), (n, 3)), R
    if kind == "sheet":
        m = int(np.ceil(np.sqrt(n)))
        g = np.stack(np.meshgrid(np.arange(m), np.arange(m), indexing="ij"), -1).reshape(-1, 2)[:n]
        return np.concatenate([0.9 * g, np.zeros((n, 1))], 1) + rng.normal(0, 0.05, (n, 3)), np.full(n, 0.5)
    pos = np.zeros((n, 3))
    pos[:, 1] = 0.9 * np.arange(n)
    return pos + rng.normal(0, 0.02, (n, 3)), np.full(n, 0.5)


@pytest.mark.parametrize("kind,n,scale,hertz", [
    ("fcc", 8192, 1.0, False), ("fcc", 8193, 1.0, False), ("hcp", 10_001, 1.0, True), ("fcc", 149_999, 1.0, False),
    ("hcp", 150_007, 1.0, True), ("dense", 9001, 1.0, False), ("mixed", 20_011, 1.0, True), ("sheet", 9999, 1.0, False),
    ("thread", 12_345, 1.0, False), ("fcc", 9000, 1e-110, False), ("hcp", 9000, 1e3, True)])
def test_tile_product_matches_oracle(ctx, kind, n, scale, hertz):
    pos, R = (np.ascontiguousarray(scale * a) for a in _system(kind, n))
    ctx.set_contact_model("hertz" if hertz else "overlap")
    g = ctx.collide(to_dev(pos), to_dev(R), 64)
    og = O.collide(pos, R, area="hertz" if hertz else "overlap")
    e = ctx.graph_export(g)
    assert np.array_equal(host(e["ei"]), og.ei) and np.array_equal(host(e["ej"]), og.ej)
    assert np.array_equal(host(e["w"]), og.w)
    A = ctx.assemble_gamma(g)
    oa = O.assemble(og)
    x = np.random.default_rng(1).normal(size=(n, 3))
    ref = O.spmv(oa, x)
    y = ctx.spmv(A, to_dev(x))
    assert np.linalg.norm(host(y) - ref) <= 1e-14 * np.linalg.norm(ref)
    assert torch.equal(y, ctx.spmv(A, to_dev(x)))
    # the diagonal blocks, formed from the cells for block Jacobi
    diag = np.stack([oa.val[oa.rowptr[i] + np.searchsorted(oa.bcol[oa.rowptr[i]:oa.rowptr[i + 1]], i)]
                     for i in range(n)])
    zo = np.linalg.solve(diag, x[:, :, None])[:, :, 0]
    z = host(ctx.prec_apply(ctx.make_jacobi(A), to_dev(x)))
    assert np.linalg.norm(z - zo) <= 1e-12 * np.linalg.norm(zo)


def test_tile_product_fp32_and_batch(ctx):
    sizes = [9000, 1, 300, 4000]
    parts = [batched_instance(k + 81, n_override=s) for k, s in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pos, R, F = (to_dev(np.concatenate([p[k] for p in parts])) for k in ("pos", "radius", "force"))
    g = ctx.collide_batched(off, pos, R)
    A = ctx.assemble_gamma(g)
    J = ctx.make_jacobi(A)
    v, infos = ctx.pcg_solve_batched(A, J, off, F)
    assert all(i["status"] == 0 and i["relres_true"] <= 1.0001e-8 for i in infos)
    for k, s in enumerate(sizes):   # against the clusters on their own (the edge form below 8193 cells)
        a, b = off[k], off[k + 1]
        gk = ctx.collide(pos[a:b].contiguous(), R[a:b].contiguous())
        Ak = ctx.assemble_gamma(gk)
        vk, ik = ctx.pcg_solve(Ak, ctx.make_jacobi(Ak), F[a:b].contiguous())
        assert abs(ik["iters"] - infos[k]["iters"]) <= 1
        if ik["iters"] == infos[k]["iters"]:
            assert float(torch.linalg.vector_norm(v[a:b] - vk) / torch.linalg.vector_norm(vk)) <= 1e-8
    # one solve over the whole batch, FP32 inside refinement
    w, i32 = ctx.pcg_solve(A, J, F, precision="f32ir", inner_rtol=1e-4)
    assert i32["status"] == 0 and i32["relres_true"] <= 1.0001e-8
