"""Collide with a cell far from all others: the grid is enlarged until its cells
can be numbered, and the contacts are the oracle's."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from workloads import sphere_cluster

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import host, to_dev  # noqa: E402


@pytest.mark.parametrize("n,far", [(300, 1e7), (300, 1e13), (9001, 1e5), (9001, 1e11)])
def test_far_cell(n, far):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = sphere_cluster(n, 3)
    pos = c["pos"].copy()
    pos[n // 2] = (far, -far, 0.5 * far)
    ctx = P.Context()
    e = ctx.graph_export(ctx.collide(to_dev(pos), to_dev(c["radius"])))
    og = O.collide(pos, c["radius"], method="brute")   # (its own cell list cannot span the box)
    assert np.array_equal(host(e["ei"]), og.ei) and np.array_equal(host(e["ej"]), og.ej)
    assert np.array_equal(host(e["w"]), og.w)
    ctx.close()
