"""The spanning tree's pointer jumps and list ranking on chains: cells on a line
whose overlaps grow along it hook into one chain as long as the system, shorter
than, as long as and beyond what one pair of launches of the jumps follows (81
links), and systems around one tile of the scans (2048).  The tree is an exact
result: equal to the oracle's."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from workloads import sphere_cluster

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import host, to_dev  # noqa: E402


def _check(pos, radius):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context()
    og = O.collide(pos, radius)
    ot = O.build_tree(og)
    g = ctx.collide(to_dev(pos), to_dev(radius))
    e = ctx.graph_export(g)
    assert np.array_equal(host(e["ei"]), og.ei) and np.array_equal(host(e["w"]), og.w)
    t = {k: host(v) for k, v in ctx.tree_export(ctx.build_tree(g), len(radius)).items()}
    assert np.array_equal(t["tree_edge"], ot.tree_edge) and np.array_equal(t["parent"], ot.parent)
    assert np.array_equal(t["depth"], ot.depth)
    ctx.close()


@pytest.mark.parametrize("n", [2, 9, 10, 81, 82, 83, 84, 700, 7000])
def test_chain(n):
    pos = np.zeros((n, 3))
    pos[1:, 0] = np.cumsum(1.9 - 0.8 * np.arange(n - 1) / n)
    _check(pos, np.ones(n))


@pytest.mark.parametrize("n", [2047, 2048, 2049])
def test_scan_tiles(n):
    c = sphere_cluster(n, 61)
    _check(c["pos"], c["radius"])
