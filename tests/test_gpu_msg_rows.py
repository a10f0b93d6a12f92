"""The network's messages on rows of every length around the groups a row's
lanes take (6, 12, 16 entries, and rows past 16): clumps of cells that all touch
one another, lone cells and pairs, forward against the oracle.  Tolerance: every
matrix product's input is rounded to BF16 (at most 2^-9 of a value), two
products a layer behind one another and one at either end, eight in all: under
2e-2 of the outputs' norm in the worst case; 3e-2 as in the network's other
parity tests.  (The backward passes walk the rows by the same code.)"""
import numpy as np
import pytest
import torch

from oracle import mpnn as N
from oracle import oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2410_04512_amd")
from tests.gpu_util import host, to_dev  # noqa: E402


@pytest.mark.parametrize("sizes", [(1, 2, 7, 8, 13, 14), (17, 18, 6, 5, 1, 33)])
def test_messages_of_row_lengths(sizes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(11)
    # clumps in which every cell touches every other: rows of size - 1 entries
    pos = np.concatenate([np.array([20.0 * k, 0, 0]) + 0.4 * rng.normal(size=(s, 3)) for k, s in enumerate(sizes * 3)])
    R = np.full(len(pos), 1.5)
    F, vprev, v = rng.normal(size=(3, len(pos), 3))
    og = O.collide(pos, R)
    deg = np.diff(og.rowptr)
    assert set(deg) == {s - 1 for s in sizes}
    scales = (1.0, 1.0, 1.0)
    theta = N.bf16_round(N.init_params(4) + 0.02 * rng.normal(size=N.param_count()))
    ctx = P.Context()
    M = P.Mpnn(ctx)
    M.set_params(theta, *scales)
    g = ctx.collide(to_dev(pos), to_dev(R), 40)
    ee = N.entry_edges(og.rowptr, og.col, og.ei, og.ej)
    rows, e = N.edge_features(og.rowptr, og.col, og.ei, og.ej, og.w, og.u, ee, scales[2])
    _, _, out = N.loss_grad(theta, F, vprev, v, og.rowptr, og.col, e, rows, scales)
    vh = host(M.forward(g, to_dev(F), to_dev(vprev)))
    assert np.linalg.norm(vh - out) <= 3e-2 * np.linalg.norm(out)
    ctx.close()
