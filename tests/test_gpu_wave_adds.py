"""Atomic adds of whole rows by the wavefront (d <= 64): several rows per instruction, laid out by lane group.

Every source has one partner of its own and nothing is drawn but positives, so no row is written twice and a
concurrent epoch is the sequential one: a float added to the wrong row, column or not at all shows."""
import numpy as np
import pytest
import torch

import paper_2008_12336_amd as G
from oracle import gosh_oracle as O
from tests.test_gpu_layout import DEV, TOL, hot_degree, start_matrix, upload  # noqa: F401
from tests.util import HOT_ALL, HOT_BITMAP, last_hot_mode, rel_err

pytestmark = pytest.mark.gpu


def pairs_graph(pairs, seed):
    """2 * pairs vertices: v has v + pairs as its only neighbour, twice, once or not at all; the partners
    name themselves (no update) twice.  Rows of degree two are hot where the rule says so; a partner's must be,
    since its own turn writes it back too."""
    rng = np.random.default_rng(seed)
    deg = np.concatenate((rng.integers(0, 3, pairs), np.full(pairs, 2)))
    to = np.concatenate((np.arange(pairs, 2 * pairs), np.arange(pairs, 2 * pairs)))
    return np.concatenate(([0], np.cumsum(deg))).astype(np.int64), np.repeat(to, deg).astype(np.int32)


# lane groups of 1 to 16 lanes, full and partly used rows; 4 * 64 / LPG sources a workgroup, the last one ragged
@pytest.mark.parametrize("mode", [HOT_ALL, HOT_BITMAP])
@pytest.mark.parametrize("d", [4, 8, 12, 16, 20, 32, 36, 64])
def test_rows_added_side_by_side(d, mode, hot_degree):  # noqa: F811
    pairs = 4 * 64 + 37
    xadj, adj = pairs_graph(pairs, d)
    n = 2 * pairs
    if mode == HOT_BITMAP:
        hot_degree(2)
    g, keep = upload(n, xadj, adj, d % 8 == 0)
    want = start_matrix(n, d, 5, 1.0)
    M = torch.from_numpy(want.copy()).to(DEV)
    for epoch in range(2):
        G.gosh_train_epoch(g, M, 0, 0.3, 11, epoch)
        torch.cuda.synchronize()
        assert last_hot_mode() == mode
        O.train_epoch(xadj, adj, want, 0, 0.3, 11, epoch, 0)
    assert rel_err(M.cpu().numpy(), want) <= TOL  # (the bar of the sequential order)
