"""The divergence check at the edges of its tiles of 2,048 units of 128 bits."""
import pytest
import torch

import paper_2008_12336_amd as G

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

@pytest.mark.parametrize("n", [1, 255, 256, 257, 2047, 2048, 2049, 4096, 5 * 2048 + 1, 2048 * 2048 + 17])
def test_check_counts_every_entry_once(n):
    """n units of four floats: the largest finite magnitude and the number of non-finite entries,
    with marked entries at both ends of the matrix and of a tile."""
    M = torch.zeros(n, 4, device=DEV)
    M.view(-1)[:] = torch.arange(4 * n, device=DEV) % 1009
    top, bad = G.gosh_matrix_check(M)
    assert (top, bad) == (float(min(4 * n - 1, 1008)), 0)
    flat = M.view(-1)
    marks = sorted({0, 4 * n - 1, min(4 * n - 1, 4 * 2048 - 1), min(4 * n - 1, 4 * 2048)})
    for i, at in enumerate(marks):
        flat[at] = [float("nan"), float("inf"), -float("inf"), float("nan")][i % 4]
    at = 4 * n // 2 if 4 * n // 2 not in marks else None
    if at is not None:
        flat[at] = -3.0e38
    top, bad = G.gosh_matrix_check(M)
    finite = flat[torch.isfinite(flat)]
    assert bad == len(marks)
    assert top == (finite.abs().max().item() if finite.numel() else 0.0)
