"""The tile-walking kernels (initial matrix, projection, divergence check) at the edges of their
tiles: units of 128 bits, 1,024 or 256 to a tile of the initial matrix, 2,048 (or 256 rows) to one of the
projection, 2,048 per turn of the check."""
import numpy as np
import pytest
import torch

import paper_2008_12336_amd as G
from oracle import gosh_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# a row of one unit, rows that do not divide a tile, the largest row; 1 row, a tile less one row,
# a whole tile, one row more, several tiles
SHAPES = [(d, n) for d in (4, 36, 100, 128, 260, 508, 512)
          for t in [min(256, 2048 // (d // 4))] for n in (1, t - 1, t, t + 1, 5 * t + 3)]


@pytest.mark.parametrize("d,n", SHAPES)
def test_initial_rows_and_projection_bit_for_bit(d, n):
    seed, level = 0x1234567890ABCDEF, 3
    M = torch.full((n, d), 7.0, device=DEV)
    G.gosh_init_embedding(M, seed, level)
    assert np.array_equal(M.cpu().numpy(), O.init_embedding(n, d, seed, level))
    coarse_n = max(1, n // 3)
    rng = np.random.default_rng(n * 1000 + d)
    coarse = rng.standard_normal((coarse_n, d)).astype(np.float32)
    cmap = rng.integers(0, coarse_n, n).astype(np.int32)
    cmap[rng.integers(0, n)] = -1        # names no coarse vertex: a row of zeros
    cmap[rng.integers(0, n)] = coarse_n  # the same
    fine = torch.full((n + 1, d), 7.0, device=DEV)
    G.gosh_project(torch.from_numpy(coarse).to(DEV), torch.from_numpy(cmap).to(DEV), fine[:n])
    ok = (cmap >= 0) & (cmap < coarse_n)
    want = np.where(ok[:, None], coarse[np.where(ok, cmap, 0)], np.float32(0))
    got = fine.cpu().numpy()
    assert np.array_equal(got[:n], want)
    assert (got[n] == 7.0).all()  # nothing past the last row


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


@pytest.mark.parametrize("d,mb", [(36, 127), (36, 129), (128, 200), (508, 140)])
def test_projection_of_matrices_around_the_memory_side_cache(d, mb):
    """From 128 MB on the rows are written past the caches."""
    n, coarse_n = mb * (1 << 20) // (4 * d) + 1, 70_001
    g = torch.Generator(device=DEV).manual_seed(d)
    coarse = torch.randn(coarse_n, d, generator=g, device=DEV)
    cmap = torch.randint(0, coarse_n, (n,), generator=g, device=DEV, dtype=torch.int32)
    fine = torch.full((n + 1, d), 7.0, device=DEV)
    G.gosh_project(coarse, cmap, fine[:n])
    assert torch.equal(fine[:n], coarse[cmap.long()]) and (fine[n] == 7.0).all()


def test_check_of_tiles_shared_unevenly():
    """301 tiles for 256 workgroups."""
    M = torch.zeros(300 * 2048 + 5, 4, device=DEV)
    for at in (0, 255 * 2048, 256 * 2048 + 1, 300 * 2048 + 4):
        M[at, 3] = float("inf")
    M[256 * 2048, 0] = -5.0
    assert G.gosh_matrix_check(M) == (5.0, 4)


@pytest.mark.parametrize("tiles", [2047, 2048, 2053, 4000])
def test_check_of_tiles_beyond_its_workgroups(tiles):
    """512 workgroups from 2,048 tiles on."""
    M = torch.zeros((tiles - 1) * 2048 + 7, 4, device=DEV)
    M.view(-1)[:: 2048 * 4] = 2.0  # the first float of every tile
    at = [(tiles - 1) * 2048 + 6, 1536 * 2048, 512 * 2048 - 1, 0]
    for row in at:
        M[row, 3] = float("nan")
    M[1024 * 2048 + 5, 2] = -9.0
    assert G.gosh_matrix_check(M) == (9.0, len(at))
    M.fill_(float("inf"))
    assert G.gosh_matrix_check(M) == (0.0, M.numel())


@pytest.mark.parametrize("d,mb", [(4, 257), (8, 257), (100, 255), (100, 257), (260, 300), (512, 300),
                                  (4, 321), (8, 321), (100, 319), (100, 321), (260, 340), (512, 340)])
def test_initial_rows_of_matrices_around_a_cache(d, mb):
    """More than 320 MB are written by other tiles (rows of one unit excepted)."""
    n = mb * (1 << 20) // (4 * d) + 1
    M = torch.full((n + 1, d), 7.0, device=DEV)
    G.gosh_init_embedding(M[:n], 0x1234567890ABCDEF, 3)
    assert (M[n] == 7.0).all()
    assert np.array_equal(M[:n].cpu().numpy(), O.init_embedding(n, d, 0x1234567890ABCDEF, 3))
