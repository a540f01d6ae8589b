"""The GEMM tiles' operand loads, address by address: every 16-byte chunk that a
thread loads lies inside its operand, for every tile of the dispatch, at partial
last tiles and at K that is no multiple of a K step."""
import numpy as np
import pytest

TK = 64
# (waves over channels, over tokens, fragments of 16 channels, of 16 tokens a
# wave, K bytes a step)
TILES = [(2, 2, 2, 2, 64), (1, 1, 4, 4, 64), (2, 2, 4, 2, 64), (3, 2, 4, 4, 64), (3, 1, 4, 4, 64),
         (2, 4, 4, 2, 64), (4, 2, 4, 4, 64), (6, 1, 2, 1, 64), (3, 4, 4, 2, 64), (8, 1, 2, 1, 64),
         (4, 2, 4, 2, 64), (6, 1, 4, 1, 64), (6, 2, 4, 2, 64), (6, 2, 4, 2, 128)]


def chunk_ends(rows, tile_rows, threads, cpr, K, fixed=True):
    """End offsets of the 16-byte loads of the last tile of an operand of `rows`
    rows of K bytes."""
    base = (rows - 1) // tile_rows * tile_rows
    tid = np.arange(threads)[:, None, None]
    i = np.arange(-(-tile_rows * cpr // threads))[None, :, None]
    kb = np.arange(-(-K // (16 * cpr)))[None, None, :] * 16 * cpr
    divides = tile_rows * cpr % threads == 0
    last = tile_rows * cpr - cpr + tid % cpr if fixed and not divides else tile_rows * cpr - 1
    c = np.minimum(tid + i * threads, last)
    col = c % cpr * 16
    src = np.minimum(base + c // cpr, rows - 1) * K + (np.minimum(col, K - 16) if fixed else col)
    kofs = (tid + i * threads) % cpr * 16
    ok = (kb + kofs < K) if K % (16 * cpr) else np.ones_like(kb + kofs, bool)
    return src + np.where(ok, kb, 0) + 16


@pytest.mark.parametrize("tile", TILES)
def test_operand_loads_stay_inside(tile):
    wn, wm, fi, fj, kstep = tile
    threads, cpr = 64 * wn * wm, kstep // 16
    assert threads % cpr == 0
    for tile_rows in (16 * fi * wn, 16 * fj * wm):
        for rows in (1, 16, tile_rows - 1, tile_rows, tile_rows + 1, 3 * tile_rows - 16):
            for K in (16, 32, 48, 64, 80, 112, 128, 208, 784):
                if rows > 0 and (kstep == 64 or K % kstep == 0):
                    ends = chunk_ends(rows, tile_rows, threads, cpr, K)
                    assert 16 <= ends.min() and ends.max() <= rows * K, (rows, K)


def test_clamped_chunk_would_run_past():
    """Clamping the chunk, not its row, or a column past K reads up to 48 bytes
    past the operand."""
    assert chunk_ends(64, 64, 192, 4, 80, fixed=False).max() > 64 * 80
    assert chunk_ends(64, 64, 256, 4, 16, fixed=False).max() == 64 * 16 + 48
