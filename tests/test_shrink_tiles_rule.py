"""Row tiles of a grouped shrink block from 33 rows on, read from the grid that a call is launched with: one where
all blocks find a place at once, four where they do with four, where every wave has tiles of its own or where
that makes at most 300 blocks, else 8 (16 in blocks of 64 rows).  Both sides of the lines were timed, see SHRINK_FEW_BLOCKS."""
import pytest

import paper_2604_18655_amd as lib


def grid_x(shapes, adapters, rank, M):
    projs = [lib.Proj(K, N, 32, None) for K, N in shapes]
    for p in projs:
        p.n_adapters, p.rank = adapters, rank
    return lib.layer_step_plan(projs, M)["grid_x"]


def shrink_blocks(shapes, adapters, rank, M, tiles):
    bound = min(min(M, 64), min(M, 64) // 16 + min(adapters, M, 64))
    n = 0
    for K, _ in shapes:
        chunks = max(1, min(16, K // (2048 if K > 4096 else 1024)))
        n += -(-M // 64) * -(-bound // tiles) * -(-rank // 16) * chunks
    return -(-n // 8) * 8


@pytest.mark.parametrize("shapes,adapters,rank,M,tiles", [
    ([(8192, 2048)], 8, 16, 64, 1),                 # 192 base blocks and 96
    ([(4096, 14336)], 32, 64, 64, 4),               # 448 and 576, or 144 with four tiles
    ([(4352, 5466)], 10, 32, 441, 4),               # more base blocks than places, 112 shrink blocks
    ([(4480, 12672)], 21, 16, 320, 4),              # blocks of 64 rows: 70
    ([(3328, 3563)], 2, 128, 593, 8),               # 480
    ([(3072, 12191)], 25, 32, 871, 16),             # blocks of 64 rows: 672
    ([(256, 256)], 40, 16, 150, 1),                 # what tests/test_gpu_shrink_tiles.py runs
    ([(256, 256)] * 12, 40, 16, 40, 4),
    ([(256, 256)] * 9, 40, 16, 150, 4),
    ([(256, 256)] * 16, 40, 16, 150, 8),
    ([(256, 4096)] * 16, 40, 16, 192, 16),
    ([(128, 4991)], 1, 128, 276, 4),                # a tile of 128 inputs is one wave's
    ([(128, 4991), (256, 64)], 1, 16, 40, 1),       # not of 256 inputs
])
def test_tiles_of_a_shrink_block(shapes, adapters, rank, M, tiles):
    more = grid_x(shapes, adapters, rank, M) - grid_x(shapes, 0, rank, M)
    assert more == shrink_blocks(shapes, adapters, rank, M, tiles)
