"""K units of wide blocks, read from the grid that a call is launched with: about 512 inputs up to K = 4096 where the
launch then has at most 230 base blocks, without adapters 320, else about 1024 below 210 blocks of 2048 inputs, else
2048 (both sides of every line were timed, see unit_of).  What a workspace is sized for is never less."""
import pytest

import paper_2604_18655_amd as lib
from test_shrink_tiles_rule import grid_x, shrink_blocks


@pytest.mark.parametrize("K,N,adapters,M,tiles,units", [
    (1024, 4096, 8, 200, 1, 2),           # 112 blocks, 224 after the cut
    (1152, 3194, 1, 281, 1, 1),           # 117 and 234
    (4096, 2672, 1, 104, 1, 4),           # 44 and 352: units of 1024 inputs
    (4096, 3354, 1, 45, 1, 8),            # 28 and 224
    (2048, 5120, 0, 100, 0, 4),           # 80 and 320, no adapters
    (2048, 5121, 0, 100, 0, 2),           # 84 and 336
    (4224, 256, 0, 40, 0, 4),             # above K = 4096: units of 1024
    (640, 256, 0, 40, 0, 1),              # five super-steps: not cut
    (768, 256, 0, 40, 0, 2),
    (2048, 14336, 0, 100, 0, 1),          # 224 blocks of 2048 inputs
])
def test_units_of_a_projection(K, N, adapters, M, tiles, units):
    rows = -(-M // 32)
    blocks = grid_x([(K, N)], adapters, 16, M)
    if adapters:
        blocks -= shrink_blocks([(K, N)], adapters, 16, M, tiles)
    assert blocks == -(-(-(-N // 256) * units) // 8) * 8 * rows


@pytest.mark.parametrize("M", [33, 64, 65, 128, 300])
@pytest.mark.parametrize("K", [128, 640, 1024, 2176, 4096, 4224, 14336])
@pytest.mark.parametrize("N", [2048, 4096, 8192])                     # whole runs of eight blocks
def test_partial_tiles_fit_the_workspace(K, N, M):
    """Partial tiles (fp32, the rows filled up to chunks of 64) of every unit but one; half of a workspace is theirs."""
    p = lib.Proj(K, N, 32, None)
    units = lib.layer_step_plan([p], M)["grid_x"] // -(-M // lib.layer_step_block_rows([p], M)) // (N // 256)
    assert units >= 1
    assert lib.workspace_bytes([p], M) >= 2 * (units - 1) * N * -(-M // 64) * 64 * 4
