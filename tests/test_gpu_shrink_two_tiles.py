"""Row tiles per grouped shrink block where launches are short or inputs are long: the grid, and outputs against the
oracle in blocks of eight and of four waves, with a last block of one tile and rows without adapter."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check_linear, random_problem
from test_shrink_tiles_rule import grid_x, shrink_blocks


CASES = [                                 # inputs, outputs, group, rank, adapters, rows, row tiles per block
    (2688, 1103, 64, 128, 4, 251, 2),     # eight waves: two tiles fit
    (2688, 457, 128, 64, 20, 255, 4),     # eight waves: two tiles are too many blocks
    (3456, 865, 128, 64, 5, 72, 2),
    (1152, 4261, 64, 128, 7, 65, 4),      # eight waves: one tile would make more than 160
    (4480, 470, 64, 32, 5, 268, 2),
    (640, 1399, 64, 64, 2, 354, 1),
    (2432, 9000, 64, 64, 4, 130, 2),      # four waves
    (12928, 4198, 64, 64, 23, 56, 4),     # four waves: two tiles would make 312
    (4480, 5658, 64, 24, 19, 302, 4),     # blocks of 64 rows
]


@pytest.mark.parametrize("K,N,G,rank,adapters,M,tiles", CASES)
def test_grid(K, N, G, rank, adapters, M, tiles):
    more = grid_x([(K, N)], adapters, rank, M) - grid_x([(K, N)], 0, rank, M)
    assert more == shrink_blocks([(K, N)], adapters, rank, M, tiles)


@pytest.mark.gpu
@pytest.mark.parametrize("K,N,G,rank,adapters,M,tiles", CASES)
def test_outputs(gpu, K, N, G, rank, adapters, M, tiles):
    rng = np.random.default_rng(M)
    x = wl.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
    rows = rng.integers(-1, adapters, size=M).astype(np.int32)
    check_linear(gpu, random_problem(K + N, K, N, G, rank, adapters), x, rows, f"K{K} N{N} r{rank} a{adapters} M{M}")
