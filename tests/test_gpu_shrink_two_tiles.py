"""Two row tiles per grouped shrink block (long inputs, launches that have room for the blocks): the grid, and outputs
against the oracle in blocks of eight and of four waves, with a last block of one tile and rows without adapter."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check_linear, random_problem
from test_shrink_tiles_rule import grid_x, shrink_blocks


@pytest.mark.parametrize("K,N,adapters,rank,M", [
    (2688, 457, 20, 64, 255),             # 128 base blocks, eight waves
    (2688, 1103, 4, 128, 251),            # 256, four waves
])
def test_two_tiles(K, N, adapters, rank, M):
    more = grid_x([(K, N)], adapters, rank, M) - grid_x([(K, N)], 0, rank, M)
    assert more == shrink_blocks([(K, N)], adapters, rank, M, 2)


@pytest.mark.gpu
@pytest.mark.parametrize("K,N,G,rank,adapters,M", [
    (2688, 457, 128, 64, 20, 255),
    (2688, 1103, 64, 128, 4, 251),
])
def test_outputs(gpu, K, N, G, rank, adapters, M):
    rng = np.random.default_rng(M)
    x = wl.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
    rows = rng.integers(-1, adapters, size=M).astype(np.int32)
    check_linear(gpu, random_problem(K + N, K, N, G, rank, adapters), x, rows, f"K{K} N{N} r{rank} a{adapters} M{M}")
