"""Grouped shrink blocks (more than 16 rows): row tiles with one row and with sixteen, more tiles than a block
takes at a time, waves with fewer k-steps than others, ranks that end inside a block of 16, rows without
adapter, K units of 512 inputs, against the oracle.  Bars as everywhere: 5e-3 of max|y_ref| with bf16 outputs
(rounding alone reaches 2^-8), 2e-4 with fp32 outputs, 5e-3 of the LoRA term's own maximum."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check_linear, random_problem

pytestmark = pytest.mark.gpu


def rows_of(kind, M, n_ad):
    if kind == "one":
        return np.zeros(M, np.int32)                               # full tiles
    if kind == "each":
        return (np.arange(M) % n_ad).astype(np.int32)              # as many tiles as adapters
    if kind == "seventeen":
        return (np.arange(M) // 17 % n_ad).astype(np.int32)        # a full tile and one of a row
    rows = np.random.default_rng(M).integers(-1, n_ad, size=M).astype(np.int32)
    rows[: M // 2] = -1                                            # whole chunks without adapter
    return rows


@pytest.mark.parametrize("kind", ["one", "each", "seventeen", "absent"])
@pytest.mark.parametrize("M,K,N,G,r,n_ad", [(17, 128, 19264, 32, 8, 3),        # tile blocks; one k-step per wave
                                            (32, 640, 19264, 64, 40, 32),      # 512 inputs per K chunk, 5 k-steps each
                                            (33, 128, 70, 32, 16, 33),         # wide blocks; 128 inputs: two of the eight waves share a tile
                                            (190, 128, 200, 64, 24, 17),       # several tiles of one batch
                                            (150, 256, 130, 64, 24, 9),        # 256 inputs: four of the eight waves share a tile
                                            (300, 256, 4000, 128, 8, 3),
                                            (64, 2176, 321, 128, 24, 64),      # 17 super-steps: units of 512 inputs
                                            (65, 4224, 64, 32, 8, 5),          # two chunks, the second of one row
                                            (127, 1152, 130, 64, 72, 16),
                                            (200, 8320, 64, 32, 16, 64)])      # 2048 inputs per K chunk
def test_row_tiles(gpu, kind, M, K, N, G, r, n_ad):
    prob = random_problem(M + K, K, N, G, r, n_ad)
    x = wl.f32_to_bf16_bits(np.random.default_rng(K).standard_normal((M, K)).astype(np.float32))
    check_linear(gpu, prob, x, rows_of(kind, M, n_ad), f"{kind} M{M} K{K} N{N} G{G} r{r}")


@pytest.mark.parametrize("n_proj,N,M,block_rows", [(1, 256, 40, 32), (1, 256, 150, 32),      # one tile per block
                                                   (12, 256, 40, 32), (30, 256, 40, 32),     # four: ten blocks for 40 tiles ...
                                                   (9, 256, 150, 32),                        # ... and three chunks of up to 44
                                                   (120, 256, 40, 32), (16, 256, 150, 32), (120, 256, 150, 32),   # eight
                                                   (16, 4096, 192, 64)])                     # sixteen: blocks of 64 rows, three per chunk
def test_tiles_per_block(gpu, n_proj, N, M, block_rows):
    lib, device, torch = gpu
    K, n_ad = 256, 40
    prob = random_problem(7, K, N, 32, 16, n_ad)
    p = device.upload_problem(prob)
    assert lib.layer_step_block_rows([p] * n_proj, M) == block_rows
    x = device.to_device(wl.f32_to_bf16_bits(np.random.default_rng(1).standard_normal((M, K)).astype(np.float32)))
    ra = torch.from_numpy(rows_of("each", M, n_ad)).cuda()
    alone = device.alloc_y(M, N, 1)
    lib.linear(p, x, ra, M, alone, 1, device.alloc_workspace([p], M))
    ys = [device.alloc_y(M, N, 1) for _ in range(n_proj)]
    lib.layer_step([p] * n_proj, [x] * n_proj, ys, ra, M, 1, device.alloc_workspace([p] * n_proj, M))
    torch.cuda.synchronize()
    # sums of 256 products in another order, fp32: far below 2e-4 of the largest
    bar = 2e-4 * float(alone.abs().max())
    assert all(float((y - alone).abs().max()) <= bar for y in ys)
