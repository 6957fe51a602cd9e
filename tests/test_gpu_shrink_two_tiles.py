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
    (128, 4442, 128, 128, 2, 341, 8),     # 128 inputs, eight waves: 198 base blocks, four tiles would make 96 more
    (128, 3779, 128, 64, 2, 299, 4),
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


def layer(h, kv, f):
    return [(h, h), (h, kv), (h, kv), (h, h), (h, f), (h, f), (f, h)]


LAYERS = [                                # projections, group, rank, adapters, rows, row tiles per block (all in blocks of eight waves)
    (layer(512, 256, 1536), 128, 16, 11, 177, 2),
    (layer(768, 384, 1536) * 2, 32, 32, 8, 37, 2),
    (layer(768, 256, 2048), 32, 32, 8, 235, 4),         # two tiles would make 384
    (layer(512, 256, 896), 32, 32, 3, 188, 4),          # no input of 1024
    (layer(512, 192, 1920), 32, 8, 4, 117, 1),
]


@pytest.mark.parametrize("shapes,G,rank,adapters,M,tiles", LAYERS)
def test_grid_of_several_projections(shapes, G, rank, adapters, M, tiles):
    more = grid_x(shapes, adapters, rank, M) - grid_x(shapes, 0, rank, M)
    assert more == shrink_blocks(shapes, adapters, rank, M, tiles)


@pytest.mark.gpu
@pytest.mark.parametrize("shapes,G,rank,adapters,M,tiles", LAYERS)
def test_outputs_of_several_projections(gpu, shapes, G, rank, adapters, M, tiles):
    """As each projection by itself, up to the order of fp32 sums (2e-4 of the largest output, far above it)."""
    lib, device, torch = gpu
    rng = np.random.default_rng(M)
    ra = torch.from_numpy(rng.integers(-1, adapters, size=M).astype(np.int32)).cuda()
    projs, xs, ys, alone = [], [], [], []
    for i, (K, N) in enumerate(shapes):
        projs.append(device.upload_problem(random_problem(i, K, N, G, rank, adapters)))
        xs.append(device.to_device(wl.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))))
        ys.append(device.alloc_y(M, N, lib.Y_FP32))
        alone.append(device.alloc_y(M, N, lib.Y_FP32))
        lib.linear(projs[i], xs[i], ra, M, alone[i], lib.Y_FP32, device.alloc_workspace([projs[i]], M))
    lib.layer_step(projs, xs, ys, ra, M, lib.Y_FP32, device.alloc_workspace(projs, M))
    torch.cuda.synchronize()
    for y, one in zip(ys, alone):
        assert float((y - one).abs().max()) <= 2e-4 * float(one.abs().max())
