"""Weights with and without codes -8, which the blob stores in two ways (a flag per blob): every block
family against the oracle, the only -8 in the first or the last place of the weight, or everywhere.
Bars as everywhere: 5e-3 of max|y_ref| with bf16 outputs (rounding alone reaches 2^-8), 2e-4 with fp32 outputs."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_util import TOL_F32, check_linear, random_problem, rel_err

pytestmark = pytest.mark.gpu

PLACES = ("none", "first", "last", "many")


def problem(place, K, N, G, r=8, n_ad=3):
    prob = random_problem(K + N + G, K, N, G, r, n_ad)
    rng = np.random.default_rng(K + N)
    codes = rng.integers(-7, 8, size=(N, K)).astype(np.int8)
    if place == "first":
        codes[0, 0] = -8
    elif place == "last":
        codes[-1, -1] = -8
    elif place == "many":
        codes[rng.random((N, K)) < 0.3] = -8
    return wl.Problem(prob.shape, wl.pack_nibbles(codes), prob.scales, prob.lora_a, prob.lora_b), codes


def rows_and_x(M, K, n_ad=3):
    rng = np.random.default_rng(M)
    # (rows with a mean: an offset of the codes that was not taken out would show)
    x = wl.f32_to_bf16_bits((rng.standard_normal((M, K)) + 2.0).astype(np.float32))
    return x, rng.integers(-1, n_ad, size=M).astype(np.int32)


@pytest.mark.parametrize("place", PLACES)
@pytest.mark.parametrize("M,K,N,G", [(1, 640, 70, 32), (8, 384, 130, 64), (13, 2176, 64, 128),    # tile blocks of up to 16 rows
                                     (9, 128, 70, 32), (16, 1024, 130, 64), (27, 640, 64, 128),   # units of at most two super-steps per wave
                                     (12, 1152, 70, 64),                                          # and of one more
                                     (20, 128, 19264, 32), (32, 256, 19264, 128),                 # tile blocks of up to 32 rows
                                     (40, 384, 321, 32), (70, 256, 130, 64), (64, 640, 64, 128)])  # wide blocks of 32 rows
def test_every_code(gpu, place, M, K, N, G):
    prob, _ = problem(place, K, N, G)
    x, rows = rows_and_x(M, K)
    check_linear(gpu, prob, x, rows, f"{place} M{M} K{K} N{N} G{G}")


@pytest.mark.parametrize("place", PLACES)
@pytest.mark.parametrize("G", [32, 64, 128])
def test_blocks_of_64_rows_and_int8_rows(gpu, place, G):
    lib, device, torch = gpu
    K, N, M, n = 384, 512, 250, 128
    prob, _ = problem(place, K, N, G)
    x, rows = rows_and_x(M, K)
    p, ra = device.upload_problem(prob), torch.from_numpy(rows).cuda()
    assert lib.layer_step_block_rows([p] * n, M) == 64
    ref = oracle.linear(prob.wq, prob.scales, G, prob.lora_a, prob.lora_b, prob.shape.alpha, x, rows)
    ys = [device.alloc_y(M, N, 1) for _ in range(n)]
    lib.layer_step([p] * n, [device.to_device(x)] * n, ys, ra, M, 1, torch.zeros(lib.workspace_bytes([p] * n, M), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert all(torch.equal(ys[0], y) for y in ys[1:])
    assert rel_err(device.y_to_numpy(ys[0]), ref) <= TOL_F32
    for rows8 in (4, M):                                  # int8 rows: blocks of 32 rows and of 64
        xq, s = wl.make_x_int8(rows8, K, 5, 0, 0)
        ref = oracle.linear_a8(prob.wq, prob.scales, G, prob.lora_a, prob.lora_b, prob.shape.alpha, xq, float(s), rows[:rows8])
        ys = [device.alloc_y(rows8, N, 1) for _ in range(n)]
        ws = torch.zeros(lib.a8_workspace_bytes([p] * n, rows8), dtype=torch.uint8, device="cuda")
        lib.LayerPlanA8([p] * n, [torch.from_numpy(xq).cuda()] * n, [float(s)] * n, ys, ra[:rows8].contiguous(), rows8, 1, ws).run()
        torch.cuda.synchronize()
        assert rel_err(device.y_to_numpy(ys[-1]), ref) <= TOL_F32


def test_blob_of_another_weight_is_overwritten_whole(gpu):
    """A blob that held codes -8 takes a weight without any, and the other way round: the codes come back."""
    lib, device, torch = gpu
    K, N, G = 256, 130, 32
    blob = torch.empty(lib.blob_bytes(K, N, G), dtype=torch.uint8, device="cuda")
    for place in ("many", "none", "last", "none"):
        prob, codes = problem(place, K, N, G)
        lib.prepack(K, N, G, torch.from_numpy(prob.wq).cuda(), device.to_device(prob.scales), blob)
        out = torch.empty((N, K), dtype=torch.int8, device="cuda")
        lib.unpack(lib.Proj(K, N, G, blob), out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), codes)
