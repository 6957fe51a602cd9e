"""Blocks of four column tiles from 33 rows on: two blocks of 32 rows per chunk of 64 in ordinary
launches, blocks of 64 rows in long ones.  Edges of both against the
oracle: rows around the block sizes, spare waves (column tiles not a multiple of four), units that
end on half a stage, ranks from one run of 16 to the largest, all group sizes, every output stage.
Bars as everywhere: 5e-3 of max|y_ref| with bf16 outputs (rounding alone reaches 2^-8), 2e-4 with
fp32 outputs."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_util import TOL, TOL_F32, check_linear, random_problem, rel_err

pytestmark = pytest.mark.gpu


def rows_and_x(seed, M, K, n_ad):
    rng = np.random.default_rng(seed)
    x = wl.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
    return x, rng.integers(-1, n_ad, size=M).astype(np.int32)


@pytest.mark.parametrize("K,N,G,r,n_ad,M", [
    (128, 64, 32, 8, 1, 33),          # the smallest: one super-step, three spare waves, one row in the second block
    (1408, 1408, 32, 16, 5, 64),      # 22 tiles: two spare waves; 11 super-steps in units that end on half a stage
    (2304, 321, 64, 24, 7, 65),       # a third block of 32 rows with one row; ragged last tile
    (4224, 640, 128, 128, 3, 95),     # 33 super-steps; the largest rank
    (1152, 1088, 64, 64, 40, 97),     # more adapters than rows of a block, 17 tiles
    (8320, 192, 32, 40, 2, 129),      # many K units, a rank of three runs of 16
])
def test_blocks_of_32_rows(gpu, K, N, G, r, n_ad, M):
    x, rows = rows_and_x(M, M, K, n_ad)
    assert gpu[0].layer_step_block_rows([gpu[0].Proj(K, N, G, None)], M) == 32
    check_linear(gpu, random_problem(K + N + M, K, N, G, r, n_ad), x, rows, f"K{K} N{N} G{G} r{r} a{n_ad} M{M}")


def plan_of_many(gpu, prob, xs, ys, rows, M, y_dtype, n, scales=None):
    lib, device, torch = gpu
    p = device.upload_problem(prob)
    assert lib.layer_step_block_rows([p] * n, M, scales is not None) == 64
    size = lib.a8_workspace_bytes if scales is not None else lib.workspace_bytes
    ws = torch.zeros(size([p] * n, M), dtype=torch.uint8, device="cuda")
    ra = torch.from_numpy(rows).cuda()
    if scales is not None:
        return lib.LayerPlanA8([p] * n, [xs] * n, [scales] * n, ys, ra, M, y_dtype, ws), ws
    return lib.LayerPlan([p] * n, [xs] * n, ys, ra, M, y_dtype, ws), ws


@pytest.mark.parametrize("K,N,G,r,n_ad,M,n", [
    (384, 1000, 32, 24, 5, 250, 128),     # last chunk of 58 rows, ragged last tile, three super-steps
    (256, 1100, 64, 128, 3, 225, 104),    # spare waves, the largest rank, one row over 32 in the last chunk
    (640, 512, 128, 8, 9, 512, 128),      # whole chunks and tiles
])
def test_blocks_of_64_rows(gpu, K, N, G, r, n_ad, M, n):
    lib, device, torch = gpu
    prob = random_problem(K + N + M, K, N, G, r, n_ad)
    x, rows = rows_and_x(M, M, K, n_ad)
    ref = oracle.linear(prob.wq, prob.scales, G, prob.lora_a, prob.lora_b, prob.shape.alpha, x, rows)
    dx = device.to_device(x)
    for y_dtype, tol in ((0, TOL), (1, TOL_F32)):
        ys = [device.alloc_y(M, N, y_dtype) for _ in range(n)]
        plan, ws = plan_of_many(gpu, prob, dx, ys, rows, M, y_dtype, n)
        plan.run()
        plan.run()                                       # the counters are back at zero
        torch.cuda.synchronize()
        assert lib.workspace_status(ws) == 0
        assert all(torch.equal(ys[0], y) for y in ys[1:])
        assert rel_err(device.y_to_numpy(ys[0]), ref) <= tol
    # int8 rows through the same blocks
    xq, s = wl.make_x_int8(M, K, 5, 0, 0)
    ref = oracle.linear_a8(prob.wq, prob.scales, G, prob.lora_a, prob.lora_b, prob.shape.alpha, xq, float(s), rows)
    ys = [device.alloc_y(M, N, 1) for _ in range(n)]
    plan, ws = plan_of_many(gpu, prob, torch.from_numpy(xq).cuda(), ys, rows, M, 1, n, float(s))
    plan.run()
    torch.cuda.synchronize()
    assert lib.workspace_status(ws) == 0
    assert all(torch.equal(ys[0], y) for y in ys[1:])
    assert rel_err(device.y_to_numpy(ys[0]), ref) <= TOL_F32


@pytest.mark.parametrize("M,n", [(70, 2), (500, 8)])      # blocks of 32 rows; 8 x 32 x 8 blocks of 64 rows
def test_fused_output_stage(gpu, M, n):
    lib, device, torch = gpu
    K, N, r, n_ad = 256, 8192, 16, 4
    prob = random_problem(M, K, N, 32, r, n_ad)
    x, rows = rows_and_x(M, M, K, n_ad)
    rng = np.random.default_rng(M)
    scale = rng.uniform(0.5, 2.0, M).astype(np.float32)
    res = wl.f32_to_bf16_bits(rng.standard_normal((M, N)).astype(np.float32))
    ref = oracle.linear(prob.wq, prob.scales, 32, prob.lora_a, prob.lora_b, prob.shape.alpha, x, rows) * scale[:, None].astype(np.float64)
    ref = ref + wl.bf16_bits_to_f32(res).astype(np.float64)
    p = device.upload_problem(prob)
    assert lib.layer_step_block_rows([p] * n, M) == (32 if M == 70 else 64)
    ws = device.alloc_workspace([p] * n, M)
    ys = [device.alloc_y(M, N, 1) for _ in range(n)]
    epi = lib.Epilogue(row_scale=torch.from_numpy(scale).cuda(), residual=device.to_device(res))
    lib.LayerPlanFused([p] * n, [epi] * n, [device.to_device(x)] * n, ys, torch.from_numpy(rows).cuda(), M, 1, ws).run()
    torch.cuda.synchronize()
    assert lib.workspace_status(ws) == 0
    assert all(torch.equal(ys[0], y) for y in ys[1:])
    assert rel_err(device.y_to_numpy(ys[0]), ref) <= TOL_F32


@pytest.mark.parametrize("lowest", [-7, -8])
@pytest.mark.parametrize("M", [8, 16, 64, 640])                    # blocks of 8, 16, 32 and 64 rows
def test_rows_with_a_mean_cost_no_precision(gpu, M, lowest):
    """Codes enter the products without an offset: with rows of mean 2 the sums on the way to a result are no
    larger than those of the weights themselves, in groups of every size and in blobs with codes -8 too.  Observed: at
    most 1.5e-7 of the result (4e-7 leaves room for sums in another order); sums with an offset of 24 are 7 times the result."""
    lib, device, torch = gpu
    K, N = 2048, 8192 if M == 640 else 512
    rng = np.random.default_rng(7)
    x = wl.f32_to_bf16_bits((rng.standard_normal((M, K)) + 2.0).astype(np.float32))
    for G in (32, 64, 128):
        codes = rng.integers(lowest, 8, size=(N, K)).astype(np.int8)
        nib = codes.view(np.uint8) & 15
        wq = torch.from_numpy(nib[:, 0::2] | (nib[:, 1::2] << 4)).cuda()
        scales = (rng.uniform(0.5, 1.5, size=(N, K // G)) * 0.01).astype(np.float16)
        blob = torch.empty(lib.blob_bytes(K, N, G), dtype=torch.uint8, device="cuda")
        lib.prepack(K, N, G, wq, torch.from_numpy(scales).cuda(), blob)
        p = lib.Proj(K, N, G, blob)
        if M > 16:
            assert lib.layer_step_block_rows([p], M) == (64 if M == 640 else 32)
        w = codes.astype(np.float64).reshape(N, K // G, G) * scales.astype(np.float64)[:, :, None]
        ref = wl.bf16_bits_to_f32(x).astype(np.float64) @ w.reshape(N, K).T
        y = device.alloc_y(M, N, 1)
        lib.linear(p, device.to_device(x), None, M, y, 1, device.alloc_workspace([p], M))
        torch.cuda.synchronize()
        error = np.linalg.norm(device.y_to_numpy(y).astype(np.float64) - ref) / np.linalg.norm(ref)
        print(f"M{M} G{G} lowest {lowest}: {error:.2e}", flush=True)
        assert error <= 4e-7, (G, error)


@pytest.mark.parametrize("K,N,M,n_ad", [(4096, 1024, 70, 8), (2048, 640, 200, 16), (8192, 256, 33, 4)])
def test_a_wait_that_runs_out_leaves_no_wrong_number(gpu, K, N, M, n_ad):
    """Few polls, so that some waves of a block give up where others still see their shrink blocks done
    (every kernel runs to its end all the same): an output is right or NaN, and a NaN is reported."""
    lib, device, torch = gpu
    prob = random_problem(K + M, K, N, 32, 16, n_ad)
    x, rows = rows_and_x(M, M, K, n_ad)
    ref = oracle.linear(prob.wq, prob.scales, 32, prob.lora_a, prob.lora_b, prob.shape.alpha, x, rows)
    p, dx, ra = device.upload_problem(prob), device.to_device(x), torch.from_numpy(rows).cuda()
    y = device.alloc_y(M, N, 1)
    ws = device.alloc_workspace([p], M)
    old = lib.debug_spin_limit(-1)
    try:
        for limit in (0, 1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64):
            lib.debug_spin_limit(limit)
            lib.linear(p, dx, ra, M, y, 1, ws)
            torch.cuda.synchronize()
            got = device.y_to_numpy(y)
            gave_up = np.isnan(got)
            assert lib.workspace_status(ws) != 0 or not gave_up.any(), limit
            assert np.max(np.abs(np.where(gave_up, ref, got) - ref)) <= TOL_F32 * np.max(np.abs(ref)), limit
            lib.workspace_init(ws)
            torch.cuda.synchronize()
    finally:
        lib.debug_spin_limit(old)


@pytest.mark.parametrize("M", [8, 24, 40, 200])
def test_t_close_to_the_largest_number(gpu, M):
    """t between the largest bf16 and the largest fp32 is a number: alpha * (A x) = 1.003 * 2^127 * 1.9921875,
    which a bf16 half would round to infinity; times B = 2^-100.  Codes of 0, so the base product is 0.  Bar: 17 bits
    of t."""
    lib, device, torch = gpu
    K, N, r = 128, 128, 8
    prob = random_problem(3, K, N, 32, r, 1)
    prob.wq[:] = 0
    a, b = np.zeros((1, r, K), np.float32), np.zeros((1, N, r), np.float32)
    a[0, 0, 0], b[0, :, 0] = 2.0 ** 64 * 1.9921875, 2.0 ** -100
    x = np.zeros((M, K), np.float32)
    x[:, 0] = 2.0 ** 63
    blob = device.upload_problem(prob).w_blob
    p = lib.Proj(K, N, 32, blob, device.to_device(wl.f32_to_bf16_bits(a)), device.to_device(wl.f32_to_bf16_bits(b)), 1.003)
    y = device.alloc_y(M, N, 1)
    lib.LayerPlan([p], [device.to_device(wl.f32_to_bf16_bits(x))], [y], torch.zeros(M, dtype=torch.int32, device="cuda"), M, 1,
                  device.alloc_workspace([p], M)).run()
    torch.cuda.synchronize()
    ref = float(np.float32(1.003)) * 1.9921875 * 2.0 ** 27
    assert np.max(np.abs(device.y_to_numpy(y) - ref)) <= 2.0 ** -16 * ref
