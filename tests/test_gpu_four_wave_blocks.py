"""Blocks of 32 rows and four column tiles in both their forms: eight waves in short launches (one group of projections, up to
230 base blocks), four in the others.  The same edges through both, the second by repeating the projection until the launch
has two groups (17 projections) or more than 230 blocks, against the oracle: rows around the block sizes, spare waves, units
that end on half a stage, ranks from a run of 16 to the largest, K chunks of the shrink blocks for one, two and
four waves, int8 rows with one block of rows and several, the fused output stage, waits that run out.  Bars as everywhere:
5e-3 of max|y_ref| with bf16 outputs, 2e-4 with fp32 outputs, 5e-3 of the LoRA term's own maximum."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_util import TOL, TOL_F32, random_problem, rel_err

MANY = 17                                         # two groups
EDGES = [                                         # K, N, group, rank, adapters, rows
    (128, 64, 32, 8, 1, 33),                      # the smallest: one super-step, three spare waves, one row in the second block
    (1408, 1408, 32, 16, 5, 64),                  # 22 tiles: two spare waves; 11 super-steps in units that end on half a stage
    (2304, 321, 64, 24, 7, 65),                   # a third block of 32 rows with one row; ragged last tile
    (4224, 640, 128, 128, 3, 95),                 # 33 super-steps; the largest rank
    (1152, 1088, 64, 64, 40, 97),                 # more adapters than rows of a block, dealt over the K units
    (8320, 192, 32, 40, 2, 129),                  # many K units, a rank of three runs of 16
    (128, 200, 64, 24, 17, 190),                  # 128 inputs: every wave of a shrink block has tiles of its own
    (256, 130, 64, 24, 9, 150),                   # 256: two (four) waves share one
]
INT8_EDGES = EDGES[:5] + [(256, 64, 32, 8, 2, 1), (2048, 512, 64, 16, 4, 17), (4096, 256, 128, 24, 3, 32), (128, 1000, 32, 72, 5, 20)]


def waves(shape, n, int8=False):
    import paper_2604_18655_amd as lib
    K, N, G, r, n_ad, M = shape
    projs = [lib.Proj(K, N, G, None, None, None, 1.0, n_ad, r)] * n
    assert lib.layer_step_block_rows(projs, M, int8) == 32
    return lib.layer_step_waves_per_tile(projs, M, int8)


@pytest.mark.parametrize("int8,shapes", [(False, EDGES), (True, INT8_EDGES)])
def test_the_forms_that_the_shapes_run(int8, shapes):
    for shape in shapes:
        assert waves(shape, 1, int8) == 2 and waves(shape, MANY, int8) == 1, shape


def test_waves_of_other_launches():
    import paper_2604_18655_amd as lib
    p = lib.Proj(2048, 8192, 32, None, None, None, 1.0, 8, 16)
    assert lib.layer_step_waves_per_tile([p], 16) == 1                   # blocks of one column tile
    assert lib.layer_step_waves_per_tile([p] * 8, 500) == 1              # blocks of 64 rows
    assert lib.layer_step_waves_per_tile([p], 16, True) == 2             # int8 rows run blocks of four tiles at any row count
    assert lib.layer_step_waves_per_tile([p] * 3, 70) == 1               # 288 base blocks
    assert lib.layer_step_waves_per_tile([lib.Proj(100, 64, 32, None)], 64) == 0
    assert lib.layer_step_waves_per_tile([p], 4097) == 0


def run(gpu, proj, x, rows, M, n, y_dtype, scale=None):
    """Outputs of n copies of a projection, which have to be the same bits, after two calls on one workspace."""
    lib, device, torch = gpu
    projs = [proj] * n
    ys = [device.alloc_y(M, proj.N, y_dtype) for _ in range(n)]
    size = lib.workspace_bytes if scale is None else lib.a8_workspace_bytes
    ws = torch.zeros(max(size(projs, M), 256), dtype=torch.uint8, device="cuda")
    ra = None if rows is None else torch.from_numpy(rows).cuda()
    plan = lib.LayerPlan(projs, [x] * n, ys, ra, M, y_dtype, ws) if scale is None else \
        lib.LayerPlanA8(projs, [x] * n, [scale] * n, ys, ra, M, y_dtype, ws)
    plan.run()
    plan.run()                                            # the counters are back at zero
    torch.cuda.synchronize()
    assert lib.workspace_status(ws) == 0
    assert all(torch.equal(ys[0], y) for y in ys[1:])
    return device.y_to_numpy(ys[0])


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, MANY], ids=["eight waves", "four waves"])
@pytest.mark.parametrize("int8,shape", [(False, s) for s in EDGES] + [(True, s) for s in INT8_EDGES], ids=str)
def test_edges(gpu, int8, shape, n):
    lib, device, torch = gpu
    K, N, G, r, n_ad, M = shape
    prob = random_problem(K + N + M, K, N, G, r, n_ad)
    p = device.upload_problem(prob)
    rng = np.random.default_rng(M)
    rows = rng.integers(-1, n_ad, size=M).astype(np.int32)
    if int8:
        xq, s = wl.make_x_int8(M, K, 5, 0, 0)
        x, s = torch.from_numpy(xq).cuda(), float(s)
        ref, base = (oracle.linear_a8(prob.wq, prob.scales, G, prob.lora_a, prob.lora_b, prob.shape.alpha, xq, s, ra) for ra in (rows, None))
    else:
        bits = wl.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
        x, s = device.to_device(bits), None
        ref, base = (oracle.linear(prob.wq, prob.scales, G, prob.lora_a, prob.lora_b, prob.shape.alpha, bits, ra) for ra in (rows, None))
    y16, y32, b32 = run(gpu, p, x, rows, M, n, 0, s), run(gpu, p, x, rows, M, n, 1, s), run(gpu, p, x, None, M, n, 1, s)
    assert rel_err(y16, ref) <= TOL and rel_err(y32, ref) <= TOL_F32 and rel_err(b32, base) <= TOL_F32
    delta = ref - base
    if np.max(np.abs(delta)) > 0:
        assert np.max(np.abs((y32 - b32) - delta)) <= TOL * np.max(np.abs(delta))


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 3], ids=["eight waves", "four waves"])
def test_fused_output_stage(gpu, n):
    lib, device, torch = gpu
    K, N, r, n_ad, M = 256, 8192, 16, 4, 70
    assert waves((K, N, 32, r, n_ad, M), n) == (2 if n == 1 else 1)
    prob = random_problem(M, K, N, 32, r, n_ad)
    rng = np.random.default_rng(M)
    x = wl.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
    rows = rng.integers(-1, n_ad, size=M).astype(np.int32)
    scale = rng.uniform(0.5, 2.0, M).astype(np.float32)
    res = wl.f32_to_bf16_bits(rng.standard_normal((M, N)).astype(np.float32))
    ref = oracle.linear(prob.wq, prob.scales, 32, prob.lora_a, prob.lora_b, prob.shape.alpha, x, rows) * scale[:, None].astype(np.float64)
    ref = ref + wl.bf16_bits_to_f32(res).astype(np.float64)
    p = device.upload_problem(prob)
    ws = device.alloc_workspace([p] * n, M)
    ys = [device.alloc_y(M, N, 1) for _ in range(n)]
    epi = lib.Epilogue(row_scale=torch.from_numpy(scale).cuda(), residual=device.to_device(res))
    lib.LayerPlanFused([p] * n, [epi] * n, [device.to_device(x)] * n, ys, torch.from_numpy(rows).cuda(), M, 1, ws).run()
    torch.cuda.synchronize()
    assert lib.workspace_status(ws) == 0
    assert all(torch.equal(ys[0], y) for y in ys[1:])
    assert rel_err(device.y_to_numpy(ys[0]), ref) <= TOL_F32


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, MANY], ids=["eight waves", "four waves"])
@pytest.mark.parametrize("K,N,M,n_ad", [(4096, 1024, 70, 8), (2048, 640, 200, 16), (8192, 256, 33, 4)])
def test_a_wait_that_runs_out_leaves_no_wrong_number(gpu, K, N, M, n_ad, n):
    """Few polls, so that some waves of a block give up where others still see their shrink blocks done
    (every kernel runs to its end all the same): an output is right or NaN, and a NaN is reported."""
    lib, device, torch = gpu
    assert waves((K, N, 32, 16, n_ad, M), n) == (2 if n == 1 else 1)
    prob = random_problem(K + M, K, N, 32, 16, n_ad)
    rng = np.random.default_rng(M)
    x = wl.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
    rows = rng.integers(-1, n_ad, size=M).astype(np.int32)
    ref = oracle.linear(prob.wq, prob.scales, 32, prob.lora_a, prob.lora_b, prob.shape.alpha, x, rows)
    p, dx, ra = device.upload_problem(prob), device.to_device(x), torch.from_numpy(rows).cuda()
    ys = [device.alloc_y(M, N, 1) for _ in range(n)]
    ws = device.alloc_workspace([p] * n, M)
    plan = lib.LayerPlan([p] * n, [dx] * n, ys, ra, M, 1, ws)
    old = lib.debug_spin_limit(-1)
    try:
        for limit in (0, 1, 2, 4, 8, 16, 32, 64):
            lib.debug_spin_limit(limit)
            plan.run()
            torch.cuda.synchronize()
            got = np.stack([device.y_to_numpy(y) for y in ys])
            gave_up = np.isnan(got)
            assert lib.workspace_status(ws) != 0 or not gave_up.any(), limit
            assert np.max(np.abs(np.where(gave_up, ref, got) - ref)) <= TOL_F32 * np.max(np.abs(ref)), limit
            lib.workspace_init(ws)
            torch.cuda.synchronize()
    finally:
        lib.debug_spin_limit(old)
