"""mlora_ds2d_step where its kernels branch, against oracle/ds2d.py (integers: exact): winners that
share a vector or a lane, slices whose winners run out above zero, rows that end around the edges
of a slice of 4096 logits, levels whose candidates exceed what a block holds at once."""
import numpy as np
import pytest

from test_gpu_ds2d import check
from workloads.ds2d import make_ds2d_inputs
from workloads.generate import bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("V", [4095, 4096, 4097, 8191, 12305])
def test_few_values_and_slice_edges(gpu, V, bf16):
    S, m, branch, nxt = 3, 2, (2, 2), (9, 1)
    rng = np.random.default_rng(V)
    _, tokens = make_ds2d_inputs(V, S, branch, m, V, True)
    R = 7 * 3
    logits = rng.choice(np.array([-3.0, -1.0, 0.5, 1.0], np.float32), size=(S * R, V))     # ties everywhere
    logits[R:2 * R] = -np.abs(rng.standard_normal((R, V)).astype(np.float32))              # nothing above zero ...
    logits[R:2 * R, 8::4096] = 2.0                                                         # ... but one logit per slice
    logits[2 * R:] = np.sort(rng.standard_normal((R, V)).astype(np.float32), axis=1)       # the best in one lane's vectors
    logits[2 * R + 3, ::5] = np.nan
    logits[2 * R + 4, -9:] = np.inf
    if bf16:
        logits = f32_to_bf16_bits(np.nan_to_num(logits, nan=7.0, posinf=np.inf))
        logits[2 * R + 3, ::5] = 0x7FC1
    check(gpu, S, m, branch, nxt, V, logits, tokens, bf16)


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("V", [1200, 4099, 9000])
def test_logits_not_above_zero(gpu, V, bf16):
    """Winners of either sign, zeros of both signs, infinities and NaN: every order a slice can be taken in."""
    S, m, branch, nxt = 4, 2, (2,), (10, 1)
    rng = np.random.default_rng(V)
    _, tokens = make_ds2d_inputs(V, S, branch, m, V, True)
    R = 3 * 3
    logits = (rng.standard_normal((S * R, V)) - 50.0).astype(np.float32)                   # all negative
    logits[1] = -np.inf
    logits[1, 700:703] = -1e30
    logits[2, :] = np.where(rng.random(V) < 0.5, np.float32(-0.0), np.float32(0.0))        # only zeros
    logits[R:2 * R] = np.where(rng.random((R, V)) < 0.997, -np.abs(logits[R:2 * R]), 3.0)  # a few above zero
    logits[R, ::3] = 0.0
    logits[R + 4, 5::7] = -0.0
    logits[R + 5, :] = -0.0
    logits[R + 5, 11] = 0.0
    logits[2 * R:3 * R, 1::2] = np.nan                                                     # every other one
    logits[2 * R + 3, :] = np.nan
    logits[2 * R + 4, 5:] = -np.nan
    logits[2 * R + 5, 9:] = -np.inf
    logits[3 * R:] = rng.choice(np.array([-2.0, -1.0, -np.inf, np.inf, -0.0, 0.0], np.float32), size=(R, V))
    if bf16:
        nan = np.isnan(logits)
        sign = np.signbit(logits)
        logits = f32_to_bf16_bits(np.where(nan, np.float32(0.0), logits))
        logits[nan & ~sign] = 0x7FC1
        logits[nan & sign] = 0xFFFF
    check(gpu, S, m, branch, nxt, V, logits, tokens, bf16)


def step_time(gpu, S, m, branch, nxt, V, shift):
    """Best time of ten steps in a row, in ms."""
    lib, device, torch = gpu
    T, R = lib.ds2d_rows(branch, m)
    step = lib.Ds2dStep(S, m, branch, nxt, V, lib.Y_BF16)
    rows = (torch.randn((S * R, V), generator=torch.Generator("cuda").manual_seed(1), device="cuda") + shift).to(torch.bfloat16)
    tokens = torch.zeros((S, T), dtype=torch.int32, device="cuda")
    sizes = ((S,), (S, m + 1), (S, m + 1), (S, lib.ds2d_rows(nxt, m)[0]))
    out = [torch.zeros(n, dtype=torch.int32, device="cuda") for n in sizes]
    ws = torch.empty(step.workspace_bytes(), dtype=torch.uint8, device="cuda")
    best = float("inf")
    for _ in range(30):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        begin.record()
        for _ in range(10):
            step.run(rows, tokens, *out, ws)
        end.record()
        torch.cuda.synchronize()
        best = min(best, begin.elapsed_time(end))
    return best


def test_time_does_not_depend_on_the_logits_sign(gpu):
    """A soft-max does not care about a shift, nor may the step's time (three times as long where a slice
    without winners above zero was read again per winner; 1.6 leaves room for noise)."""
    args = (gpu, 8, 2, (3, 2), (3, 2), 128256)
    assert step_time(*args, -50.0) <= 1.6 * step_time(*args, 0.0)


def test_time_does_not_depend_on_the_last_vector(gpu):
    """Rows that end inside a vector of 16 bytes (2.6 times as long where the array's last slice was read
    element by element once per winner)."""
    args = (gpu, 1, 1, (1,), (16,))
    assert step_time(*args, 32001, 0.0) <= 1.6 * step_time(*args, 32000, 0.0)


@pytest.mark.parametrize("V,S,branch,nxt,m", [
    (128256, 1, (15,), (16,), 1),       # candidates of all nodes do not fit the block, those of one do
    (540000, 1, (1,), (16,), 1),        # one level of one node does not fit either
    (540001, 2, (1,), (9, 1), 2),       # rows at odd offsets, a second level after a long one
    (262144, 3, (1,), (4, 2), 2),       # candidates just above those that are all ranked at once
    (66000, 1, (1,), (16,), 1),         # one slice more than winners
    (61435, 1, (2,), (16,), 1),         # a last slice of few logits
    (32001, 1, (1,), (16,), 1),         # the array ends inside a vector
    (4163, 1, (1,), (8,), 1),           # a last slice of 66 or 67 logits, and that vector in it
    (4099, 1, (1,), (16,), 1),
    (5, 1, (), (5,), 1),                # less than two vectors in all
])
def test_many_candidates(gpu, V, S, branch, nxt, m):
    logits, tokens = make_ds2d_inputs(V, S, branch, m, V, True, accept=0.5)
    check(gpu, S, m, branch, nxt, V, logits, tokens, True)
