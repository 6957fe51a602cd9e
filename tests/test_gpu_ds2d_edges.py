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


@pytest.mark.parametrize("V,S,branch,nxt,m", [
    (128256, 1, (15,), (16,), 1),       # candidates of all nodes do not fit the block, those of one do
    (540000, 1, (1,), (16,), 1),        # one level of one node does not fit either
    (540001, 2, (1,), (9, 1), 2),       # rows at odd offsets, a second level after a long one
])
def test_many_candidates(gpu, V, S, branch, nxt, m):
    logits, tokens = make_ds2d_inputs(V, S, branch, m, V, True, accept=0.5)
    check(gpu, S, m, branch, nxt, V, logits, tokens, True)
