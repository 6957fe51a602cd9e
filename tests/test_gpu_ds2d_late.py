"""mlora_ds2d_step where the forecast rows wait for the walk (more than 22 MB of logits spared), against oracle/ds2d.py
(integers: exact): rows at odd offsets, both types, walks of every length, more candidates than a block holds at once,
winners below zero."""
import numpy as np
import pytest

from test_gpu_ds2d import check
from workloads.ds2d import make_ds2d_inputs
from workloads.generate import bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,m,branch,next_branch,V,bf16", [
    (12, 2, (3, 2), (3, 2), 56003, True),
    (5, 3, (2, 2), (5, 1, 1), 90001, False),
    (2, 1, (15,), (16,), 700001, True),            # 171 slices x 16 candidates
])
def test_forecast_rows_after_the_walk(gpu, S, m, branch, next_branch, V, bf16):
    logits, tokens = make_ds2d_inputs(V, S, branch, m, V, bf16, accept=0.7)
    R = len(logits) // S
    below = logits[R:2 * R]                         # the second stream: nothing above zero
    logits[R:2 * R] = f32_to_bf16_bits(bf16_bits_to_f32(below) - np.float32(60.0)) if bf16 else below - np.float32(60.0)
    lengths = check(gpu, S, m, branch, next_branch, V, logits, tokens, bf16)
    assert S < 5 or len(set(lengths)) >= 2
