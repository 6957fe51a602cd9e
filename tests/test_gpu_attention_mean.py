"""Masked tree attention whose keys all carry the same weight and the same values: sums of up to 3064 equal bf16 numbers are
exact in fp32 (8 + 12 bits), so the quotient by the sum of the weights is the value itself, bit for bit."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_tree_attention import gpu_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Lp", [0, 3000])          # 1 to 64 keys in one launch; 3001 to 3064, shared by several blocks
def test_equal_values_come_back(gpu, D, Lp):
    lib = gpu[0]
    parent, is_forecast = wl.chain_tree(64)
    inp = wl.make_attention_inputs(D + Lp, 1, parent, is_forecast, 2, 1, D, Lp, 0, 0)
    inp.q[:] = 0
    value = inp.v_new[0, 0].copy()
    inp.v_new[:] = value
    inp.v_prefill[:] = value
    out = gpu_attention(gpu, inp, lib.Y_FP32, 2, 1, D)
    want = wl.bf16_bits_to_f32(value)
    bad = [r for r in range(64) if not np.array_equal(out[r], np.broadcast_to(want, (2, D)))]
    assert not bad, f"rows with {[Lp + r + 1 for r in bad][:8]} keys"
