"""Masked tree attention where the cut of its keys changes: chunks of 32, four and eight waves, one and two query tiles per
block, blocks that share the keys of a tile (some of them without any).  Bars as in test_gpu_tree_attention."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_tree_attention import check, gpu_attention
from workloads.attention import ds2d_tree, make_attention_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("S,Hq,Hkv,Lp,Lf,cap,lens", [
    (2, 6, 3, 31, 32, 33, [33, 0]),            # four waves, chunks that are just not full, full and one over
    (3, 8, 1, 353, 0, 64, [64, 32, 31]),       # eight waves, 15 x 8 query vectors in eight tiles
    (2, 4, 2, 900, 1, 700, [700, 0]),          # shared keys: the second stream has far fewer chunks than its blocks
    (4, 16, 8, 3000, 40, 1, [1, 0, 1, 0]),     # two tiles per block, the second one not full
    (1, 2, 1, 4897, 0, 2, [2]),                # a long call: as many blocks as the merging kernel takes in two trips
])
def test_cuts(gpu, D, S, Hq, Hkv, Lp, Lf, cap, lens):
    parent, is_forecast = ds2d_tree((2, 1))
    inp = make_attention_inputs(Lp, S, parent, is_forecast, Hq, Hkv, D, Lp, Lf, cap, len_stream=lens)
    check(gpu, inp, Hq, Hkv, D, f"D{D} S{S} Lp{Lp} Lf{Lf} cap{cap}")


@pytest.mark.parametrize("Lp", [40, 2000])
def test_a_prefix_that_a_row_may_not_see_does_not_touch_it(gpu, Lp):
    """Values of infinity in the forecast prefix: rows of tokens are what they are without it."""
    lib = gpu[0]
    parent, is_forecast = ds2d_tree((3, 2))
    inp = make_attention_inputs(7, 2, parent, is_forecast, 4, 2, 64, Lp, 70, 9)
    inp.v_fprefix[:] = wl.f32_to_bf16_bits(np.full(inp.v_fprefix.shape, np.inf, np.float32))
    out = gpu_attention(gpu, inp, lib.Y_FP32, 4, 2, 64)
    clean = make_attention_inputs(7, 2, parent, is_forecast, 4, 2, 64, Lp, 70, 9)
    want = gpu_attention(gpu, clean, lib.Y_FP32, 4, 2, 64)
    tokens = inp.is_forecast == 0
    assert np.array_equal(out[tokens], want[tokens])
    assert not np.isfinite(out[~tokens]).any()
