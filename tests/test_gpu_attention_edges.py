"""Masked tree attention at the edges of its chunks of 32 keys (segments that end with a chunk, one key before and one
after it, empty and full streams side by side) in one launch and with shared keys, and scores of very different
size.  Same bars as test_gpu_tree_attention."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_tree_attention import check
from workloads.attention import ds2d_tree, make_attention_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Lp,Lf,cap", [(1, 0, 1), (63, 1, 0), (64, 63, 65), (65, 64, 128), (129, 65, 63), (700, 5, 640), (1300, 0, 2)])
def test_chunk_edges(gpu, D, Lp, Lf, cap):
    parent, is_forecast = ds2d_tree((2, 1))
    inp = make_attention_inputs(Lp + cap, 3, parent, is_forecast, 6, 3, D, Lp, Lf, cap, len_stream=[0, cap, max(0, cap - 1)])
    check(gpu, inp, 6, 3, D, f"D{D} Lp{Lp} Lf{Lf} cap{cap}")


def test_large_scores(gpu):
    """Scores of +-hundreds: weights of 0 and 1 next to keys a row may not see."""
    parent, is_forecast = ds2d_tree((3, 2))
    inp = make_attention_inputs(5, 2, parent, is_forecast, 4, 1, 64, 190, 9, 70, k_std=40.0)
    inp.k_fprefix[:] = wl.f32_to_bf16_bits(np.full(inp.k_fprefix.shape, 60.0, np.float32))
    check(gpu, inp, 4, 1, 64, "large scores")
