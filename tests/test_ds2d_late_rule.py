"""Steps of DS2D whose forecast rows wait for the walk: where that spares enough logits, and the walk that every block then
makes for itself stays short beside them."""
import pytest

import paper_2604_18655_amd as lib


@pytest.mark.parametrize("S,m,branch,next_branch,V,dtype,late", [
    (8, 2, (3, 2), (3, 2), 128256, lib.Y_BF16, True),        # 37 MB spared
    (1, 2, (3, 2), (3, 2), 128256, lib.Y_BF16, False),       # 5 MB
    (8, 1, (), (1,), 160000, lib.Y_FP32, False),             # a lone root: nothing to spare
    (8, 2, (3, 2), (), 160000, lib.Y_FP32, False),           # nothing to draft
    (8, 2, (3, 2), (3, 2), 2000003, lib.Y_BF16, True),       # walks of 2.1 times the bytes spared: 262 us, late 229
    (8, 2, (3, 2), (3, 2), 9000001, lib.Y_BF16, False),      # 9.6 times: 1172 us, late 1414
    (8, 2, (3, 2), (3, 2), 20000003, lib.Y_BF16, False),     # 21 times: 2646 us, late 6844
    (8, 2, (3, 2), (3, 2), 6000001, lib.Y_FP32, True),       # 3.2 times: 1234 us, late 925
    (8, 2, (3, 2), (3, 2), 13000001, lib.Y_FP32, False),     # 6.9 times: 2693 us, late 2910
    (8, 1, (1,), (1,), 4000037, lib.Y_BF16, False),          # 7.7 times (a tree of two tokens): 135 us, late 154
    (200, 2, (3, 2), (3, 2), 0x7FFFFFFE, lib.Y_FP32, False),  # the largest vocabulary
])
def test_forecast_rows_wait_for_the_walk(S, m, branch, next_branch, V, dtype, late):
    assert lib.Ds2dStep(S, m, branch, next_branch, V, dtype).late_drafts() is late


def test_refused_steps_are_not_late():
    assert lib.Ds2dStep(0, 2, (3, 2), (3, 2), 128256, lib.Y_BF16).late_drafts() is False
