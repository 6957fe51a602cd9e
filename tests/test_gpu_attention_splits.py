"""Masked tree attention where the cut of its keys changes: chunks of 32, four and eight waves, one and two query tiles per
block, blocks that share the keys of a tile (some of them without any), and all sixteen forms of the kernel.  Bars as in
test_gpu_tree_attention."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_tree_attention import check, gpu_attention
from workloads.attention import ds2d_tree, make_attention_inputs


@pytest.mark.gpu
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


@pytest.mark.gpu
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


# (D, query tiles of a block, waves, keys shared by several blocks) -> streams, heads, kv heads, rows, forecast prefix, prefill, cap
FORMS = {
    (64, 1, 4, False): (2, 6, 3, "ds2d15", 0, 31, 33),
    (64, 1, 4, True): (3, 4, 2, "ds2d15", 3, 900, 65),
    (64, 1, 8, False): (3, 8, 1, "ds2d15", 0, 353, 64),
    (64, 1, 8, True): (23, 4, 2, "chain3", 5, 2600, 33),
    (64, 2, 4, False): (25, 16, 2, "random64", 7, 40, 1),            # 32 tiles of a stream and head
    (64, 2, 4, True): (24, 8, 4, "random9", 0, 901, 33),
    (64, 2, 8, False): (31, 16, 8, "random9", 0, 333, 33),           # a second tile of two query vectors
    (64, 2, 8, True): (23, 4, 2, "random9", 33, 2600, 0),
    (128, 1, 4, False): (2, 6, 3, "ds2d15", 1, 31, 20),
    (128, 1, 4, True): (3, 4, 2, "ds2d15", 0, 700, 65),
    (128, 1, 8, False): (3, 8, 1, "ds2d15", 0, 190, 64),
    (128, 1, 8, True): (23, 4, 2, "chain3", 5, 2600, 33),
    (128, 2, 4, False): (25, 8, 1, "random64", 0, 40, 1),
    (128, 2, 4, True): (24, 4, 2, "random9", 0, 901, 33),
    (128, 2, 8, False): (31, 4, 1, "random64", 7, 70, 33),           # 137 KB of LDS
    (128, 2, 8, True): (23, 4, 1, "random9", 33, 2600, 0),
}


def rows_of(tree, seed):
    rng = np.random.default_rng(seed)
    return {"ds2d15": lambda: ds2d_tree((2, 1)), "chain3": lambda: wl.chain_tree(3), "random9": lambda: wl.random_tree(9, rng),
            "random64": lambda: wl.random_tree(64, rng)}[tree]()


def test_every_form_has_a_shape():
    import torch

    import paper_2604_18655_amd as lib
    some = torch.zeros(64)                         # (the plan reads no memory, but refuses missing or unaligned tensors)
    assert some.data_ptr() % 16 == 0
    assert set(FORMS) == {(D, t, w, s) for D in (64, 128) for t in (1, 2) for w in (4, 8) for s in (False, True)}
    for form, (S, Hq, Hkv, tree, Lf, Lp, cap) in FORMS.items():
        call = lib.TreeAttention(Hq, Hkv, form[0], S, len(rows_of(tree, 0)[0]), 0.125, some, some, some, some, some, some, some,
                                 some, some, some, some, Lp, Lf, cap)
        plan = call.plan()
        assert (form[0], plan["tiles"], plan["waves"], plan["splits"] > 1) == form, (form, plan)


@pytest.mark.gpu
@pytest.mark.parametrize("form", list(FORMS), ids=str)
def test_every_form(gpu, form):
    S, Hq, Hkv, tree, Lf, Lp, cap = FORMS[form]
    parent, is_forecast = rows_of(tree, S)
    rng = np.random.default_rng(Lp)
    inp = make_attention_inputs(Lp + S, S, parent, is_forecast, Hq, Hkv, form[0], Lp, Lf, cap,
                                len_stream=rng.integers(0, cap + 1, size=S))
    check(gpu, inp, Hq, Hkv, form[0], f"{form} {FORMS[form]}")
