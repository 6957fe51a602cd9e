"""The library's work as timed cases: decoding steps, prefill chunks and what stands between them.

A case is a dict of plain values.  Its "kind" names the public call it stands for:

    linear      binding.linear, one projection with an adapter index per row
    layers      binding.LayerPlan: the projections of one or several decoder layers in one call
                (lora "int16": stacks stored as 16-bit integers, expanded once when they are loaded)
    layers_a8   binding.LayerPlanA8: the same with int8 rows
    decoder     decoder.DecoderLayerStep: one decoder layer in dependency order
    attention   binding.TreeAttention: masked tree attention over a segmented cache
    ds2d        binding.Ds2dStep: verification of a draft tree and the drafts of the next step

Inputs follow the distributions of workloads/ (weights N(0, 0.02) quantised per group, adapters
A ~ N(0, 1/K), B ~ N(0, 0.01^2), rows N(0, 1)), drawn on the GPU from the seed.  exact() computes
the same outputs in float64 with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2604_18655_amd as lib
from paper_2604_18655_amd import device as dev
from paper_2604_18655_amd.decoder import DecoderLayerStep

DEVICE = "cuda:0"
EPS = 1e-5

# (name, K, N, input slot) of a decoder layer's projections, by hidden width h, key/value width v, MLP width f
_LAYER = (("q", "h", "h", "attn_in"), ("k", "h", "v", "attn_in"), ("v", "h", "v", "attn_in"), ("o", "h", "h", "attn_out"),
          ("gate", "h", "f", "mlp_in"), ("up", "h", "f", "mlp_in"), ("down", "f", "h", "mlp_act"))

# draft trees in use: the worked example, the evaluated configurations' neighbourhood, a lone root
_BRANCHES = ("", "1", "3", "2,1", "3,2", "4,2", "3,1", "2,2", "1,1,1", "2,1,1")


def _linear(name, K, N, M, group, rank, adapters, alpha, rows, y):
    return {"name": name, "kind": "linear", "K": K, "N": N, "M": M, "group": group, "rank": rank,
            "adapters": adapters, "alpha": alpha, "rows": rows, "y": y}


def _layers(name, kind, M, layers, rows, hidden=2048, kv=512, ffn=8192, group=32, rank=16, adapters=8, lora="bf16"):
    return {"name": name, "kind": kind, "M": M, "layers": layers, "rows": rows, "hidden": hidden, "kv": kv, "ffn": ffn,
            "group": group, "rank": rank, "adapters": adapters, "alpha": 2.0, "lora": lora, "y": "bf16"}


def listed():
    return [
        # the smallest call: one projection, 8 streams of one token (launch and host cost)
        _linear("linear_tiny", 256, 256, 8, 32, 8, 8, 2.0, "one_to_one", "bf16"),
        # a projection whose sizes fit nothing: odd rows and columns, some rows without adapter, fp32 outputs
        _linear("linear_ragged", 1408, 1003, 13, 64, 24, 5, 1.5, "mixed", "fp32"),
        # one decoding step of one layer: 8 streams of one token, the seven projections of a 1B-like layer
        _layers("decode_layer", "layers", 8, 1, "one_to_one"),
        # the decoding step of a whole 16-layer stack, 8 streams of a 4-token draft tree
        _layers("decode_stack", "layers", 32, 16, "block:4"),
        # the same with int8 activations
        _layers("decode_stack_int8", "layers_a8", 32, 16, "block:4"),
        # a prefill chunk of 512 rows of one adapter through the stack
        _layers("prefill_stack", "layers", 512, 16, "const:0"),
        # verification of wide draft trees: 8 streams of 16 tokens through one MLP projection
        _linear("tree_rows", 3072, 8192, 128, 64, 16, 8, 2.0, "block:16", "bf16"),
        # many tenants: 64 rows over 32 adapters of rank 64, up and down projection of a large model
        _linear("tenants_up", 4096, 14336, 64, 128, 64, 32, 1.0, "zipf:1.1", "bf16"),
        _linear("tenants_down", 14336, 4096, 64, 128, 64, 32, 1.0, "zipf:1.1", "bf16"),
        # one decoder layer as a program runs it, each call waiting for the one before
        {"name": "decoder_layer", "kind": "decoder", "streams": 8, "branch": "1", "forecast": 1, "hidden": 2048, "kv_heads": 8,
         "ffn": 8192, "group": 32, "rank": 16, "adapters": 8, "prefill": 2048, "cap": 128},
        # the attention of that step on its own
        {"name": "attention", "kind": "attention", "streams": 8, "branch": "1", "forecast": 1, "heads": 32, "kv_heads": 8, "dim": 64,
         "prefill": 2048, "prefix": 0, "cap": 128, "y": "bf16"},
        # the token side of a step: the worked example's tree (30 rows) in 8 streams over a large vocabulary
        {"name": "ds2d_step", "kind": "ds2d", "streams": 8, "branch": "3,2", "next": "3,2", "forecast": 2, "vocab": 128256, "y": "bf16"},
    ]


# ------------------------------------------------------------------------------------------
# more cases of the same ranges
# ------------------------------------------------------------------------------------------
def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _rows_kind(rng):
    return rng.choice(("one_to_one", "block:4", "block:16", "const:0", "mixed", "zipf:1.1"))


def _macs(case):
    """Multiply-adds of the projections of one pass (0 for the calls without projections)."""
    return sum(n * K * N * case["M"] for _, K, N, _, n in _projections(case)) if case["kind"] in ("linear", "layers", "layers_a8") else 0


def draw(rng):
    kind = rng.choice(("linear", "linear", "linear", "layers", "layers", "layers_a8", "decoder", "attention", "attention", "ds2d"))
    group = rng.choice((32, 32, 64, 128))
    if kind == "linear":
        case = _linear("", 128 * _log_int(rng, 1, 112), _log_int(rng, 48, 14336), _log_int(rng, 1, 512), group,
                       rng.choice((8, 16, 24, 32, 64, 128)), _log_int(rng, 1, 32), rng.choice((1.0, 1.5, 2.0)), _rows_kind(rng),
                       rng.choice(("bf16", "bf16", "fp32")))
    elif kind in ("layers", "layers_a8"):
        hidden = 128 * _log_int(rng, 4, 32)
        kv = 64 * rng.randint(1, max(1, hidden // 128))
        ffn = 128 * max(1, int(round(hidden * rng.uniform(2.0, 4.0) / 128)))
        lora = rng.choice(("bf16", "bf16", "int16")) if kind == "layers" else "bf16"
        case = _layers("", kind, _log_int(rng, 1, 512), _log_int(rng, 1, 16), _rows_kind(rng), hidden, kv, ffn, group,
                       rng.choice((8, 16, 32)), _log_int(rng, 1, 16), lora)
        # no drawn case is larger than the largest listed one, in weights or in products
        while case["layers"] > 1 and (_macs(case) > 4.9e11 or _macs(case) / case["M"] > 9.7e8):
            case["layers"] -= 1
        while _macs(case) > 4.9e11:
            case["M"] -= 1 + case["M"] // 16
    elif kind == "decoder":
        kv_heads = rng.choice((2, 4, 8))
        hidden = 64 * kv_heads * rng.choice((2, 4, 8))
        branch = rng.choice(_BRANCHES)
        case = {"kind": "decoder", "streams": _log_int(rng, 1, 8), "branch": branch, "forecast": max(1, len(_branch(branch))),
                "hidden": hidden, "kv_heads": kv_heads, "ffn": 128 * max(1, int(round(hidden * rng.uniform(2.0, 4.0) / 128))),
                "group": group, "rank": rng.choice((8, 16, 32)), "adapters": _log_int(rng, 1, 16),
                "prefill": _log_int(rng, 16, 8192), "cap": _log_int(rng, 8, 512)}
    elif kind == "attention":
        branch, kv_heads = rng.choice(_BRANCHES), rng.choice((1, 2, 4, 8))
        m = max(1, len(_branch(branch)))
        case = {"kind": "attention", "streams": _log_int(rng, 1, 16), "branch": branch, "forecast": m,
                "heads": kv_heads * rng.choice((1, 2, 4, 8)), "kv_heads": kv_heads, "dim": rng.choice((64, 64, 128)),
                "prefill": _log_int(rng, 1, 32768), "prefix": rng.choice((0, 5, 16)), "cap": _log_int(rng, 1, 1024),
                "y": rng.choice(("bf16", "bf16", "fp32"))}
        while _attention_work(case, case["heads"], kv_heads, case["dim"], case["prefix"], 2)[1] > 5e10:
            case["prefill"] = case["prefill"] * 3 // 4
            case["cap"] = max(1, case["cap"] * 3 // 4)
    else:
        branch, nxt = rng.choice(_BRANCHES), rng.choice(_BRANCHES)
        case = {"kind": "ds2d", "streams": _log_int(rng, 1, 16), "branch": branch, "next": nxt,
                "forecast": max(1, len(_branch(branch)), len(_branch(nxt))), "vocab": _log_int(rng, 2048, 160000),
                "y": rng.choice(("bf16", "bf16", "fp32"))}
    case.pop("name", None)
    return case


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------
def _branch(text):
    return [int(b) for b in text.split(",")] if text else []


def _tree(branch, m):
    """(parent, is_forecast) of one stream's rows: tokens level by level, then each token's m forecast embeddings."""
    parent, level = [-1], [0]
    for b in branch:
        grown = []
        for node in level:
            for _ in range(b):
                parent.append(node)
                grown.append(len(parent) - 1)
        level = grown
    tokens = len(parent)
    forecast = [0] * tokens
    for t in range(tokens):
        prev = t
        for _ in range(m):
            parent.append(prev)
            forecast.append(1)
            prev = len(parent) - 1
    return parent, forecast, tokens


def _projections(case):
    """(name, K, N, input slot, copies) of the projections of a case."""
    if case["kind"] == "linear":
        return [("y", case["K"], case["N"], "x", 1)]
    size = {"h": case["hidden"], "v": case["kv"], "f": case["ffn"]}
    return [(name, size[k], size[n], slot, case["layers"]) for name, k, n, slot in _LAYER]


def _generator(seed, *more):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(np.random.SeedSequence([int(seed), *more]).generate_state(1, np.uint64)[0] >> np.uint64(1)))
    return g


def _normal(g, shape, std=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float32) * std).to(dtype)


def _rows(case, seed, M, adapters):
    kind, _, arg = case["rows"].partition(":")
    m = np.arange(M)
    rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence([int(seed), 11])))
    if kind == "one_to_one":
        a = m % adapters
    elif kind == "block":
        a = (m // int(arg)) % adapters
    elif kind == "const":
        a = np.full(M, int(arg))
    elif kind == "mixed":                              # rows of several adapters in any order, some on the base model
        a = rng.integers(-1, adapters, size=M)
    else:
        p = (np.arange(adapters) + 1.0) ** (-float(arg))
        a = rng.choice(adapters, size=M, p=p / p.sum())
    return torch.from_numpy(a.astype(np.int32)).to(DEVICE)


def _weight(g, K, N, group):
    """Codes int8 [N][K] in [-8, 7] and fp16 scales [N][K / group] of a weight w ~ N(0, 0.02)."""
    w = torch.randn((N, K // group, group), generator=g, device=DEVICE) * 0.02
    scale = (w.abs().amax(dim=2) / 7.0).to(torch.float16)
    scale[scale == 0] = 1.0
    codes = torch.round(w / scale.float()[:, :, None]).clamp_(-8, 7).to(torch.int8)
    return codes.view(N, K), scale


def _int16_stack(t):
    """A float32 stack as int16 with one scale: (int16 tensor, scale as a float32 number)."""
    s = (t.abs().max() / 32767.0).item() or 1.0
    return torch.round(t / s).clamp_(-32767, 32767).to(torch.int16), float(np.float32(s))


def _projection_inputs(case, seed, layer, index, K, N, rank, adapters):
    """One projection's tensors: codes, scales and its LoRA stacks (bf16, or int16 with two scales)."""
    g = _generator(seed, 1, layer, index)
    codes, scale = _weight(g, K, N, case["group"])
    a = torch.randn((adapters, rank, K), generator=g, device=DEVICE) / math.sqrt(K)
    b = torch.randn((adapters, N, rank), generator=g, device=DEVICE) * 0.01
    if case.get("lora") == "int16":
        return codes, scale, _int16_stack(a), _int16_stack(b)
    return codes, scale, a.to(torch.bfloat16), b.to(torch.bfloat16)


def _blob(codes, scale, K, N, group):
    nib = codes.view(torch.uint8) & 15
    wq = (nib[:, 0::2] | (nib[:, 1::2] << 4)).contiguous()
    blob = torch.empty(lib.blob_bytes(K, N, group), dtype=torch.uint8, device=DEVICE)
    lib.prepack(K, N, group, wq, scale, blob)
    return blob


def _proj(case, K, N, codes, scale, a, b, alpha):
    blob = _blob(codes, scale, K, N, case["group"])
    if not isinstance(a, tuple):
        return lib.Proj(K, N, case["group"], blob, a, b, alpha)
    (aq, s_a), (bq, s_b) = a, b
    n, rank = aq.shape[0], aq.shape[1]
    lora_a = torch.empty((n, 4 * rank, K), dtype=torch.bfloat16, device=DEVICE)
    lora_b = torch.empty((n, N, 4 * rank), dtype=torch.bfloat16, device=DEVICE)
    alpha4 = lib.lora_int16_expand(aq, bq, n, rank, K, N, alpha, s_a, s_b, lora_a, lora_b)
    return lib.Proj(K, N, case["group"], blob, lora_a, lora_b, alpha4)


def _x(case, seed, layer, slot, M, K):
    """Rows of one input: bf16, or (int8 rows, scale) for int8 activations."""
    slots = sorted({p[3] for p in _projections(case)})
    x = _normal(_generator(seed, 2, layer, slots.index(slot)), (M, K), dtype=torch.float32)
    if case["kind"] != "layers_a8":
        return x.to(torch.bfloat16)
    s = float(np.float32((x.abs().max() / 127.0).item()))
    return torch.round(x / s).clamp_(-127, 127).to(torch.int8), s


def _y_dtype(case):
    return (lib.Y_FP32, torch.float32) if case["y"] == "fp32" else (lib.Y_BF16, torch.bfloat16)


def _prepare_projections(case, seed):
    M, y_code, y_type = case["M"], *_y_dtype(case)
    rows = _rows(case, seed, M, case["adapters"])
    projs, xs, scales, ys, out = [], [], [], [], {}
    for name, K, N, slot, n in _projections(case):
        out[name] = torch.zeros((n, M, N), dtype=y_type, device=DEVICE)
        # (outputs of a call are 16-byte aligned: every one of several layers has a tensor of its own
        # unless its size keeps the next one aligned)
        assert n == 1 or (M * N * out[name].element_size()) % 16 == 0
    held = {}
    for layer in range(case.get("layers", 1)):
        for index, (name, K, N, slot, _) in enumerate(_projections(case)):
            if (layer, slot) not in held:
                held[layer, slot] = _x(case, seed, layer, slot, M, K)
            x = held[layer, slot]
            x, s = x if isinstance(x, tuple) else (x, 1.0)
            projs.append(_proj(case, K, N, *_projection_inputs(case, seed, layer, index, K, N, case["rank"], case["adapters"]), case["alpha"]))
            xs.append(x)
            scales.append(s)
            ys.append(out[name][layer])
    state = {"kind": case["kind"], "out": out}
    if case["kind"] == "linear":
        state.update(proj=projs[0], x=xs[0], rows=rows, M=M, y=ys[0], y_code=y_code, ws=dev.alloc_workspace(projs, M, DEVICE))
    elif case["kind"] == "layers":
        ws = dev.alloc_workspace(projs, M, DEVICE)
        state["plan"] = lib.LayerPlan(projs, xs, ys, rows, M, y_code, ws)
    else:
        ws = torch.empty(max(lib.a8_workspace_bytes(projs, M), 256), dtype=torch.uint8, device=DEVICE)
        lib.workspace_init(ws)
        state["plan"] = lib.LayerPlanA8(projs, xs, scales, ys, rows, M, y_code, ws)
    return state


def _attention_inputs(case, seed, heads, kv_heads, dim, prefix):
    g = _generator(seed, 3)
    parent, forecast, _ = _tree(_branch(case["branch"]), case["forecast"])
    S, R = case["streams"], len(parent)
    t = {"S": S, "R": R, "parent": parent, "forecast": forecast}
    for name, shape in (("q", (S * R, heads, dim)), ("k_prefill", (kv_heads, case["prefill"], dim)), ("v_prefill", (kv_heads, case["prefill"], dim)),
                        ("k_fprefix", (kv_heads, prefix, dim)), ("v_fprefix", (kv_heads, prefix, dim)),
                        ("k_stream", (S, kv_heads, case["cap"], dim)), ("v_stream", (S, kv_heads, case["cap"], dim)),
                        ("k_new", (S * R, kv_heads, dim)), ("v_new", (S * R, kv_heads, dim))):
        t[name] = _normal(g, shape)
    t["len_stream"] = np.random.Generator(np.random.PCG64(np.random.SeedSequence([int(seed), 12]))).integers(0, case["cap"] + 1, size=S)
    return t


def _attention(t, heads, kv_heads, dim):
    i32 = lambda v: torch.tensor(np.asarray(v), dtype=torch.int32, device=DEVICE)  # noqa: E731
    parent, forecast = i32(t["parent"] * t["S"]), torch.tensor(t["forecast"] * t["S"], dtype=torch.uint8, device=DEVICE)
    some = lambda k: t[k] if t[k].numel() else None  # noqa: E731
    return lib.TreeAttention(heads, kv_heads, dim, t["S"], t["R"], 1.0 / math.sqrt(dim), t["k_prefill"], t["v_prefill"], some("k_fprefix"),
                             some("v_fprefix"), t["k_stream"], t["v_stream"], i32(t["len_stream"]), t["k_new"], t["v_new"], parent, forecast,
                             t["k_prefill"].shape[1], t["k_fprefix"].shape[1], t["k_stream"].shape[2])


def _decoder_case(case):
    """The projections of a decoder layer: gate and up are one projection of interleaved tiles."""
    h, kv = case["hidden"], 64 * case["kv_heads"]
    return (("q", h, h, 1), ("k", h, kv, 1), ("v", h, kv, 1), ("o", h, h, 1), ("gate_up", h, 2 * case["ffn"], 2), ("down", case["ffn"], h, 1))


def _decoder_inputs(case, seed):
    t = _attention_inputs(case, seed, case["hidden"] // 64, case["kv_heads"], 64, 0)
    M = t["S"] * t["R"]
    g = _generator(seed, 4)
    t["h"] = _normal(g, (M, case["hidden"]))
    angle = torch.rand((M, 32), generator=g, device=DEVICE) * (2 * math.pi)
    t["cos"], t["sin"] = torch.cos(angle), torch.sin(angle)
    t["rows"] = torch.arange(M, device=DEVICE, dtype=torch.int32).div(t["R"], rounding_mode="floor").remainder(case["adapters"]).to(torch.int32)
    t["projections"] = {}
    for index, (name, K, N, pair) in enumerate(_decoder_case(case)):
        codes, scale, a, b = _projection_inputs(case, seed, 0, index, K, N, case["rank"] * pair, case["adapters"])
        if pair == 2:                                    # gate columns use the first half of the ranks, up columns the second
            up = (torch.arange(N, device=DEVICE) % 64) >= 32
            second = torch.arange(2 * case["rank"], device=DEVICE) >= case["rank"]
            b = b * (up[:, None] == second[None, :]).to(b.dtype)[None]
        t["projections"][name] = (K, N, codes, scale, a, b)
    return t


def _ds2d_inputs(case, seed):
    rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence([int(seed), 13])))
    parent, _, T = _tree(_branch(case["branch"]), case["forecast"])
    S, R, V = case["streams"], len(parent), case["vocab"]
    logits = torch.randn((S * R, V), generator=_generator(seed, 5), device=DEVICE) * 2.0
    tokens = rng.integers(0, V, size=(S, T)).astype(np.int32)
    at = []
    for s in range(S):
        for node in range(T):
            kids = [c for c in range(1, T) if parent[c] == node]
            if kids:
                tokens[s, kids] = rng.choice(V, size=len(kids), replace=False)
                if rng.random() < 0.6:                    # a draft the model agrees with
                    at.append((s * R + node, int(tokens[s, kids[int(rng.integers(0, len(kids)))]])))
    if at:
        r, c = torch.tensor(at, device=DEVICE).unbind(1)
        logits[r, c] = 40.0
    return logits.to(torch.float32 if case["y"] == "fp32" else torch.bfloat16), torch.from_numpy(tokens).to(DEVICE), S, R, T


def prepare(case, seed):
    if case["kind"] in ("linear", "layers", "layers_a8"):
        return _prepare_projections(case, seed)
    if case["kind"] == "attention":
        t = _attention_inputs(case, seed, case["heads"], case["kv_heads"], case["dim"], case["prefix"])
        call = _attention(t, case["heads"], case["kv_heads"], case["dim"])
        y_code, y_type = _y_dtype(case)
        return {"kind": "attention", "call": call, "q": t["q"], "out": torch.zeros(call.shape, dtype=y_type, device=DEVICE), "y_code": y_code,
                "ws": torch.empty(max(call.workspace_bytes(), 256), dtype=torch.uint8, device=DEVICE)}
    if case["kind"] == "decoder":
        t = _decoder_inputs(case, seed)
        projs = [_proj(case, K, N, codes, scale, a, b, 2.0) for K, N, codes, scale, a, b in t["projections"].values()]
        call = _attention(t, case["hidden"] // 64, case["kv_heads"], 64)
        layer = DecoderLayerStep(*projs, call, t["h"], t["cos"], t["sin"], t["rows"], t["S"] * t["R"], eps=EPS)
        out = {"out": layer.out.view(torch.bfloat16), "k": t["k_new"], "v": t["v_new"], "squares": layer.out_sq}
        return {"kind": "decoder", "layer": layer, "out": out}
    logits, tokens, S, R, T = _ds2d_inputs(case, seed)
    m = case["forecast"]
    step = lib.Ds2dStep(S, m, _branch(case["branch"]), _branch(case["next"]), case["vocab"], lib.Y_FP32 if case["y"] == "fp32" else lib.Y_BF16)
    T_next = _tree(_branch(case["next"]), m)[2]
    i32 = lambda *shape: torch.zeros(shape, dtype=torch.int32, device=DEVICE)  # noqa: E731
    return {"kind": "ds2d", "step": step, "logits": logits, "tokens": tokens,
            "out": {"n_accepted": i32(S), "accepted_rows": i32(S, m + 1), "emitted": i32(S, m + 1), "next_tokens": i32(S, T_next)},
            "ws": torch.empty(max(step.workspace_bytes(), 256), dtype=torch.uint8, device=DEVICE)}


def run(state):
    kind, out = state["kind"], state["out"]
    if kind == "linear":
        lib.linear(state["proj"], state["x"], state["rows"], state["M"], state["y"], state["y_code"], state["ws"])
    elif kind in ("layers", "layers_a8"):
        state["plan"].run()
    elif kind == "attention":
        state["call"].run(state["q"], out, state["y_code"], state["ws"])
    elif kind == "decoder":
        state["layer"].run()
    else:
        state["step"].run(state["logits"], state["tokens"], out["n_accepted"], out["accepted_rows"], out["emitted"], out["next_tokens"], state["ws"])
    return out


# ------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------
def _present(case, M, adapters):
    """Distinct adapters among M rows (the expected number where the rows are drawn)."""
    kind, _, arg = case["rows"].partition(":")
    if kind == "const":
        return 1
    if kind == "block":
        return min(adapters, -(-M // int(arg)))
    if kind == "one_to_one":
        return min(adapters, M)
    p = (np.arange(adapters) + 1.0) ** (-float(arg)) if kind == "zipf" else np.ones(adapters + 1)
    p = (p / p.sum())[:adapters]
    return float(np.sum(1.0 - (1.0 - p) ** M))


def _projection_work(K, N, M, group, rank, present, x_bytes, y_bytes, lora_bytes):
    """(bytes without x, flops) of one projection."""
    return (N * K / 2 + 2 * N * (K // group) + y_bytes * M * N + lora_bytes * present * rank * (K + N), 2.0 * M * N * K + 2.0 * M * rank * (K + N))


def _attention_work(case, heads, kv_heads, dim, prefix, y_bytes):
    parent, forecast, tokens = _tree(_branch(case["branch"]), case["forecast"])
    S, R = case["streams"], len(parent)
    keys = case["prefill"] + prefix + S * (case["cap"] / 2 + R)
    seen = S * R * (case["prefill"] + case["cap"] / 2 + 2) + S * sum(forecast) * prefix
    return 4.0 * keys * kv_heads * dim + (2 + y_bytes) * S * R * heads * dim, 4.0 * seen * heads * dim


def work(case):
    kind = case["kind"]
    if kind in ("linear", "layers", "layers_a8"):
        M, present = case["M"], _present(case, case["M"], case["adapters"])
        y_bytes, x_bytes = 4 if case["y"] == "fp32" else 2, 1 if kind == "layers_a8" else 2
        total, flops, slots = 4.0 * M, 0.0, set()
        for _, K, N, slot, n in _projections(case):
            b, f = _projection_work(K, N, M, case["group"], case["rank"], present, x_bytes, y_bytes, 2)
            total, flops = total + n * b, flops + n * f
            if slot not in slots:
                slots.add(slot)
                total += n * x_bytes * M * K
        return {"bytes": total, "flops": flops}
    if kind == "attention":
        b, f = _attention_work(case, case["heads"], case["kv_heads"], case["dim"], case["prefix"], 4 if case["y"] == "fp32" else 2)
        return {"bytes": b, "flops": f}
    parent, forecast, T = _tree(_branch(case["branch"]), case["forecast"])
    if kind == "ds2d":
        rows = case["streams"] * T * (1 + len(_branch(case["next"])))   # of the forecast rows only those a next level may draw from
        return {"bytes": float(rows * case["vocab"] * (4 if case["y"] == "fp32" else 2)), "flops": 0.0}
    M = case["streams"] * len(parent)
    total, flops = _attention_work(case, case["hidden"] // 64, case["kv_heads"], 64, 0, 2)
    present = min(case["streams"], case["adapters"])
    for name, K, N, pair in _decoder_case(case):
        # (the fused pair of gate and up: each of the two has a rank of its own)
        b, f = _projection_work(K, N // pair, M, case["group"], case["rank"], present, 2, 2, 2)
        total, flops = total + pair * b, flops + pair * f
    # rows in and between the calls: h and h2 (each read twice), attention output, MLP rows
    total += 2.0 * M * (5 * case["hidden"] + case["ffn"])
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] == "ds2d":
        return "exact"
    if case["kind"] == "decoder":
        return {"rel": 1.2e-2, "max": 5e-2}              # bf16 rows between the calls
    if case["y"] == "fp32":
        # four times the largest error against float64 seen over the ranges: 4.5e-6 (few inputs, many ranks) and 8.8e-6
        return {"rel": 2e-5, "max": 1.2e-4} if case["kind"] == "linear" else {"rel": 3.5e-5, "max": 2e-4}
    return {"rel": 7e-3, "max": 1.6e-2}                  # bf16 outputs: half a unit in the last place, four times over


# ------------------------------------------------------------------------------------------
# the same outputs in float64
# ------------------------------------------------------------------------------------------
def _exact_projection(case, x, rows, codes, scale, a, b, alpha):
    """x W^T + alpha * B (A x) in float64, x [M][K] float64, rows a CPU array of adapter indices."""
    group = codes.shape[1] // scale.shape[1]
    w = codes.double().view(scale.shape[0], scale.shape[1], group) * scale.double()[:, :, None]
    y = x @ w.view(codes.shape).t()
    if isinstance(a, tuple):
        (a, s_a), (b, s_b) = a, b
        alpha = alpha * s_a * s_b
    for ad in sorted(set(rows.tolist()) - {-1}):
        at = torch.from_numpy(np.nonzero(rows == ad)[0]).to(DEVICE)
        y[at] += alpha * ((x[at] @ a[ad].double().t()) @ b[ad].double().t())
    return y


def _exact_attention(t, q, k_new, v_new, heads, kv_heads, dim):
    """q [M][heads][dim], k_new / v_new [M][kv_heads][dim], all float64 -> [M][heads][dim]."""
    S, R, G = t["S"], t["R"], heads // kv_heads
    see = torch.zeros((R, R), dtype=torch.bool, device=DEVICE)
    for r in range(R):
        u = r
        while u >= 0:
            see[r, u] = True
            u = t["parent"][u]
    fc = torch.tensor(t["forecast"], dtype=torch.bool, device=DEVICE)
    out = torch.empty((S * R, heads, dim), dtype=torch.float64, device=DEVICE)
    for s in range(S):
        n, own = int(t["len_stream"][s]), slice(s * R, (s + 1) * R)
        Lp, Lf = t["k_prefill"].shape[1], t["k_fprefix"].shape[1]
        visible = torch.cat([torch.ones((R, Lp), dtype=torch.bool, device=DEVICE), fc[:, None].expand(R, Lf),
                             torch.ones((R, n), dtype=torch.bool, device=DEVICE), see], dim=1)
        for hk in range(kv_heads):
            k = torch.cat([t["k_prefill"][hk].double(), t["k_fprefix"][hk].double(), t["k_stream"][s, hk, :n].double(), k_new[own, hk]])
            v = torch.cat([t["v_prefill"][hk].double(), t["v_fprefix"][hk].double(), t["v_stream"][s, hk, :n].double(), v_new[own, hk]])
            for h in range(hk * G, (hk + 1) * G):
                p = (q[own, h] @ k.t() / math.sqrt(dim)).masked_fill(~visible, float("-inf")).softmax(dim=1)
                out[own, h] = p @ v
    return out


def _exact_decoder(case, seed):
    t = _decoder_inputs(case, seed)
    rows, h = t["rows"].cpu().numpy(), t["h"].double()
    project = lambda name, x: _exact_projection(case, x, rows, *t["projections"][name][2:], 2.0)  # noqa: E731
    norm = lambda x: x / torch.sqrt((x * x).mean(dim=1, keepdim=True) + EPS)  # noqa: E731
    cos, sin = t["cos"].double()[:, None, :], t["sin"].double()[:, None, :]

    def rope(x):
        x = x.view(x.shape[0], -1, 64)
        return torch.cat([x[..., :32] * cos - x[..., 32:] * sin, x[..., 32:] * cos + x[..., :32] * sin], dim=2)

    # (the norm's weight is folded into the projections: the LoRA term sees the normalised rows too)
    q, k = rope(project("q", norm(h))), rope(project("k", norm(h)))
    v = project("v", norm(h)).view(h.shape[0], -1, 64)
    attn = _exact_attention(t, q, k, v, case["hidden"] // 64, case["kv_heads"], 64)
    h2 = h + project("o", attn.reshape(h.shape))
    gu = project("gate_up", norm(h2)).view(h.shape[0], -1, 2, 32)
    act = (torch.nn.functional.silu(gu[:, :, 0]) * gu[:, :, 1]).reshape(h.shape[0], -1)
    out = h2 + project("down", act)
    pad = torch.nn.functional.pad(out, (0, -out.shape[1] % 64)).view(out.shape[0], -1, 64)
    return {"out": out, "k": k, "v": v, "squares": (pad * pad).sum(dim=2)}


def exact(case, seed):
    if case["kind"] == "ds2d":
        return None                                       # token ids and row numbers
    if case["kind"] == "decoder":
        return _exact_decoder(case, seed)
    if case["kind"] == "attention":
        t = _attention_inputs(case, seed, case["heads"], case["kv_heads"], case["dim"], case["prefix"])
        return _exact_attention(t, t["q"].double(), t["k_new"].double(), t["v_new"].double(), case["heads"], case["kv_heads"], case["dim"])
    M = case["M"]
    rows = _rows(case, seed, M, case["adapters"]).cpu().numpy()
    out = {name: torch.empty((n, M, N), dtype=torch.float64, device=DEVICE) for name, _, N, _, n in _projections(case)}
    for layer in range(case.get("layers", 1)):
        for index, (name, K, N, slot, _) in enumerate(_projections(case)):
            x = _x(case, seed, layer, slot, M, K)
            x = x[0].double() * x[1] if isinstance(x, tuple) else x.double()
            out[name][layer] = _exact_projection(case, x, rows, *_projection_inputs(case, seed, layer, index, K, N, case["rank"], case["adapters"]),
                                                 case["alpha"])
    return out
