"""Timed cases of the library's public calls: decode steps, prefill, prefill chunks on a cache, single linears, quantizing.

A case is a dict of plain values.  "kind" says which call it times; the remaining entries are its sizes and options.
The model shapes are the ones of synth_inputs.py (7B-, 8B-GQA- and 13B-shaped decoder layers) and a generic one with
64-wide heads.  Inputs follow synth_inputs.py: weights N(0, 0.02) (1.28 / sqrt(hidden) where hidden is smaller), hidden
states and cached keys and values N(0, 1), RMSNorm gains 1 + N(0, 0.02).
"""
import math

import torch

import paper_2602_10431_amd as qt

# hidden, heads, key/value heads, head size, SwiGLU width
SHAPES = {
    "7b": (4096, 32, 32, 128, 11008),
    "8b_gqa": (4096, 32, 8, 128, 14336),
    "13b": (5120, 40, 40, 128, 13824),
    "d64_gqa": (2048, 32, 8, 64, 5632),
}
EPS, ROPE_BASE = 1e-5, 10000.0
MLP_HIDDEN = 16


def _layer_case(kind, shape, dtype, seqs, tokens, cached, mode="ratio", value=1.0, bits=4, group=128, layers=1,
                ragged=False, router="linear", keep=True):
    return dict(kind=kind, shape=shape, dtype=dtype, seqs=seqs, tokens=tokens, cached=cached, mode=mode, value=value,
                bits=bits, group=group, layers=layers, ragged=ragged, router=router, keep=keep)


def listed():
    return [
        # one user in a chat: the smallest call there is, one token on a short context
        dict(name="decode_1x700_7b", **_layer_case("layer", "7b", "fp16", 1, 1, 700)),
        # a few users, whole calls through several layers (every token executes, so that the selection of a later
        # layer does not hang on the last bit of an earlier one)
        dict(name="decode_stack4_8x1500_gqa", **_layer_case("stack", "8b_gqa", "bf16", 8, 1, 1500, layers=4, ragged=True)),
        # half of the tokens of an ordinary serving batch skip the layer
        dict(name="decode_33x3000_gqa_r60", **_layer_case("layer", "8b_gqa", "bf16", 33, 1, 3000, value=0.6, ragged=True)),
        # the decode batch of bench.py
        dict(name="decode_64x2048_7b", **_layer_case("layer", "7b", "fp16", 64, 1, 2048)),
        # a large decode batch of the wide shape, the threshold decides
        dict(name="decode_128x1536_13b_th", **_layer_case("layer", "13b", "bf16", 128, 1, 1536, mode="threshold", value=0.45)),
        # one prompt, written to an empty cache
        dict(name="prefill_1x1000_7b_r50", **_layer_case("layer", "7b", "bf16", 1, 1000, 0, value=0.5)),
        # the next piece of two long prompts on top of what is cached, 64-wide heads, small groups, two-output router
        dict(name="chunk_2x700_on_1400_d64", **_layer_case("layer", "d64_gqa", "fp16", 2, 700, 1400, value=0.8, group=32,
                                                            ragged=True, router="mlp")),
        # prompts of mixed lengths in one call, 3-bit weights, the threshold decides
        dict(name="prefill_12x420_13b_w3_th", **_layer_case("layer", "13b", "fp16", 12, 420, 0, mode="threshold", value=0.5,
                                                             bits=3, ragged=True)),
        # the prefill batch of bench.py: no cache, half of the tokens execute
        dict(name="prefill_8x1024_7b_r50", **_layer_case("layer", "7b", "bf16", 8, 1024, 0, value=0.5, keep=False)),
        # long prompts, the largest call
        dict(name="prefill_4x4096_gqa_r60", **_layer_case("layer", "8b_gqa", "bf16", 4, 4096, 0, value=0.6, keep=False)),
        # the MLP's first half alone at a row count between decode and prefill
        dict(name="swiglu_150_7b", kind="swiglu", shape="7b", rows=150, bits=4, group=128),
        # loading a model: one of its largest linears is quantized and laid out
        dict(name="quantize_7b_gate", kind="quantize", n=11008, k=4096, bits=4, group=128),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    pick = rng.random()
    bits = rng.choice([4, 4, 4, 3, 2])
    group = rng.choice([128, 128, 64, 32])
    shape = rng.choice(sorted(SHAPES))
    if pick < 0.12:
        return dict(kind=rng.choice(["swiglu", "linear"]), shape=shape, rows=_log(rng, 1, 6000), bits=bits, group=group)
    if pick < 0.2:
        return dict(kind="quantize", n=8 * _log(rng, 64, 1700), k=8 * _log(rng, 64, 1700), bits=bits, group=group)
    dtype = rng.choice(["fp16", "bf16"])
    mode = rng.choice(["ratio", "ratio", "threshold"])
    value = round(rng.uniform(0.3, 0.55), 2) if mode == "threshold" else rng.choice([1.0, round(rng.uniform(0.25, 1.0), 2)])
    common = dict(mode=mode, value=value, bits=bits, group=group, ragged=rng.random() < 0.6,
                  router="mlp" if mode == "ratio" and rng.random() < 0.3 else "linear")
    if pick < 0.62:
        seqs = _log(rng, 1, 128)
        if rng.random() < 0.25:
            common.update(mode="ratio", value=1.0)                 # see decode_stack4 above
            return _layer_case("stack", shape, dtype, seqs, 1, _log(rng, 100, 1500), layers=rng.choice([2, 3, 4]), **common)
        return _layer_case("layer", shape, dtype, seqs, 1, _log(rng, 100, 4000 if seqs <= 64 else 1500), **common)
    if pick < 0.74:
        seqs = _log(rng, 1, 8)
        return _layer_case("layer", shape, dtype, seqs, _log(rng, 60, 4000 // seqs), _log(rng, 100, 3000), **common)
    seqs = _log(rng, 1, 16)
    tokens = _log(rng, 60, min(4000, 6500 // seqs))
    return _layer_case("layer", shape, dtype, seqs, tokens, 0, keep=rng.random() < 0.5, **common)


# ---- sizes that follow from a case -------------------------------------------------------------------------------
def _linears(shape):
    H, nh, nkv, d, I = SHAPES[shape]
    return [("q", nh * d, H), ("k", nkv * d, H), ("v", nkv * d, H), ("o", H, nh * d), ("gate", I, H), ("up", I, H), ("down", H, I)]


def _spread(n, count, ragged):
    """`count` lengths: all n, or spread evenly from n / 2 to 3 n / 2 (the same total whatever the order)."""
    if not ragged or count == 1:
        return [n] * count
    return [max(1, n // 2 + (n * i) // (count - 1)) for i in range(count)]


def _lengths(case, gen=None):
    new = _spread(case["tokens"], case["seqs"], case["ragged"] and case["tokens"] > 1)
    old = _spread(case["cached"], case["seqs"], case["ragged"]) if case["cached"] else [0] * case["seqs"]
    if gen is not None:                                          # which sequence is the long one changes with the inputs
        new = [new[i] for i in torch.randperm(len(new), generator=gen).tolist()]
        old = [old[i] for i in torch.randperm(len(old), generator=gen).tolist()]
    return new, old


def _std(hidden):
    return max(0.02, 1.28 / math.sqrt(hidden))


def _share(case):
    """Expected share of executed tokens."""
    if case["mode"] == "ratio":
        return case["value"]
    H = SHAPES[case["shape"]][0]
    logit = math.log(case["value"] / (1.0 - case["value"]))
    return 0.5 * math.erfc(logit / (_std(H) * math.sqrt(H)) / math.sqrt(2.0))


def _weight_bytes(n, k, bits, group):
    return n * k * bits / 8 + 4 * n * math.ceil(k / group)


def work(case):
    if case["kind"] == "quantize":
        n, k = case["n"], case["k"]
        out = n * k * case["bits"] / 8
        return {"bytes": 4 * n * k + 2 * out + 8 * n * math.ceil(k / case["group"]), "flops": 0}
    H, nh, nkv, d, I = SHAPES[case["shape"]]
    if case["kind"] in ("swiglu", "linear"):
        m = case["rows"]
        mats, n, k = (2, I, H) if case["kind"] == "swiglu" else (1, H, I)
        return {"bytes": mats * _weight_bytes(n, k, case["bits"], case["group"]) + 2 * m * (k + n), "flops": 2 * m * mats * n * k}
    new, old = _lengths(case)
    T, share = sum(new), _share(case)
    rows = share * T
    bytes_, flops = 0.0, 0.0
    for _, n, k in _linears(case["shape"]):
        bytes_ += _weight_bytes(n, k, case["bits"], case["group"])
        flops += 2 * rows * n * k
    bytes_ += 2 * T * H + 2 * rows * H + 4 * H                     # all rows are scored, executed rows are written
    if case["router"] == "mlp":
        bytes_ += 4 * MLP_HIDDEN * H
        flops += 2 * T * MLP_HIDDEN * H
    for a, o in zip(new, old):
        n = share * a
        seen = n * o + n * n / 2                                 # (query, key) pairs of the causal triangle on top of the cache
        flops += 4 * seen * nh * d
        if case["keep"]:
            live = share if a == 1 else 1.0                       # a bypassed decode token reads nothing
            bytes_ += 4 * (live * o + n) * nkv * d
    return {"bytes": bytes_ * case["layers"], "flops": flops * case["layers"]}


# ---- inputs ----------------------------------------------------------------------------------------------------
def _rng(seed, slot):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + slot * 7919) % (1 << 62))
    return g


def _randn(gen, *size, dtype=torch.float32):
    return torch.randn(*size, generator=gen, device="cuda", dtype=dtype)


def _act(case):
    return torch.float16 if case["dtype"] == "fp16" else torch.bfloat16


def _raw_layer(case, seed, layer):
    """The unquantized tensors of a layer, one at a time: (name, tensor)."""
    H = SHAPES[case["shape"]][0]
    std = _std(H)
    for i, (name, n, k) in enumerate(_linears(case["shape"])):
        yield name, _randn(_rng(seed, 100 * layer + i), n, k) * std
    g = _rng(seed, 100 * layer + 10)
    yield "g1", (1.0 + 0.02 * _randn(g, H)).to(_act(case))
    yield "g2", (1.0 + 0.02 * _randn(g, H)).to(_act(case))
    yield "router_w", _randn(g, H) * std
    if case["router"] == "mlp":
        R = MLP_HIDDEN
        yield "router_mlp", (_randn(g, R, H) * std, _randn(g, R) * std, _randn(g, 2, R) * 0.25, _randn(g, 2) * std)


def _inputs(case, seed):
    """Hidden states, sequence offsets, positions, cached lengths, and the caches' contents per layer."""
    H, nh, nkv, d, I = SHAPES[case["shape"]]
    new, old = _lengths(case, torch.Generator().manual_seed(int(seed) % (1 << 62)))
    x = _randn(_rng(seed, 1001), sum(new), H).to(_act(case))
    offs = torch.tensor([0] + new, dtype=torch.int32).cumsum(0).to(torch.int32)
    pos = torch.cat([torch.arange(o, o + a, dtype=torch.int32) for a, o in zip(new, old)])
    caches = []
    if case["keep"]:
        cap = (max(new) + max(old) + 63) // 64 * 64
        for l in range(case["layers"]):
            g = _rng(seed, 2000 + l)
            caches.append(tuple(_randn(g, case["seqs"], nkv, cap, d, dtype=torch.float16) for _ in range(2)))
    return x, offs, pos, old, caches


def prepare(case, seed):
    if case["kind"] == "quantize":
        return dict(case=case, w=_randn(_rng(seed, 0), case["n"], case["k"]) * 0.02)
    H, nh, nkv, d, I = SHAPES[case["shape"]]
    if case["kind"] in ("swiglu", "linear"):
        n, k = (I, H) if case["kind"] == "swiglu" else (H, I)
        lins = [qt.qtale_quantize(_randn(_rng(seed, i), n, k) * _std(H), case["bits"], case["group"])
                for i in range(2 if case["kind"] == "swiglu" else 1)]
        a = _randn(_rng(seed, 10), case["rows"], k).to(torch.float16)
        out = torch.empty(case["rows"], n, dtype=torch.float16, device="cuda")
        return dict(case=case, lins=lins, a=a, out=out)
    layers = [qt.quantize_layer(dict(_raw_layer(case, seed, l)), case["bits"], case["group"], keep_canonical=False)
              for l in range(case["layers"])]
    x, offs, pos, old, caches = _inputs(case, seed)
    T, B, L = x.shape[0], case["seqs"], case["layers"]
    # What a step brings is staged in one buffer: the rows of the step's tokens and the caches' lengths.  A pass moves
    # it to where the call works on it in place, as a serving loop does with every step's inputs.
    x_bytes = x.numel() * 2
    staged = torch.empty(x_bytes + 4 * L * B, dtype=torch.uint8, device="cuda")
    staged[:x_bytes] = x.reshape(-1).view(torch.uint8)
    staged[x_bytes:] = torch.tensor([old] * L, dtype=torch.int32, device="cuda").reshape(-1).view(torch.uint8)
    live = torch.empty_like(staged)
    x = live[:x_bytes].view(_act(case)).view(T, H)
    kv_len = live[x_bytes:].view(torch.int32).view(L, B)
    kvs = [qt.KVCache(k, v, kv_len[l]) for l, (k, v) in enumerate(caches)] or None
    cfg = qt.make_cfg(H, nh, nkv, d, I, case["bits"], case["group"], case["dtype"], EPS, ROPE_BASE)
    ctx = qt.Context()
    (qt.qtale_set_exec_ratio if case["mode"] == "ratio" else qt.qtale_set_threshold)(ctx, case["value"])
    return dict(case=case, ctx=ctx, cfg=cfg, layers=layers, kvs=kvs, stack=qt.Stack(cfg, layers, kvs) if case["kind"] == "stack" else None,
                staged=staged, live=live, x=x, kv_len=kv_len, offs=offs.cuda(), pos=pos.cuda(),
                idx=torch.full((L, T), -1, dtype=torch.int32, device="cuda"),
                count=torch.zeros(L, dtype=torch.int32, device="cuda"), scores=torch.zeros(L, T, device="cuda"),
                workspace=qt.alloc_workspace(cfg, T, B))


def run(state):
    case = state["case"]
    if case["kind"] == "quantize":
        q = qt.qtale_quantize(state["w"], case["bits"], case["group"])
        return dict(codes=q.codes, scales=q.scales.view(torch.int16), zeros=q.zeros.view(torch.int16), prepacked=q.prepacked)
    if case["kind"] == "linear":
        return qt.qtale_linear_w4a16(state["lins"][0], state["a"], state["out"])
    if case["kind"] == "swiglu":
        return qt.qtale_swiglu_w4a16(state["lins"][0], state["lins"][1], state["a"], state["out"])
    s = state
    s["live"].copy_(s["staged"])
    if case["kind"] == "stack":
        qt.qtale_stack_forward(s["ctx"], s["stack"], s["x"], s["offs"], s["pos"], s["idx"], s["count"], s["scores"],
                               workspace=s["workspace"])
    else:
        qt.qtale_layer_forward(s["ctx"], s["cfg"], s["layers"][0], s["x"], s["offs"], s["pos"], s["kvs"][0] if s["kvs"] else None,
                               s["idx"][0], s["count"][0:1], s["scores"][0], s["workspace"])
    out = dict(x=s["x"], idx=s["idx"], count=s["count"], scores=s["scores"])
    if s["kvs"]:
        out.update(kv_len=s["kv_len"], k=[c.k for c in s["kvs"]], v=[c.v for c in s["kvs"]])
    return out


def tolerance(case):
    # About four times what was seen against exact(): 1.7e-3 with the bf16 stream (the rows' own rounding; 4.3e-3 after
    # four layers), up to 1.1e-3 with the fp16 stream, 3.8e-4 for a single linear or SwiGLU.
    if case["kind"] == "quantize":
        return "exact"
    if case["kind"] in ("swiglu", "linear"):
        return {"rel": 2e-3, "max": 3e-2}
    return {"rel": (7e-3 if case["dtype"] == "bf16" else 4e-3) * (2 if case["layers"] > 1 else 1), "max": 6e-2, "differ": 0.0}


# ---- the same results in 64 bits ------------------------------------------------------------------------------
def _quantize(w, bits, group):
    """(code - zero) * scale of the group-wise min/max quantizer, as float64, and its scale, zero and codes."""
    n, k = w.shape
    top = float(2 ** bits - 1)
    ng = (k + group - 1) // group
    g = torch.nn.functional.pad(w, (0, ng * group - k)).view(n, ng, group)          # zeros change neither bound
    lo, hi = g.amin(2).clamp(max=0.0), g.amax(2).clamp(min=0.0)
    scale = ((hi - lo) / top).to(torch.float16)
    bad = (scale == 0) | ~torch.isfinite(scale)
    scale = torch.where(bad, torch.ones_like(scale), scale)
    s = scale.float().unsqueeze(2)
    zero = (-lo.unsqueeze(2) / s).round().clamp(0.0, top)
    code = ((g / s).round() + zero).clamp(0.0, top)
    deq = (code.double() - zero.double()) * s.double()
    return deq.view(n, ng * group)[:, :k].contiguous(), code.view(n, ng * group)[:, :k], scale, zero.squeeze(2)


def _rotate(t, pos):
    """t [n, heads, d] float64, half-split pairs at absolute positions pos [n]."""
    d = t.shape[2]
    freq = ROPE_BASE ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=t.device) / d)
    ang = pos.double().unsqueeze(1) * freq.unsqueeze(0)
    c, s = ang.cos().unsqueeze(1), ang.sin().unsqueeze(1)
    lo, hi = t[..., : d // 2], t[..., d // 2:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], dim=2)


def _norm(t, gain):
    return t / torch.sqrt((t * t).mean(1, keepdim=True) + EPS) * gain.double()


def _attend(q, k, v, first):
    """q [n, nh, d] at places first .. first + n - 1 of k, v [nkv, m, d]."""
    n, nh, d = q.shape
    nkv, m = k.shape[0], k.shape[1]
    out = torch.empty_like(q)
    hidden = torch.arange(m, device=q.device).unsqueeze(0) > (first + torch.arange(n, device=q.device)).unsqueeze(1)
    for h in range(nkv):
        r = nh // nkv
        for j in range(h * r, (h + 1) * r):
            s = (q[:, j] @ k[h].t().contiguous()) / math.sqrt(d)
            out[:, j] = torch.softmax(s.masked_fill(hidden, -math.inf), 1) @ v[h]
    return out


def _layer64(case, w, x, offs, pos, old, cache):
    """One layer in float64, in place on x and on cache; returns (scores, ascending executed tokens, lengths of the caches)."""
    H, nh, nkv, d, I = SHAPES[case["shape"]]
    T = x.shape[0]
    if case["router"] == "mlp":
        w1, b1, w2, b2 = (t.double() for t in w["router_mlp"])
        z = (torch.relu(x @ w1.t() + b1) @ w2.t() + b2)
        z = (z[:, 0] - z[:, 1]).float()
    else:
        z = (x @ w["router_w"].double()).float()
    if case["mode"] == "ratio":
        k = min(T, int(math.floor(float(torch.tensor(case["value"]).float()) * T + 0.5)))
        idx = torch.sort(torch.sort(z, descending=True, stable=True)[1][:k])[0]
    else:
        t = float(torch.tensor(case["value"]).float())
        idx = torch.nonzero(z >= float(torch.tensor(math.log(t / (1.0 - t))).float())).flatten()
    lengths = list(old)
    if idx.numel() == 0:
        return z, idx, lengths
    n1 = _norm(x[idx], w["g1"])
    p = pos[idx]
    q = _rotate((n1 @ w["q"].t()).view(-1, nh, d), p)
    k = _rotate((n1 @ w["k"].t()).view(-1, nkv, d), p)
    v = (n1 @ w["v"].t()).view(-1, nkv, d)
    a = torch.empty_like(q)
    cut = torch.searchsorted(idx, offs.to(idx.dtype)).tolist()
    for b in range(len(cut) - 1):
        r0, r1 = cut[b], cut[b + 1]
        if r0 == r1:
            continue
        kb, vb = k[r0:r1].transpose(0, 1), v[r0:r1].transpose(0, 1)
        if cache is not None:
            o, e = old[b], old[b] + r1 - r0
            cache[0][b, :, o:e], cache[1][b, :, o:e] = kb, vb
            kb, vb, lengths[b] = cache[0][b, :, :e], cache[1][b, :, :e], e
        a[r0:r1] = _attend(q[r0:r1], kb.contiguous(), vb.contiguous(), kb.shape[1] - (r1 - r0))
    h = x[idx] + a.reshape(-1, nh * d) @ w["o"].t()
    n2 = _norm(h, w["g2"])
    x[idx] = h + (torch.nn.functional.silu(n2 @ w["gate"].t()) * (n2 @ w["up"].t())) @ w["down"].t()
    return z, idx, lengths


def exact(case, seed):
    if case["kind"] == "quantize":
        return None                                              # whole numbers: both sides are compared bit for bit
    if case["kind"] in ("swiglu", "linear"):
        H, nh, nkv, d, I = SHAPES[case["shape"]]
        n, k = (I, H) if case["kind"] == "swiglu" else (H, I)
        a = _randn(_rng(seed, 10), case["rows"], k).to(torch.float16).double()
        deq = [_quantize(_randn(_rng(seed, i), n, k) * _std(H), case["bits"], case["group"])[0]
               for i in range(2 if case["kind"] == "swiglu" else 1)]
        if case["kind"] == "linear":
            return a @ deq[0].t()
        return torch.nn.functional.silu(a @ deq[0].t()) * (a @ deq[1].t())
    x, offs, pos, old, caches = _inputs(case, seed)
    x, offs, pos = x.double(), offs.cuda(), pos.cuda()
    caches = [tuple(t.double() for t in c) for c in caches]
    out = dict(idx=[], count=[], scores=[], kv_len=[])
    for l in range(case["layers"]):
        w = {}
        for name, t in _raw_layer(case, seed, l):
            w[name] = _quantize(t, case["bits"], case["group"])[0] if name in ("q", "k", "v", "o", "gate", "up", "down") else t
        z, idx, lengths = _layer64(case, w, x, offs, pos, old, caches[l] if caches else None)
        out["idx"].append(torch.cat([idx.int(), torch.full((x.shape[0] - idx.numel(),), -1, dtype=torch.int32, device="cuda")]))
        out["count"].append(idx.numel())
        out["scores"].append(z.double())
        out["kv_len"].append(lengths)
    got = dict(x=x, idx=torch.stack(out["idx"]), count=torch.tensor(out["count"], dtype=torch.int32), scores=torch.stack(out["scores"]))
    if caches:
        got.update(kv_len=torch.tensor(out["kv_len"], dtype=torch.int32), k=[c[0] for c in caches], v=[c[1] for c in caches])
    return got
