"""Timed cases of the LoRA-delta library: the layer calls that a LoRA server makes, through the
library's public entry points, over the sizes it meets.

A case is one layer's worth of calls on one batch: the segment build and every projection of the
layer (dense: q/k/v, output, gate/up and down, or fewer; MoE: gate/up and down per expert), or the
loading of one adapter's layer and the small decode call that waits for it.  Every state holds a
pool of its own in HBM, ids, activations and base outputs; a pass adds the update to the base outputs
in place, as a server does after its base GEMMs.

Fields of a case:
  kind       "dense", "moe" or "load" (one adapter's layer repacked into its slot, then a MoE call)
  tokens     rows of the batch (dense) or tokens, each routed to top_k experts (moe)
  adapters, rank, experts, top_k, hidden, ffn, kv      shapes (kv: width of k and v)
  projs      dense: "one" (hidden x ffn), "two" (hidden x hidden and hidden x ffn), "layer" (all seven)
  ids        adapter ids: "uniform", "zipf" (exponent `zipf`), "requests" (`requests` contiguous runs
             of uneven length) or "mixed" (one long prompt, the rest zipf decode tokens)
  none       share of the tokens without adapter
  mixed_ranks    every other adapter has half the pool's rank
  f32        fp32 base outputs instead of bf16
  fused_out  the outputs of a group are column ranges of one buffer (q|k|v, gate|up)
  combine    MoE: the down projection ends in the routing-weighted sum of a token's experts
"""
import numpy as np
import torch

import paper_2604_07173_amd as L

_DEFAULTS = dict(kind="dense", projs="layer", tokens=64, adapters=4, rank=16, experts=1, top_k=1, hidden=4096,
                 ffn=14336, kv=1024, ids="zipf", zipf=1.0, requests=0, none=0.0, mixed_ranks=False, f32=False,
                 fused_out=False, combine=False)


def _case(name=None, **kw):
    unknown = set(kw) - set(_DEFAULTS)
    if unknown:
        raise ValueError(f"unknown fields {sorted(unknown)}")
    c = dict(_DEFAULTS, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one narrow projection of a small batch: latency of a single call
        _case("dense_small", projs="one", tokens=64, adapters=4, rank=8, hidden=1024, ffn=1024, ids="uniform"),
        # a Llama-3-8B-shaped layer with a handful of interactive users
        _case("llama_decode_8", tokens=8, adapters=64),
        # the same layer at a full decode batch
        _case("llama_decode_256", tokens=256, adapters=64),
        # odd widths and an odd batch, fp32 base outputs in fused buffers, adapters of two ranks, some
        # rows without adapter
        _case("dense_ragged_f32", tokens=333, adapters=24, rank=32, hidden=2568, ffn=6920, kv=648, none=0.1,
              mixed_ranks=True, f32=True, fused_out=True),
        # chunked prefill: one prompt takes most of the batch, decode tokens of other users the rest
        _case("llama_mixed_2048", tokens=2048, adapters=64, ids="mixed"),
        # prefill of eight requests of about 2048 tokens at rank 64
        _case("prefill_16384", projs="two", tokens=16384, adapters=8, rank=64, ids="requests", requests=8),
        # Mixtral-8x7B-shaped MoE decode: a small batch with the routing-weighted down projection,
        # a full decode batch, and a batch of many decode or prompt tokens
        _case("mixtral_combine_64", kind="moe", tokens=64, adapters=32, experts=8, top_k=2, combine=True),
        _case("mixtral_decode_512", kind="moe", tokens=512, adapters=32, experts=8, top_k=2),
        _case("mixtral_2048", kind="moe", tokens=2048, adapters=32, experts=8, top_k=2),
        # fine-grained MoE decode: thousands of (adapter, expert) cells with a row or two each
        _case("finegrained_1024", kind="moe", tokens=1024, adapters=256, rank=8, experts=128, top_k=8, hidden=2048,
              ffn=768, zipf=1.2),
        # the kernel-microbenchmark shape: 512 adapters at rank 64, most cells with few rows
        _case("mixtral_r64_1024", kind="moe", tokens=1024, adapters=512, rank=64, experts=8, top_k=2, zipf=1.2),
        # an adapter that was not resident: its layer, already in device memory, is repacked into
        # the slot and the decode batch that waited for it runs
        _case("adapter_load_32", kind="load", tokens=32, adapters=32, experts=8, top_k=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(float(np.exp(rng.uniform(np.log(lo), np.log(hi))))))


def _none(c):
    """Small batches have no rows without adapter, so that a drawn case always has work."""
    return dict(c, none=0.0) if c["tokens"] < 8 else c


def _width(rng, lo, hi):
    """A width: a multiple of 128 in two of three draws, else any multiple of 8."""
    w = _log_int(rng, lo, hi)
    return max(lo, w // 128 * 128 if rng.random() < 0.67 else w // 8 * 8)


def draw(rng):
    return _none(_draw(rng))


def _draw(rng):
    family = rng.choice(["one", "decode", "decode", "prompt", "moe", "moe", "fine", "load"])
    none = rng.choice([0.0, 0.0, 0.05, 0.2])
    f32 = rng.random() < 0.25
    mixed = rng.random() < 0.25
    fused = rng.random() < 0.3
    rank = rng.choice([8, 16, 16, 32, 64])
    if family == "one":
        return _case(projs="one", tokens=_log_int(rng, 1, 512), adapters=_log_int(rng, 1, 64), rank=rank,
                     hidden=_width(rng, 512, 4096), ffn=_width(rng, 512, 4096), ids=rng.choice(["uniform", "zipf"]),
                     none=none, f32=f32, mixed_ranks=mixed)
    if family == "decode":
        return _case(tokens=_log_int(rng, 1, 1024), adapters=_log_int(rng, 4, 128), rank=rank,
                     hidden=_width(rng, 1024, 4096), ffn=_width(rng, 2048, 14336), kv=_width(rng, 256, 1024),
                     ids=rng.choice(["uniform", "zipf"]), zipf=rng.choice([0.8, 1.0, 1.2]), none=none, f32=f32,
                     mixed_ranks=mixed, fused_out=fused)
    if family == "prompt":
        ids = rng.choice(["requests", "mixed"])
        return _case(projs=rng.choice(["two", "layer"]), tokens=_log_int(rng, 1024, 8192),
                     adapters=_log_int(rng, 4, 64), rank=rank, hidden=_width(rng, 1024, 4096),
                     ffn=_width(rng, 2048, 14336), kv=_width(rng, 256, 1024), ids=ids,
                     requests=_log_int(rng, 2, 32) if ids == "requests" else 0, none=0.0, f32=f32,
                     mixed_ranks=mixed, fused_out=fused)
    if family == "fine":
        return _case(kind="moe", tokens=_log_int(rng, 16, 4096), adapters=_log_int(rng, 16, 256),
                     rank=rng.choice([8, 16]), experts=rng.choice([64, 128]), top_k=rng.choice([4, 6, 8]),
                     hidden=_width(rng, 1024, 2048), ffn=_width(rng, 512, 1024), zipf=rng.choice([1.0, 1.2]),
                     none=none, combine=rng.random() < 0.3)
    return _case(kind="load" if family == "load" else "moe",
                 tokens=_log_int(rng, 1, 64) if family == "load" else _log_int(rng, 1, 2048),
                 adapters=_log_int(rng, 4, 48), rank=rank if family == "load" else rng.choice([8, 16, 32]),
                 experts=8, top_k=2, hidden=_width(rng, 2048, 4096), ffn=_width(rng, 4096, 14336),
                 zipf=rng.choice([0.8, 1.0, 1.2]), none=none, mixed_ranks=mixed,
                 combine=family == "moe" and rng.random() < 0.4)


# ---- shapes, ids and weights -----------------------------------------------------------------


def _projs(c):
    """(h_in, h_out, name of the input) per projection of the pool."""
    h, f, kv = c["hidden"], c["ffn"], c["kv"]
    if c["kind"] != "dense":
        return [(h, f, "x"), (h, f, "x"), (f, h, "mid")]
    if c["projs"] == "one":
        return [(h, f, "x")]
    if c["projs"] == "two":
        return [(h, h, "x"), (h, f, "x")]
    return [(h, h, "x"), (h, kv, "x"), (h, kv, "x"), (h, h, "attn"), (h, f, "xn"), (h, f, "xn"), (f, h, "mid")]


def _groups(c):
    """Runs of projections that read the same input: (first, count)."""
    return {"one": [(0, 1)], "two": [(0, 2)], "layer": [(0, 3), (3, 1), (4, 2), (6, 1)]}[c["projs"]]


def _ids(c, seed):
    """adapter_id and expert_id (or None) per row, token of every row, routing weights per row."""
    r = np.random.default_rng(seed)
    T, n, k = c["tokens"], c["adapters"], c["top_k"]

    def zipf(m):
        p = np.arange(1, n + 1, dtype=np.float64) ** -c["zipf"]
        return np.minimum(np.searchsorted(np.cumsum(p / p.sum()), r.random(m), side="right"), n - 1)

    if c["ids"] == "uniform":
        a = r.integers(0, n, T)
    elif c["ids"] == "zipf":
        a = zipf(T)
    elif c["ids"] == "requests":            # uneven lengths (half to one and a half times the mean)
        m = min(c["requests"], T)
        w = r.uniform(0.5, 1.5, m)
        cut = np.floor(np.cumsum(w) / w.sum() * T).astype(np.int64)
        cut[-1] = T
        a = np.searchsorted(cut, np.arange(T), side="right") % n
    else:                                   # "mixed": one prompt of 7/8 of the rows, then decode tokens
        head = T - T // 8
        a = np.concatenate([np.full(head, r.integers(0, n)), zipf(T - head)])
    a = a.astype(np.int32)
    if c["none"] > 0:
        a[r.random(T) < c["none"]] = -1
    if c["kind"] == "dense":
        return a, None, np.arange(T, dtype=np.int32), None
    logits = r.standard_normal((T, c["experts"])).astype(np.float32)
    top = np.argsort(-logits, axis=1, kind="stable")[:, :k]
    w = np.exp(np.take_along_axis(logits, top, 1))
    w = (w / w.sum(1, keepdims=True)).astype(np.float32)
    token = np.repeat(np.arange(T, dtype=np.int32), k)
    return a[token], top.reshape(-1).astype(np.int32), token, w.reshape(-1)


def _ranks(c):
    return [c["rank"] // 2 if c["mixed_ranks"] and a % 2 else c["rank"] for a in range(c["adapters"])]


def _inputs(c, seed):
    """Everything a call reads, made from the seed: ids, activations, base outputs, weights."""
    projs = _projs(c)
    a, e, token, w = _ids(c, seed)
    P, T = a.size, c["tokens"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape, dtype=torch.bfloat16, std=1.0):
        return (torch.randn(*shape, generator=g, device="cuda") * std).to(dtype)

    acts = {}
    for h_in, _, name in projs:
        if name not in acts:
            acts[name] = normal(P if name == "mid" else T, h_in)
    out = torch.float32 if c["f32"] else torch.bfloat16
    if c["kind"] == "dense":
        bases = []
        for first, n in _groups(c):
            widths = [projs[j][1] for j in range(first, first + n)]
            bases += [normal(P, sum(widths), dtype=out)] if c["fused_out"] else [normal(P, v, dtype=out) for v in widths]
    else:
        bases = [normal(P, c["ffn"]), normal(P, c["ffn"]), normal(T if c["combine"] else P, c["hidden"])]
    # weights: windows of one bank of N(0, 0.02) values, one window per adapter, laid out
    # [expert][projection]{A[h_in][r], B[r][h_out]}; windows may overlap
    need = c["experts"] * sum((i + o) * c["rank"] for i, o, _ in projs)
    bank = normal(max(1 << 24, 2 * need), std=0.02)
    r = np.random.default_rng(seed + 1)
    window = r.integers(0, (bank.numel() - need) // 8 + 1, c["adapters"]) * 8
    scale = [(0.5, 1.0, 1.5, 2.0)[i % 4] for i in range(c["adapters"])]
    return dict(a=a, e=e, token=token, w=w, acts=acts, bases=bases, bank=bank, window=window, scale=scale)


def _columns(c, bases):
    """The output of every projection: the buffers themselves, or column ranges of them."""
    if c["kind"] != "dense" or not c["fused_out"]:
        return list(bases)
    projs, ys = _projs(c), []
    for (first, n), buf in zip(_groups(c), bases):
        at = 0
        for j in range(first, first + n):
            ys.append(buf[:, at:at + projs[j][1]])
            at += projs[j][1]
    return ys


# ---- one pass -----------------------------------------------------------------------------------


def prepare(case, seed):
    """The pool with every adapter resident, and a batch's ids, activations and base outputs in HBM."""
    c = _case(**{k: v for k, v in case.items() if k != "name"})
    s = _inputs(c, seed)
    projs = _projs(c)
    ranks = _ranks(c)
    desc = L.PoolDesc(c["adapters"], 1, c["experts"], [(i, o) for i, o, _ in projs], c["rank"], scale=s["scale"],
                      adapter_rank=ranks)
    slab = torch.empty(L.lora_pool_bytes(desc), dtype=torch.uint8, device="cuda")
    pool = L.lora_register_pool(desc, slab)
    for a in range(c["adapters"]):
        L.lora_pool_load_adapter_layer(pool, a, 0, s["bank"].data_ptr() + 2 * int(s["window"][a]))
    dev = lambda v: None if v is None else torch.from_numpy(v).cuda()  # noqa: E731
    P = s["a"].size
    st = dict(case=c, pool=pool, P=P, a=dev(s["a"]), e=dev(s["e"]), token=dev(s["token"]), w=dev(s["w"]),
              acts=s["acts"], bases=s["bases"], ys=_columns(c, s["bases"]), seg=L.Segments(P), projs=projs,
              dtype=L.LORA_DTYPE_F32 if c["f32"] else L.LORA_DTYPE_BF16)
    if c["kind"] == "dense":
        n = max(L.lora_group_ws_bytes(pool, j, k, P) for j, k in _groups(c))
    else:
        n = L.lora_moe_combine_ws_bytes(pool, P) if c["combine"] else L.lora_moe_ws_bytes(pool, P)
    st["ws"] = torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
    if c["kind"] == "load":
        # the adapter that arrives: the batch's most frequent one, under its own rank and scale
        on = s["a"][s["a"] >= 0]
        slot = int(np.bincount(on).argmax()) if on.size else 0
        size = L.lora_pool_adapter_layer_bytes(pool, slot) // 2
        at = int(s["window"][slot])
        st.update(slot=slot, rank=ranks[slot], scale=s["scale"][slot], arrived=s["bank"][at:at + size].clone())
    return st


def run(st):
    """One layer's calls."""
    c, pool, seg, P, ys, acts = st["case"], st["pool"], st["seg"], st["P"], st["ys"], st["acts"]
    if c["kind"] == "dense":
        for i, (j, n) in enumerate(_groups(c)):
            x = acts[st["projs"][j][2]]
            out = ys[j:j + n]
            ld = [y.stride(0) for y in out]
            if i == 0:
                L.lora_build_apply_group(pool, 0, j, x, x.stride(0), None, st["a"], None, P, seg, out, ld, st["ws"],
                                         st["dtype"])
            else:
                L.lora_apply_group(pool, 0, j, x, x.stride(0), None, seg, out, ld, st["ws"], st["dtype"])
        return st["bases"]
    if c["kind"] == "load":
        L.lora_pool_set_adapter(pool, st["slot"], st["rank"], st["scale"])
        L.lora_pool_load_adapter_layer(pool, st["slot"], 0, st["arrived"])
    x, mid = acts["x"], acts["mid"]
    L.lora_moe_build_apply(pool, 0, L.LORA_MOE_UPGATE, x, x.stride(0), st["token"], st["a"], st["e"], P, seg, ys[0],
                           ys[1], ys[0].stride(0), st["ws"])
    if c["combine"]:
        L.lora_moe_down_combine(pool, 0, mid, mid.stride(0), st["a"], st["e"], seg, st["w"], c["top_k"], ys[2],
                                ys[2].stride(0), st["ws"])
    else:
        L.lora_moe_apply(pool, 0, L.LORA_MOE_DOWN, mid, mid.stride(0), None, seg, ys[2], None, ys[2].stride(0),
                         st["ws"])
    return st["bases"]


# ---- what a pass cannot do without, and what it should return ---------------------------------------


def work(case):
    """Touched weights read once, input rows read once, output rows read and written once, ids."""
    c = _case(**{k: v for k, v in case.items() if k != "name"})
    a, e, token, _ = _ids(c, 0)
    on = a >= 0
    projs, ranks = _projs(c), _ranks(c)
    keys = np.unique(a[on].astype(np.int64) * c["experts"] + (0 if e is None else e[on]))
    rank_rows = sum(ranks[int(k) // c["experts"]] for k in keys)          # sum of ranks over the touched units
    rank_pairs = sum(ranks[int(v)] for v in a[on])
    P, T = int(on.sum()), int(np.unique(token[on]).size)
    size = 4 if c["f32"] else 2
    n_bytes, flops, seen = 12 * a.size, 0, set()
    for i, o, name in projs:
        n_bytes += 2 * rank_rows * (i + o)
        flops += 2 * rank_pairs * (i + o)
        if name not in seen:
            n_bytes += 2 * i * (P if name == "mid" else T)
            seen.add(name)
        rows = T if c["combine"] and name == "mid" else P
        n_bytes += 2 * size * rows * o
    if c["kind"] == "load":                  # the arriving layer is read once and written once
        n_bytes += 2 * 2 * c["experts"] * c["rank"] * sum(i + o for i, o, _ in projs)
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    # y = base + update in fp32, rounded once: bf16 outputs are 1.7e-3 off in the 2-norm from that
    # rounding alone, and one step (2^-7 of the value) where two sums fall on either side of a tie;
    # the combined form rounds every expert's update to bf16 once more.  fp32 outputs carry the
    # rounding of the fp32 sums and of the two-part bf16 operand of the second product.
    if case.get("f32"):
        return {"rel": 6e-6, "max": 6e-5}
    return {"rel": 7e-3, "max": 2e-2}


def exact(case, seed):
    """The base outputs after one pass, in 64 bits."""
    c = _case(**{k: v for k, v in case.items() if k != "name"})
    s = _inputs(c, seed)
    projs, ranks = _projs(c), _ranks(c)
    bases = [b.double() for b in s["bases"]]
    ys = _columns(c, bases)
    acts = s["acts"]
    on = np.nonzero(s["a"] >= 0)[0]
    e = np.zeros_like(s["a"]) if s["e"] is None else s["e"]
    key = s["a"][on].astype(np.int64) * c["experts"] + e[on]
    order = np.argsort(key, kind="stable")
    rows, key = on[order], key[order]
    cuts = np.nonzero(np.diff(key))[0] + 1
    for part in np.split(np.arange(rows.size), cuts):
        if not part.size:
            continue
        a, ex = divmod(int(key[part[0]]), c["experts"])
        r = ranks[a]
        at = int(s["window"][a]) + ex * sum((i + o) * r for i, o, _ in projs)
        idx = torch.from_numpy(rows[part]).cuda()
        tok = torch.from_numpy(s["token"][rows[part]].astype(np.int64)).cuda()
        for j, (i, o, name) in enumerate(projs):
            A = s["bank"][at:at + i * r].view(i, r).double()
            B = s["bank"][at + i * r:at + (i + o) * r].view(r, o).double()
            at += (i + o) * r
            x = acts[name][idx if name == "mid" else tok].double()
            d = s["scale"][a] * ((x @ A) @ B)
            if c["combine"] and name == "mid":
                w = torch.from_numpy(s["w"][rows[part]]).cuda().double()
                ys[j].index_add_(0, tok, d * w[:, None])
            else:
                ys[j].index_add_(0, idx, d)
    return bases
