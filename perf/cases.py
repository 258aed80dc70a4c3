"""Performance cases of the MPCache hot path: what a program that serves prompts has this package do.

Three kinds of call, all through the package's public entry points:

  prefill   MPCachePath.prefill: look-once static eviction of a prompt and the cluster representatives
            of the kept cache, for a block of layers (a whole model, one sharing block, one layer);
  decode    one decode step over such a block: the two calls of MPCachePath.decode ("two") or the one
            call of MPCachePath.decode_fused ("one");
  generate  a run of decoded tokens on a growing cache: append, select, attend per token, starting
            near the end of the tail so that one of the appends seals a cluster.

Sizes are those of the synthetic workloads of this repository (GPT-2, LLaMA-2-7B and a grouped-query
shape, 512 to 128K tokens), or lie between them; budgets follow the same rules.
"""
import math

import torch

import paper_2501_06807_amd as M

DTYPE = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
ALPHA = 0.6

_BASE = dict(layer0=0, similarity="linear", group="sum", mode="two", tokens=0)


def _case(**kw):
    return dict(_BASE, **kw)


def listed():
    return [
        # the smallest call: one layer of a small model, a short prompt, fp32; launches and latency
        _case(name="prefill-tiny-512", kind="prefill", L=1, B=1, Hq=12, Hkv=12, d=64, dtype="fp32", T=512, ratio=0.5,
              eta=0.5, cluster=16, fanout=4, period=1),
        # a GPT-2 sized model (head dim 64, fp16), all layers of a 2K prompt in one call
        _case(name="prefill-2k-gpt2", kind="prefill", L=12, B=1, Hq=12, Hkv=12, d=64, dtype="fp16", T=2048, ratio=0.5,
              eta=0.125, cluster=16, fanout=4, period=2),
        # one layer at a time, as a model's forward pass produces q, k, v; a prompt of odd length
        _case(name="prefill-layer-7177", kind="prefill", layer0=2, L=1, B=1, Hq=32, Hkv=32, d=128, dtype="bf16",
              T=7177, ratio=0.5, eta=0.10, cluster=32, fanout=8, period=4),
        # the LLaMA-2-7B shape, 8K tokens, all 32 layers in one call
        _case(name="prefill-8k-7b", kind="prefill", L=32, B=1, Hq=32, Hkv=32, d=128, dtype="bf16", T=8192, ratio=0.5,
              eta=0.10, cluster=32, fanout=8, period=4),
        # four 32K prompts, one block of layers that share a kept set
        _case(name="prefill-32k-b4", kind="prefill", layer0=2, L=4, B=4, Hq=32, Hkv=32, d=128, dtype="bf16", T=32768,
              ratio=0.30, eta=0.05, cluster=32, fanout=8, period=4),
        # the longest prompt, grouped query heads, one sharing block
        _case(name="prefill-128k-gqa", kind="prefill", layer0=2, L=4, B=1, Hq=32, Hkv=8, d=128, dtype="bf16", T=131072,
              ratio=0.25, eta=0.02, cluster=64, fanout=8, period=4),
        # eight short summarisation prompts, small clusters, pairs of layers sharing
        _case(name="prefill-xsum-b8", kind="prefill", L=32, B=8, Hq=32, Hkv=32, d=128, dtype="bf16", T=1024, ratio=0.5,
              eta=0.10, cluster=4, fanout=2, period=2),
        # a decode step of one layer, as inside a model's own layer loop
        _case(name="decode-layer-8k", kind="decode", layer0=2, L=1, B=1, Hq=32, Hkv=32, d=128, dtype="bf16", T=8192,
              ratio=0.5, eta=0.10, cluster=32, fanout=8, period=4, mode="one"),
        # four tokens generated on a growing 8K cache, all 32 layers
        _case(name="generate-8k-7b", kind="generate", L=32, B=1, Hq=32, Hkv=32, d=128, dtype="bf16", T=8192, ratio=0.5,
              eta=0.10, cluster=32, fanout=8, period=4, tokens=4),
        # the decode step of four 32K sequences: the bandwidth-bound headline step
        _case(name="decode-32k-b4", kind="decode", L=32, B=4, Hq=32, Hkv=32, d=128, dtype="bf16", T=32768, ratio=0.30,
              eta=0.05, cluster=32, fanout=8, period=4),
        # the decode step of one 128K sequence with grouped query heads
        _case(name="decode-128k-gqa", kind="decode", L=32, B=1, Hq=32, Hkv=8, d=128, dtype="bf16", T=131072, ratio=0.25,
              eta=0.02, cluster=64, fanout=8, period=4, mode="one"),
        # the decode step of eight short prompts: selection over many small clusters outweighs attention
        _case(name="decode-xsum-b8", kind="decode", L=32, B=8, Hq=32, Hkv=32, d=128, dtype="bf16", T=1024, ratio=0.5,
              eta=0.10, cluster=4, fanout=2, period=2),
    ]


def draw(rng):
    """One more case of the same ranges: any of the three kinds, 300 to 128K tokens, odd lengths, every
    element type, head dim, group size and sharing period; sized down to the largest listed case."""
    kind = rng.choice(["prefill", "prefill", "prefill", "decode", "decode", "generate"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "fp16", "fp16", "fp32"])
    d = rng.choice([64, 128, 128])
    Hkv = rng.choice([2, 4, 8, 8, 12, 16, 32])
    G = rng.choice([1, 1, 2, 4, 8])
    while Hkv * G > 64:
        G //= 2
    T = int(300 * math.exp(rng.random() * math.log(131072 / 300))) | rng.choice([0, 1, 1])
    ratio = rng.choice([0.25, 0.3, 0.5, 0.6])
    cluster = rng.choice([4, 8, 16, 24, 32, 64])
    while ratio * T / cluster > 900:  # the selection ranks at most 1024 candidates
        cluster *= 2
    L, B = rng.choice([1, 1, 2, 4, 7, 12, 32]), rng.choice([1, 1, 2, 3, 4, 8])
    c = _case(kind=kind, layer0=rng.choice([0, 2, 2]), L=L, B=B, Hq=Hkv * G, Hkv=Hkv, d=d, dtype=dtype, T=T, ratio=ratio,
              eta=rng.choice([0.02, 0.05, 0.1, 0.125, 0.25]), cluster=cluster, fanout=rng.choice([2, 4, 8]),
              period=rng.choice([1, 2, 4]))
    if kind == "prefill":
        c["similarity"] = rng.choice(["linear", "linear", "linear", "mean", "maxprod"])
    else:
        c["similarity"] = rng.choice(["linear", "linear", "linear", "linear", "mean", "maxprod"])
        c["group"] = rng.choice(["sum", "sum", "sum", "max", "head"]) if G > 1 else "sum"
        c["mode"] = rng.choice(["one", "two"])
        c["tokens"] = rng.choice([2, 3, 5]) if kind == "generate" else 0
    # the largest listed prefill scores 1.34e13 flop in 16 bits (an eighth of that rate in fp32)
    while (kind == "prefill" and _score_flops(c) > (1.2e13 if dtype != "fp32" else 8e11)) or _cache_bytes(c) > 12e9:
        if c["B"] > 1:
            c["B"] -= 1
        elif c["L"] > 1:
            c["L"] = c["L"] // 2
        elif c["Hkv"] > 2:
            c["Hkv"], c["Hq"] = c["Hkv"] // 2, c["Hq"] // c["Hkv"] * (c["Hkv"] // 2)
        else:
            c["T"] = c["T"] * 3 // 4
    return c


# ------------------------------------------------------------------ sizes
def _sizes(c):
    """Window rows, kept tokens, clusters, super-clusters and budgets: 20% of the prompt scores (10% above
    24K tokens), whole clusters are kept, half the super-clusters survive level 1 below a 0.5 ratio."""
    T, s, f = c["T"], c["cluster"], c["fanout"]
    W = max(1, int((0.1 if T > 24 * 1024 else 0.2) * T))
    keep = max(1, int(c["ratio"] * T / s)) * s
    C = keep // s
    S = -(-C // f)
    k_super = S if c["eta"] >= 0.5 else -(-S // 2)
    least = k_super * f - (f - 1)  # candidates when a last super-cluster of one cluster is among them
    k_clusters = max(1, min(int(c["eta"] * keep / s), least))
    return dict(W=W, keep=keep, local=min(32, keep), C=C, S=S, k_super=k_super, k_clusters=k_clusters)


def _owner(l, period, start=2):
    return l if period <= 1 or l < start else start + period * ((l - start) // period)


def _owners(c):
    """Local layers that select for themselves."""
    return [l for l in range(c["L"]) if _owner(c["layer0"] + l, c["period"]) == c["layer0"] + l]


def _owned_before(c):
    """Local layers whose owner precedes the block (their kept set or selection is an input)."""
    return [l for l in range(c["L"]) if _owner(c["layer0"] + l, c["period"]) < c["layer0"]]


def _elt(c):
    return 4 if c["dtype"] == "fp32" else 2


def _score_flops(c):
    W, T = _sizes(c)["W"], c["T"]
    return 2.0 * c["d"] * c["B"] * c["Hq"] * len(_owners(c)) * (W * (T - W) + W * (W + 1) / 2)


def _cache_bytes(c):
    rows = c["T"] if c["kind"] == "prefill" else _sizes(c)["keep"]
    return 2.0 * c["L"] * c["B"] * c["Hkv"] * rows * c["d"] * _elt(c)


def work(c):
    z, e, d = _sizes(c), _elt(c), c["d"]
    n_own, heads, all_heads = len(_owners(c)), c["B"] * c["Hkv"], c["L"] * c["B"] * c["Hkv"]
    R = 2 if c["similarity"] == "maxprod" else 1
    if c["kind"] == "prefill":
        b = n_own * c["B"] * c["Hq"] * z["W"] * (d * e + 4)  # window queries in, row log-sum-exp out
        b += n_own * heads * c["T"] * (d * e + 4)  # every key of the owner layers in, token scores out
        b += (c["L"] - n_own) * heads * z["keep"] * d * e  # kept keys of the other layers in
        b += all_heads * z["keep"] * (3 * d * e + 4)  # kept values in, kept keys and values and positions out
        b += n_own * heads * (z["C"] + z["S"]) * R * d * 4
        return {"bytes": b, "flops": _score_flops(c)}
    per_head = c["group"] == "head"
    lists = c["Hq"] if per_head else c["Hkv"]
    G = c["Hq"] // lists
    rows = z["k_clusters"] * c["cluster"]
    sel = n_own * c["B"] * lists * ((z["S"] + z["k_super"] * c["fanout"]) * R * d * 4 + G * d * e)
    sel += c["L"] * c["B"] * lists * z["k_clusters"] * 8
    unit = 2 * d * e + 4
    if c["kind"] == "decode":
        att = c["L"] * c["B"] * (lists * 2 * rows * d * e + c["Hq"] * unit)
        return {"bytes": sel + att, "flops": 4.0 * c["L"] * c["B"] * c["Hq"] * rows * d}
    n, s = c["tokens"], c["cluster"]
    tail = sum(_tail_state(c, i)[1] for i in range(n))
    att = c["L"] * c["B"] * (lists * 2 * (n * rows + tail) * d * e + n * c["Hq"] * unit)
    app = n * 4 * all_heads * d * e + n_own * heads * (s * d * e + 2 * R * d * 4)
    return {"bytes": n * sel + att + app, "flops": 4.0 * c["L"] * c["B"] * c["Hq"] * (n * rows + tail) * d}


def tolerance(c):
    """Four times what the outputs were measured to be off from 64 bits. Prefill: the scores and the row
    log-sum-exp are 32-bit sums of 32-bit exponentials (2.7e-7 at most over the ranges); kept rows are copies and
    the representatives two products and a sum, and the kept sets agree (see _prompt). Decode: the selections
    agree (64-bit scores of random data), the outputs carry the rounding of their type (2.2e-7, 2.2e-4, 1.7e-3)."""
    if c["kind"] == "prefill":
        return {"rel": 1e-6}
    return {"rel": {"fp32": 1e-6, "fp16": 9e-4, "bf16": 7e-3}[c["dtype"]]}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, *shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(generator=g)


def _outliers(k, g):
    """Four outlier key channels of each kv head: as in trained models, a large offset that all tokens share
    (here eight, of either sign) and twice the usual spread."""
    shape = (k.shape[0], k.shape[1], k.shape[-1])
    ch = torch.rand(shape, generator=g, device="cuda").topk(4).indices
    scale = torch.ones(shape, device="cuda", dtype=k.dtype).scatter_(-1, ch, 2.0)
    sign = torch.where(torch.rand(ch.shape, generator=g, device="cuda") < 0.5, -8.0, 8.0).to(k.dtype)
    shift = torch.zeros(shape, device="cuda", dtype=k.dtype).scatter_(-1, ch, sign)
    k.mul_(scale[:, :, None, :]).add_(shift[:, :, None, :])


def _prompt(c, seed):
    """Window queries, keys and values of a prompt of which some tokens matter to the question: queries share
    a direction per kv head, and the keys of the relevant tokens (as many as the budget keeps, none of them in
    the last quarter of the window, whose tokens few rows see) lean towards it. So the budget's edge falls where
    few tokens score, and the kept set does not depend on the order of the sums."""
    z, g, dt = _sizes(c), _gen(seed), DTYPE[c["dtype"]]
    L, B, Hq, Hkv, d, T, W = c["L"], c["B"], c["Hq"], c["Hkv"], c["d"], c["T"], z["W"]
    q = torch.empty(L, B, Hq, W, d, dtype=dt, device="cuda")
    k = torch.empty(L, B, Hkv, T, d, dtype=dt, device="cuda")
    v = _randn(g, L, B, Hkv, T, d, dtype=dt)
    n_rel, span = z["keep"] - z["local"], T - max(z["local"], W // 4)
    for l in range(L):
        u = torch.nn.functional.normalize(_randn(g, B, Hkv, d), dim=-1)
        q[l].normal_(generator=g)
        q[l].view(B, Hkv, -1, d).add_((0.5 * math.sqrt(d) * u).to(dt)[:, :, None])
        k[l].normal_(generator=g)
        _outliers(k[l], g)
        if n_rel > 0:
            idx = torch.rand(B, Hkv, span, generator=g, device="cuda").topk(min(n_rel, span)).indices
            lean = torch.zeros(B, Hkv, T, 1, dtype=dt, device="cuda")
            lean.scatter_(2, idx[..., None], 7.0)
            for b in range(B):
                k[l, b].addcmul_(lean[b], u[b].to(dt)[:, None, :])
    return q, k, v


def _path(c, keep_scores=False, capacity=None):
    z = _sizes(c)
    return M.MPCachePath(n_layers=c["L"], batch=c["B"], n_q_heads=c["Hq"], n_kv_heads=c["Hkv"], head_dim=c["d"],
                         dtype=DTYPE[c["dtype"]], T=c["T"], window=z["W"], keep=z["keep"], local_keep=z["local"],
                         cluster=c["cluster"], fanout=c["fanout"], k_super=z["k_super"], k_clusters=z["k_clusters"],
                         share_period=c["period"], layer0=c["layer0"], alpha=ALPHA, keep_scores=keep_scores,
                         similarity=c["similarity"], group=c["group"], capacity=capacity)


def _cache(c, seed, rows):
    """Keys and values of a kept cache with room for `rows` tokens, and the generator after them."""
    g, dt = _gen(seed), DTYPE[c["dtype"]]
    shape = (c["L"], c["B"], c["Hkv"], rows, c["d"])
    k, v = _randn(g, *shape, dtype=dt), _randn(g, *shape, dtype=dt)
    for l in range(c["L"]):
        _outliers(k[l], g)
    return k, v, g


def _caller_sets(c, seed, n, width):
    """Ascending index lists for layers owned before the block, which a program passes in."""
    g = _gen(seed + 7919)
    lists = c["Hq"] if c["group"] == "head" and c["kind"] != "prefill" else c["Hkv"]
    r = torch.rand(c["B"], lists, n, generator=g, device="cuda").topk(width).indices
    return r.sort(-1).values.to(torch.int32)


def _tail_start(c):
    """Tail rows before the first append: the tail fills at the second token, the third seals it."""
    return max(0, c["cluster"] - 2)


def _tail_state(c, i):
    """(Ts, n_tail) after append i (from 0)."""
    z, s = _sizes(c), c["cluster"]
    Ts, nt = z["keep"], _tail_start(c)
    for _ in range(i + 1):
        Ts, nt = (Ts + s, 1) if nt == s else (Ts, nt + 1)
    return Ts, nt


def _capacity(c):
    return _sizes(c)["keep"] + 2 * c["cluster"] + c["tokens"]


def _new_tokens(c, g):
    dt, n = DTYPE[c["dtype"]], c["tokens"]
    kv = (n, c["L"], c["B"], c["Hkv"], c["d"])
    return (_randn(g, *kv, dtype=dt), _randn(g, *kv, dtype=dt),
            _randn(g, n, c["L"], c["B"], c["Hq"], c["d"], dtype=dt))


def prepare(c, seed):
    z = _sizes(c)
    if c["kind"] == "prefill":
        q, k, v = _prompt(c, seed)
        path = _path(c, keep_scores=True)
        for l in _owned_before(c):
            path.kept[l] = _caller_sets(c, seed, c["T"], z["keep"])
        return {"kind": "prefill", "path": path, "in": (q, k, v)}
    rows = z["keep"] if c["kind"] == "decode" else _capacity(c)
    path = _path(c, capacity=rows)
    path.k_s, path.v_s, g = _cache(c, seed, rows)
    path._prepare()
    M.mpc_build_clusters(path.k_s, path.cent, path.scent, path.cfg, Ts=z["keep"], layer0=c["layer0"])
    early = _owned_before(c)
    for l in early:
        path.sel[l] = _caller_sets(c, seed, z["C"], z["k_clusters"])
    if c["kind"] == "decode":
        q = _randn(g, c["L"], c["B"], c["Hq"], c["d"], dtype=DTYPE[c["dtype"]])
        return {"kind": "decode", "path": path, "in": (q,), "one": c["mode"] == "one"}
    kn, vn, q = _new_tokens(c, g)
    n = c["tokens"]
    return {"kind": "generate", "path": path, "in": (kn, vn, q), "one": c["mode"] == "one", "start": (z["keep"], _tail_start(c)),
            "sel": path.sel.expand(n, *path.sel.shape).contiguous(), "out": torch.empty_like(q),
            "lse": torch.empty(q.shape[:-1], dtype=torch.float32, device="cuda")}


def run(state):
    p = state["path"]
    if state["kind"] == "prefill":
        p.prefill(*state["in"])
        return {"kept": p.kept, "k": p.k_s, "v": p.v_s, "cent": p.cent, "scent": p.scent, "token_score": p.token_score,
                "row_lse": p.row_lse}
    if state["kind"] == "decode":
        if state["one"]:
            p.decode_fused(*state["in"])
        else:
            p.decode(*state["in"])
        return {"sel": p.sel, "sel_score": p.sel_score, "out": p.out, "lse": p.lse}
    (Ts, nt), (kn, vn, q) = state["start"], state["in"]
    sel, out, lse = state["sel"], state["out"], state["lse"]
    for i in range(q.shape[0]):
        Ts, nt = M.mpc_append_kv(kn[i], vn[i], p.k_s, p.v_s, p.cent, p.scent, p.cfg, Ts=Ts, n_tail=nt, layer0=p.layer0)
        if state["one"]:
            M.mpc_decode_step(q[i], p.cent, p.scent, p.k_s, p.v_s, sel[i], out[i], p.cfg, sm_scale=p.sm_scale, Ts=Ts,
                              n_tail=nt, lse=lse[i], ws=p.ws_step, layer0=p.layer0)
        else:
            M.mpc_select_clusters(q[i], p.cent, p.scent, sel[i], p.cfg, Ts=Ts, layer0=p.layer0)
            M.mpc_sparse_decode_attn(q[i], p.k_s, p.v_s, sel[i], out[i], cluster_size=p.cluster, sm_scale=p.sm_scale, Ts=Ts,
                                     n_tail=nt, lse=lse[i], ws=p.ws_decode, layer0=p.layer0)
    return {"sel": sel, "out": out, "lse": lse, "k": p.k_s, "v": p.v_s, "cent": p.cent, "scent": p.scent}


# ------------------------------------------------------------------ 64-bit references
def _bounds(k, n, s):
    """Largest and smallest key of each cluster of the first n rows: [..][C][d] in fp32 (exact)."""
    C = -(-n // s)
    x = k[..., :n, :].float()
    pad = C * s - n
    if pad:
        fill = x.new_full((*x.shape[:-2], pad, x.shape[-1]), math.nan)
        x = torch.cat([x, fill], -2)
    x = x.view(*x.shape[:-2], C, s, x.shape[-1])
    bad = x.isnan()
    return x.masked_fill(bad, -math.inf).amax(-2), x.masked_fill(bad, math.inf).amin(-2)


def _reps(c, k, n, slots):
    """Representatives of one layer's keys at both levels, [B][Hkv][slots][R][d] (zeros past the clusters)."""
    s, f = c["cluster"], c["fanout"]
    made = []
    for size, count in ((s, slots), (s * f, -(-slots // f))):
        if c["similarity"] == "mean":
            x, C = k[..., :n, :].double(), -(-n // size)
            x = torch.nn.functional.pad(x, (0, 0, 0, C * size - n)).view(*x.shape[:-2], C, size, x.shape[-1]).sum(-2)
            num = torch.full((C,), float(size), dtype=torch.float64, device="cuda")
            num[-1] = n - (C - 1) * size
            r = (x / num[:, None]).float()[..., None, :]
        else:
            hi, lo = _bounds(k, n, size)
            if c["similarity"] == "maxprod":
                r = torch.stack([hi, lo], -2)
            else:  # rounded like the stored representative: two 32-bit products and their 32-bit sum
                a = torch.tensor(ALPHA, dtype=torch.float32)
                b = (1.0 - a.double()).float()
                r = (a.cuda() * hi + b.cuda() * lo)[..., None, :]
        out = r.new_zeros(*r.shape[:-3], count, *r.shape[-2:])
        out[..., :r.shape[-3], :, :] = r
        made.append(out)
    return made


def _unit_scores(c, q, rep, n):
    """Similarity of every selection unit with the first n representatives in fp64: q [B][Hq][d], rep
    [B][Hkv][slots][R][d] -> [B][units][n]."""
    B, Hq, d = q.shape
    G = Hq // c["Hkv"]
    qd = q.double().view(B, c["Hkv"], G, d)
    r = rep[..., :n, :, :].double()
    if c["similarity"] == "maxprod":
        # max(q hi, q lo) = q+ hi + q- lo with q+ = max(q, 0), q- = min(q, 0), as hi >= lo
        x = qd.clamp(min=0) @ r[..., 0, :].transpose(-1, -2).contiguous()
        x = x + qd.clamp(max=0) @ r[..., 1, :].transpose(-1, -2).contiguous()
    else:
        x = qd @ r[..., 0, :].transpose(-1, -2).contiguous()
    if c["group"] == "head":
        return x.reshape(B, Hq, n)
    return x.amax(2) if c["group"] == "max" else x.sum(2)


def _select(c, q, cent, scent, Ts):
    """Two-level selection of one layer: ascending cluster ids [B][units][k] and their scores."""
    z, f = _sizes(c), c["fanout"]
    C = Ts // c["cluster"]
    S = -(-C // f)
    up = _unit_scores(c, q, scent, S).sort(stable=True, dim=-1, descending=True).indices[..., :z["k_super"]]
    fine = _unit_scores(c, q, cent, C)
    cand = torch.zeros(*fine.shape[:2], S, dtype=torch.bool, device="cuda").scatter_(-1, up, True)
    fine = fine.masked_fill(~cand.repeat_interleave(f, -1)[..., :C], -math.inf)
    best = fine.sort(stable=True, dim=-1, descending=True).indices[..., :z["k_clusters"]].sort(-1).values
    return best, fine.gather(-1, best)


def _attend(c, q, k, v, sel, Ts, n_tail):
    """Softmax attention of one layer over its selected clusters and the tail, in fp64."""
    B, Hq, d = q.shape
    s, per = c["cluster"], sel.shape[1]
    rows = (sel.long()[..., None] * s + torch.arange(s, device="cuda")).flatten(-2)
    rows = torch.cat([rows, torch.arange(Ts, Ts + n_tail, device="cuda").expand(B, per, n_tail)], -1)
    head = torch.arange(per, device="cuda") // (per // c["Hkv"])
    at = (torch.arange(B, device="cuda")[:, None, None], head[None, :, None], rows)
    kk, vv = k[at].double(), v[at].double()
    qd = q.double().view(B, per, Hq // per, d)
    x = qd @ kk.transpose(-1, -2).contiguous() / math.sqrt(d)
    lse = x.logsumexp(-1)
    return (torch.exp(x - lse[..., None]) @ vv).reshape(B, Hq, d), lse.reshape(B, Hq)


def _exact_decode(c, k, v, q, cents, sel_in, Ts, n_tail):
    sels, scores, outs, lses = [], [], [], []
    for l in range(c["L"]):
        o = _owner(c["layer0"] + l, c["period"]) - c["layer0"]
        if o == l:
            sel, sc = _select(c, q[l], *cents[l], Ts)
        elif o >= 0:
            sel, sc = sels[o], scores[o]
        else:
            sel, sc = sel_in[l], torch.zeros_like(sel_in[l], dtype=torch.float64)
        out, lse = _attend(c, q[l], k[l], v[l], sel, Ts, n_tail)
        sels.append(sel.to(torch.int32)), scores.append(sc), outs.append(out), lses.append(lse)
    return [torch.stack(x) for x in (sels, scores, outs, lses)]


def _exact_scores(c, q, k):
    """Accumulated window attention [Hkv][T] and row log-sum-exp [Hq][W] of one layer and sequence, in fp64."""
    Hq, W, d = q.shape
    Hkv, T, _ = k.shape
    total = torch.zeros(Hkv, T, dtype=torch.float64, device="cuda")
    lse = torch.empty(Hq, W, dtype=torch.float64, device="cuda")
    cols = torch.arange(T, device="cuda")
    step = max(1, int(2e8) // T)
    for h in range(Hkv):
        kt = k[h].double().t().contiguous()
        for g in range(h * (Hq // Hkv), (h + 1) * (Hq // Hkv)):
            for r in range(0, W, step):
                n = min(step, W - r)
                x = q[g, r:r + n].double() @ kt
                x /= math.sqrt(d)
                rows = torch.arange(r, r + n, device="cuda")
                first = T - W + r + 1  # columns below it are visible to every row of the chunk
                x[:, first:].masked_fill_(cols[None, first:] > (T - W + rows)[:, None], -math.inf)
                lse[g, r:r + n] = x.logsumexp(-1)
                total[h] += x.sub_(lse[g, r:r + n, None]).exp_().sum(0)
    return total, lse


def exact(c, seed):
    z = _sizes(c)
    L, B, Hkv = c["L"], c["B"], c["Hkv"]
    own = _owners(c)
    if c["kind"] == "prefill":
        q, k, v = _prompt(c, seed)
        f64 = dict(dtype=torch.float64, device="cuda")
        score, lse = torch.zeros(L, B, Hkv, c["T"], **f64), torch.zeros(L, B, c["Hq"], z["W"], **f64)
        kept = torch.zeros(L, B, Hkv, z["keep"], dtype=torch.int32, device="cuda")
        ks, vs, cents = [], [], []
        n_old = c["T"] - z["local"]
        slots = -(-z["keep"] // c["cluster"])
        for l in range(L):
            o = _owner(c["layer0"] + l, c["period"]) - c["layer0"]
            if o == l:
                for b in range(B):
                    score[l, b], lse[l, b] = _exact_scores(c, q[l, b], k[l, b])
                best = score[l, :, :, :n_old].sort(stable=True, dim=-1, descending=True).indices[..., :z["keep"] - z["local"]]
                last = torch.arange(n_old, c["T"], device="cuda").expand(B, Hkv, -1)
                kept[l] = torch.cat([best.sort(-1).values, last], -1).to(torch.int32)
            else:
                kept[l] = kept[o] if o >= 0 else _caller_sets(c, seed, c["T"], z["keep"])
            at = kept[l].long()[..., None].expand(-1, -1, -1, c["d"])
            ks.append(k[l].gather(2, at)), vs.append(v[l].gather(2, at))
            made = _reps(c, ks[l], z["keep"], slots) if l in own else None
            cents.append(made)
        ref = next(m for m in cents if m is not None) if own else None
        flat = lambda i: torch.stack([(m[i] if m else torch.zeros_like(ref[i])) for m in cents]) if own else None  # noqa: E731
        return {"kept": kept, "k": torch.stack(ks), "v": torch.stack(vs), "cent": flat(0), "scent": flat(1),
                "token_score": score, "row_lse": lse}
    rows = z["keep"] if c["kind"] == "decode" else _capacity(c)
    k, v, g = _cache(c, seed, rows)
    sel_in = [_caller_sets(c, seed, z["C"], z["k_clusters"])] * L if _owned_before(c) else None
    slots = -(-rows // c["cluster"])
    if c["kind"] == "decode":
        q = _randn(g, L, B, c["Hq"], c["d"], dtype=DTYPE[c["dtype"]])
        cents = [_reps(c, k[l], z["keep"], slots) if l in own else None for l in range(L)]
        sel, sc, out, lse = _exact_decode(c, k, v, q, cents, sel_in, z["keep"], 0)
        return {"sel": sel, "sel_score": sc, "out": out, "lse": lse}
    kn, vn, q = _new_tokens(c, g)
    sels, outs, lses = [], [], []
    for i in range(c["tokens"]):
        Ts, nt = _tail_state(c, i)
        k[:, :, :, Ts + nt - 1], v[:, :, :, Ts + nt - 1] = kn[i], vn[i]
        cents = [_reps(c, k[l], Ts, slots) if l in own else None for l in range(L)]
        sel, _, out, lse = _exact_decode(c, k, v, q[i], cents, sel_in, Ts, nt)
        sels.append(sel), outs.append(out), lses.append(lse)
    ref = next((m for m in cents if m is not None), None)
    flat = lambda i: torch.stack([(m[i] if m else torch.zeros_like(ref[i])) for m in cents]) if own else None  # noqa: E731
    return {"sel": torch.stack(sels), "out": torch.stack(outs), "lse": torch.stack(lses), "k": k, "v": v, "cent": flat(0),
            "scent": flat(1)}
