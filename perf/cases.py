"""Performance cases: the calls that users of this library make, each a plain dict.

``listed()`` names the twelve measured cases, ``draw(rng)`` gives further ones of the same ranges, ``prepare`` makes the
device state a serving or labelling program holds before the call, ``run`` is one pass through the public entry points,
``exact`` the same outputs in float64 by plain torch, and ``work`` the bytes and operations a pass cannot do without.

Families:
  step      lsa_decode_step: score every chunk, keep the top k (union over the lookahead queries), attend
  recall    lsa_recall_step: gated multi-head indexer layers, threshold, K_max bound, attend
  twolevel  lsa_two_level_step: recall over the history, native top-k inside it, resident window, attend
  tier      lsa_tier_step: native top-k over the chunks resident in the GPU reserve, attend over their slots
  golden    lsa_golden_labels: top-p sets of raw logits, votes over layers, label union over a window
  pack      lsa_kv_pack: token-major K/V rows into the paged blocks (prefill)
"""
import math
import random
from statistics import NormalDist

import torch

import paper_2606_09079_amd as L

HEAD_DIM = 128
RHO = 0.95  # correlation of the lookahead query embeddings of one sequence

_STEP = dict(family="step", chunk=64, lookahead=1, qtok=1, emb="bf16", dim=256, q_heads=32, kv_heads=8, keep_frac=0.0,
             keep_max=0, planted=16, lengths=0)


def _step(name, **kw):
    c = dict(_STEP, **kw)
    c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a 4K-token context of one request, float32 indexer, where only latency counts
        _step("step_tiny_f32", batch=1, ctx_lo=4096, ctx_hi=4096, keep_max=8, q_heads=8, emb="f32", planted=3),
        # a small batch of 128K-token requests with a quantised indexer
        _step("step_int8_4x128k", batch=4, ctx_lo=131072, ctx_hi=131072, keep_max=256, emb="i8"),
        # the paper's serving point: one request of 1M tokens, 10% of its chunks kept
        _step("step_1m", batch=1, ctx_lo=1048576, ctx_hi=1048576, keep_max=1638, planted=64),
        # a continuous batch of 32 requests of 32K to 512K tokens at the paper's mean keep ratio
        _step("step_batch32", batch=32, ctx_lo=32768, ctx_hi=524288, keep_frac=0.135, lengths=1),
        # eight 1M-token requests with 16 lookahead queries and 16 query tokens: 128 query rows per KV head (the largest)
        _step("step_lookahead", batch=8, ctx_lo=1048576, ctx_hi=1048576, keep_max=512, chunk=128, lookahead=16,
              qtok=16, q_heads=64),
        # multi-token prediction: four draft tokens verified at once, 32 query rows per KV head, ragged contexts
        _step("step_draft4", batch=6, ctx_lo=16384, ctx_hi=262144, keep_frac=0.1, lookahead=4, qtok=4, q_heads=64,
              lengths=2),
        # a context past 1M tokens under the same recall bound: 40,003 chunks
        _step("step_2m5", batch=1, ctx_lo=2560192, ctx_hi=2560192, keep_max=1638, planted=64),
        # the full Memory Indexer at 1M tokens: three layers of 64 heads, the recall exceeds its bound
        dict(name="recall_1m", family="recall", batch=1, ctx_lo=1048576, ctx_hi=1048576, chunk=64, layers=3, heads=64,
             width=128, rate=0.05, keep_max=1638, keep_frac=0.0, q_heads=32, kv_heads=8, qtok=1, lengths=0),
        # two-level selection with the resident window, a context that ends inside a chunk
        dict(name="twolevel_1m", family="twolevel", batch=1, ctx_lo=1048613, ctx_hi=1048613, chunk=64, layers=3,
             heads=64, width=128, rate=0.05, keep_max=2048, core=1024, window=8192, q_heads=32, kv_heads=8, qtok=1,
             lengths=0),
        # one decode step between firings of the host tier: Level 2 over 1,638 resident chunks of a 1M-token context
        dict(name="tier_1m", family="tier", batch=1, ctx_lo=1048576, ctx_hi=1048576, chunk=64, heads=64, width=128,
             keep_max=1638, core=1024, q_heads=32, kv_heads=8, qtok=1, lengths=0),
        # the labels of one 64-step window of a 512K-token document, 21 layers voting
        dict(name="golden_512k", family="golden", batch=1, n_lo=131072, n_hi=131072, steps=64, layers=21, lengths=0),
        # the prefill hand-over of four ragged requests into the paged cache
        dict(name="pack_prefill", family="pack", batch=4, ctx_lo=60000, ctx_hi=500000, chunk=64, kv_heads=8,
             lengths=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["step", "step", "step", "step", "recall", "twolevel", "tier", "golden", "golden", "pack"])
    lengths = rng.randrange(1, 1 << 20)
    if family == "golden":
        batch = _log(rng, 1, 12)
        hi = _log(rng, 4096, 131072 // max(1, batch // 3))
        return dict(family=family, batch=batch, n_lo=max(1000, hi // _log(rng, 1, 16)), n_hi=hi,
                    steps=rng.choice([16, 33, 64]) if batch <= 3 else 16, layers=rng.choice([12, 21]), lengths=lengths)
    kv_heads = rng.choice([2, 4, 8, 8, 8])
    chunk = rng.choice([64, 64, 128])
    if family == "pack":
        batch = _log(rng, 1, 16)
        hi = _log(rng, 2000, 600000 // batch)
        return dict(family=family, batch=batch, ctx_lo=max(500, hi // _log(rng, 1, 16)), ctx_hi=hi, chunk=chunk,
                    kv_heads=kv_heads, lengths=lengths)
    group = rng.choice([1, 2, 4, 4, 8])
    qtok = rng.choice([1, 1, 1, 2, 3, 4, 8])
    c = dict(family=family, chunk=chunk, qtok=qtok, q_heads=group * kv_heads, kv_heads=kv_heads, lengths=lengths)
    if family == "step":
        batch = _log(rng, 1, 48)
        hi = _log(rng, 4096, min(3000000, 5000000 // batch))
        lo = max(2048, min(hi, hi // _log(rng, 1, 16)))
        lookahead = rng.choice([1, 1, 1, 2, 4, 8, 16])
        # several lookahead queries keep a union of sets, about twice as many chunks
        c.update(batch=batch, ctx_lo=lo, ctx_hi=hi, lookahead=lookahead, emb=rng.choice(["bf16", "bf16", "f32", "i8"]),
                 dim=rng.choice([64, 128, 256, 256, 512]), keep_frac=round(math.exp(rng.uniform(math.log(0.03), math.log(
                     0.16 if lookahead == 1 else 0.08))), 4), keep_max=0, planted=rng.randrange(0, 9))
        return c
    width, heads = rng.choice([64, 128]), rng.choice([16, 32, 64])
    batch = _log(rng, 1, 8)
    hi = _log(rng, 8192, min(1500000, 4000000 // batch))
    c.update(batch=batch, ctx_lo=max(8192, hi // _log(rng, 1, 8)), ctx_hi=hi, width=width, heads=heads)
    n_lo = c["ctx_lo"] // chunk
    if family == "recall":
        c.update(layers=rng.choice([1, 2, 3, 3, 4]), rate=round(rng.uniform(0.02, 0.12), 3), keep_max=0,
                 keep_frac=round(rng.uniform(0.05, 0.15), 3))
    elif family == "twolevel":
        k = max(8, int(n_lo * rng.uniform(0.08, 0.2)))
        c.update(layers=rng.choice([1, 2, 3, 3]), rate=round(rng.uniform(0.03, 0.12), 3), keep_max=k,
                 core=max(4, int(k * rng.uniform(0.3, 0.9))), window=rng.choice([512, 2048, 8192]))
    else:
        k = max(8, int(n_lo * rng.uniform(0.05, 0.15)))
        c.update(keep_max=k, core=max(4, int(k * rng.uniform(0.3, 0.9))))
    return c


# ---- shapes: from the case alone


def _ragged(case, lo, hi, unit):
    """Per-sequence lengths, log-uniform between lo and hi, whole multiples of unit."""
    r = random.Random(case["lengths"])
    if lo >= hi:
        return [max(unit, hi // unit * unit)] * case["batch"]
    return [max(unit, int(math.exp(r.uniform(math.log(lo), math.log(hi)))) // unit * unit) for _ in range(case["batch"])]


def _ctx(case):
    # the two-level path and the re-layout take contexts that end inside a chunk
    unit = 1 if case["family"] in ("twolevel", "pack") else case["chunk"]
    return _ragged(case, case["ctx_lo"], case["ctx_hi"], unit)


def _chunks(case):
    return [-(-c // case["chunk"]) for c in _ctx(case)]


def _keep(case):
    if case["family"] == "pack":
        return [1] * case["batch"]
    ns = _chunks(case)
    if case.get("keep_frac"):
        return [max(1, int(case["keep_frac"] * n)) for n in ns]
    return [min(case["keep_max"], n) for n in ns]


def _history(case):
    """First window chunk of each sequence (two-level path)."""
    C = case["chunk"]
    return [min(max(c - case["window"], 0) // C, c // C) for c in _ctx(case)]


def _union_share(k, n, q):
    """Expected share of n chunks in the union of the top k of q queries with correlation RHO."""
    if q == 1 or k >= n:
        return k / n
    nd = NormalDist()
    t = nd.inv_cdf(1.0 - k / n)
    out, step = 0.0, 0.02
    for i in range(-300, 301):
        a = i * step
        out += nd.pdf(a) * step * nd.cdf((t - math.sqrt(RHO) * a) / math.sqrt(1.0 - RHO)) ** q
    return min(1.0, 1.0 - out)


def work(case):
    fam = case["family"]
    if fam == "golden":
        n = sum(_ragged(case, case["n_lo"], case["n_hi"], 1))
        rows = case["steps"] * case["layers"]
        # every logit once and the label list; a weight is an exponential of about ten operations
        return {"bytes": 4.0 * rows * n + 8.0 * rows * case["batch"], "flops": 10.0 * rows * n}
    if fam == "pack":
        tokens, blocks = sum(_ctx(case)), sum(_chunks(case)) * case["chunk"]
        return {"bytes": 2.0 * 2 * case["kv_heads"] * HEAD_DIM * (tokens + blocks), "flops": 0.0}
    C, ns, keep = case["chunk"], _chunks(case), _keep(case)
    if fam == "step":
        es = {"f32": 4, "bf16": 2, "i8": 1}[case["emb"]]
        q = case["lookahead"]
        kept = sum(n * _union_share(k, n, q) for n, k in zip(ns, keep))
        idx_bytes = sum(ns) * case["dim"] * es
        idx_flops = 2.0 * sum(ns) * case["dim"] * q
    elif fam == "recall":
        # the union over layers of independent recalls, bounded by K_max
        u = 1.0 - (1.0 - case["rate"]) ** case["layers"]
        kept = sum(min(k, u * n) for n, k in zip(ns, keep))
        idx_bytes = sum(ns) * case["layers"] * case["width"] * 2
        idx_flops = 2.0 * sum(ns) * case["layers"] * case["heads"] * case["width"]
    elif fam == "twolevel":
        hist = _history(case)
        u = 1.0 - (1.0 - case["rate"]) ** case["layers"]
        rec = [min(k, u * h) for h, k in zip(hist, keep)]
        kept = sum(min(case["core"], r) + n - h for n, h, r in zip(ns, hist, rec))
        idx_bytes = (sum(hist) * case["layers"] + sum(rec)) * case["width"] * 2
        idx_flops = 2.0 * (sum(hist) * case["layers"] + sum(rec)) * case["heads"] * case["width"]
    else:  # tier
        kept = sum(min(case["core"], k) for k in keep)
        idx_bytes = sum(keep) * (case["width"] * 2 + 8)
        idx_flops = 2.0 * sum(keep) * case["heads"] * case["width"]
    rows = case["batch"] * case["qtok"] * case["q_heads"]
    kv = kept * C * case["kv_heads"] * HEAD_DIM * 2 * 2
    attn = 4.0 * kept * C * case["qtok"] * case["q_heads"] * HEAD_DIM
    return {"bytes": idx_bytes + kv + rows * (HEAD_DIM * 6 + 4) + 4.0 * kept, "flops": idx_flops + attn}


def tolerance(case):
    # labels, sizes and re-laid bytes are whole numbers.  Attention: bf16 inputs, float32 softmax and sums, weights in
    # two bf16 parts (16 bits); the kept ids come from float32 scores and the same on both sides
    if case["family"] in ("golden", "pack"):
        return "exact"
    return {"rel": 2e-5, "max": 2e-4}


# ---- device state


def _gen(seed, *more):
    g = torch.Generator(device="cuda")
    s = 0x9E3779B97F4A7C15 * (int(seed) + 1)
    for m in more:
        s = s * 6364136223846793005 + m + 1442695040888963407
    g.manual_seed(s & 0x7FFFFFFFFFFFFFFF)
    return g


def _randn(shape, g, dtype=torch.float32):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype)


def _unit(x):
    return x / x.norm(dim=-1, keepdim=True)


def _attention_buffers(case, state, seed, n_blocks, max_sel, ws_bytes):
    """K/V blocks (any order of N(0, 1) values is the same distribution, so the blocks are filled in place), q, outputs."""
    B, C, H = case["batch"], case["chunk"], case["kv_heads"]
    state["k"] = _randn((n_blocks, H, C * HEAD_DIM), _gen(seed, 1), torch.bfloat16)
    state["v"] = _randn((n_blocks, H, C * HEAD_DIM), _gen(seed, 2), torch.bfloat16)
    state["q"] = _randn((B, case["qtok"], case["q_heads"], HEAD_DIM), _gen(seed, 3), torch.bfloat16)
    state["out"] = torch.zeros(B, case["qtok"], case["q_heads"], HEAD_DIM, device="cuda")
    state["lse"] = torch.zeros(B, case["qtok"], case["q_heads"], device="cuda")
    state["sel"] = torch.zeros(B, max_sel, dtype=torch.int32, device="cuda")
    state["cnt"] = torch.zeros(B, dtype=torch.int32, device="cuda")
    state["ws"] = torch.zeros(ws_bytes, dtype=torch.uint8, device="cuda")
    state["ws_bytes"] = ws_bytes


def _problem(case, **kw):
    return L.Problem(_ctx(case), case["chunk"], _keep(case), case["q_heads"], case["kv_heads"], HEAD_DIM,
                     n_qtok=case["qtok"], **kw)


def _gates(q, keys, rates, g, clear=0):
    """Gates w_h = g_h - beta of mixed sign, beta such that a share `rate` of the entries scores at least 0.

    q [nh, c], keys [n, c]; beta lies between two entries' critical values, so no score sits on the threshold.
    """
    w0 = _randn((q.shape[0],), g)
    r = torch.relu(q.float() @ keys.float().t())
    ratio, _ = torch.sort((w0 @ r) / r.sum(0).clamp_min(1e-20), descending=True)
    n = ratio.numel()
    i = min(max(int(rates * n), 1), n - 1) if n > 1 else 0
    beta = (ratio[i - 1] + ratio[i]) / 2 if n > 1 else ratio[0] - 0.1
    return w0 - beta


def _indexer_inputs(case, seed, layers, rate, salt):
    """Queries, unit keys and gates of `layers` indexer layers: the shapes of lsa_recall_scores."""
    ns, B, H, W = _chunks(case), case["batch"], case["heads"], case["width"]
    total = sum(ns)
    q = _randn((B, layers, H, W), _gen(seed, salt, 1), torch.bfloat16)
    k = _unit(_randn((layers, total, W), _gen(seed, salt, 2))).to(torch.bfloat16)
    g = _gen(seed, salt, 3)
    w = torch.empty(B, layers, H, device="cuda")
    off = 0
    for b, n in enumerate(ns):
        for l in range(layers):
            w[b, l] = _gates(q[b, l], k[l, off:off + n], rate, g)
        off += n
    return q, w, k


def _prepare_step(case, seed):
    ns, B, D, Q = _chunks(case), case["batch"], case["dim"], case["lookahead"]
    total = sum(ns)
    P = _problem(case, emb_dim=D, n_lookahead=Q, emb_dtype=case["emb"])
    s = {"p": P, "case": case}
    g = _gen(seed, 10)
    r = random.Random(int(seed) * 7919 + 5)
    off, planted = 0, []
    for n in ns:
        m = min(case["planted"], n)
        planted.append([off + (2 * i + 1) * n // (2 * m) for i in range(m)])
        off += n
    if case["emb"] == "i8":
        qe = torch.randint(-127, 128, (B, Q, D), generator=g, device="cuda", dtype=torch.int8)
        E = torch.randint(-127, 128, (total, D), generator=g, device="cuda", dtype=torch.int8)
        for b in range(B):  # query-critical chunks, aligned with the query
            if planted[b]:
                E[planted[b]] = torch.where(qe[b, r.randrange(Q)] < 0, -127, 127).to(torch.int8)
    else:
        base, own = _randn((B, 1, D), g), _randn((B, Q, D), g)
        qf = _unit(math.sqrt(RHO) * base + math.sqrt(1.0 - RHO) * own)
        Ef = _unit(_randn((total, D), g))
        for b in range(B):
            if planted[b]:
                Ef[planted[b]] = _unit(Ef[planted[b]] + 0.5 * qf[b, r.randrange(Q)])
        dt = torch.float32 if case["emb"] == "f32" else torch.bfloat16
        qe, E = qf.to(dt), Ef.to(dt)
    s["qe"], s["E"] = qe, E
    _attention_buffers(case, s, seed, total, L.lsa_max_sel(P), L.lsa_workspace_size(P))
    return s


def _prepare_recall(case, seed):
    P = _problem(case)
    s = {"p": P, "case": case, "ix": L.Indexer(case["layers"], case["heads"], case["width"])}
    s["iq"], s["iw"], s["ik"] = _indexer_inputs(case, seed, case["layers"], case["rate"], 20)
    _attention_buffers(case, s, seed, sum(_chunks(case)), L.lsa_max_sel(P), L.lsa_workspace_size(P))
    return s


def _prepare_twolevel(case, seed):
    P, B = _problem(case), case["batch"]
    tl = L.TwoLevel(case["heads"], [case["core"]] * B, [case["window"]] * B)
    s = {"p": P, "case": case, "tl": tl, "ix": L.Indexer(case["layers"], case["heads"], case["width"])}
    s["iq"], s["iw"], s["ik"] = _indexer_inputs(case, seed, case["layers"], case["rate"], 20)
    nq, nw, nk = _indexer_inputs(case, seed, 1, 0.5, 30)
    s["nq"], s["nw"], s["nk"] = nq[:, 0].contiguous(), nw[:, 0].contiguous(), nk[0].contiguous()
    max_sel, ws_bytes = L.lsa_two_level_sizes(P, tl)
    _attention_buffers(case, s, seed, sum(_chunks(case)), max_sel, ws_bytes)
    return s


def _prepare_tier(case, seed):
    P, B, ns, keep = _problem(case), case["batch"], _chunks(case), _keep(case)
    slots = [2 * k for k in keep]
    tr = L.Tier(slots)
    s = {"p": P, "case": case, "tr": tr, "ix": L.Indexer(1, case["heads"], case["width"])}
    nq, nw, nk = _indexer_inputs(case, seed, 1, 0.5, 30)
    s["nq"], s["nw"], s["nk"] = nq[:, 0].contiguous(), nw[:, 0].contiguous(), nk[0].contiguous()
    pitch, total_slots, ws_bytes = L.lsa_tier_sizes(P, tr)
    _attention_buffers(case, s, seed, total_slots, pitch, ws_bytes)
    # what the last firing left: the kept list and, after some firings, slots in no particular order
    g = _gen(seed, 40)
    s["kept"] = torch.zeros(B, pitch, dtype=torch.int32, device="cuda")
    s["slot"] = torch.zeros(B, pitch, dtype=torch.int32, device="cuda")
    for b in range(B):
        ids = torch.randperm(ns[b], generator=g, device="cuda")[:keep[b]]
        s["kept"][b, :keep[b]] = torch.sort(ids)[0].to(torch.int32)
        s["slot"][b, :keep[b]] = torch.randperm(slots[b], generator=g, device="cuda")[:keep[b]].to(torch.int32)
    s["kept_cnt"] = torch.tensor(keep, dtype=torch.int32, device="cuda")
    s["core"] = [case["core"]] * B
    return s


def _prepare_golden(case, seed):
    ns, T, NL = _ragged(case, case["n_lo"], case["n_hi"], 1), case["steps"], case["layers"]
    gl = L.Golden(ns, T, NL)
    g = _gen(seed, 50)
    logits = torch.empty(T * NL * sum(ns), device="cuda")
    off = 0
    for n in ns:
        # unit normal logits; one entry in 256 is relevant and stands 8.5 above in half of the rows
        x = logits[off:off + T * NL * n].view(T * NL, n)
        x.normal_(generator=g)
        rel = torch.randperm(n, generator=g, device="cuda")[:max(1, n // 256)]
        x[:, rel] += 8.5 * (torch.rand((T * NL, rel.numel()), generator=g, device="cuda") < 0.5)
        off += T * NL * n
    ws_bytes = L.lsa_golden_sizes(gl)
    return {"case": case, "gl": gl, "logits": logits, "ws_bytes": ws_bytes,
            "labels": torch.zeros(sum(ns), dtype=torch.int32, device="cuda"),
            "count": torch.zeros(case["batch"], dtype=torch.int32, device="cuda"),
            "nucleus": torch.zeros(case["batch"], T, NL, dtype=torch.int32, device="cuda"),
            "golden": torch.zeros(case["batch"], T, dtype=torch.int32, device="cuda"),
            "ws": torch.zeros(ws_bytes, dtype=torch.uint8, device="cuda")}


def _prepare_pack(case, seed):
    ctx, H, C = _ctx(case), case["kv_heads"], case["chunk"]
    P = L.Problem(ctx, C, _keep(case), H, H, HEAD_DIM)
    s = {"p": P, "case": case}
    s["kt"] = _randn((sum(ctx), H, HEAD_DIM), _gen(seed, 1), torch.bfloat16)
    s["vt"] = _randn((sum(ctx), H, HEAD_DIM), _gen(seed, 2), torch.bfloat16)
    offs = [0]
    for c in ctx:
        offs.append(offs[-1] + c)
    s["offs"] = torch.tensor(offs, dtype=torch.int64, device="cuda")
    total = sum(_chunks(case))
    s["k"] = torch.zeros(total, H, C * HEAD_DIM, dtype=torch.bfloat16, device="cuda")
    s["v"] = torch.zeros(total, H, C * HEAD_DIM, dtype=torch.bfloat16, device="cuda")
    return s


_PREPARE = {"step": _prepare_step, "recall": _prepare_recall, "twolevel": _prepare_twolevel, "tier": _prepare_tier,
            "golden": _prepare_golden, "pack": _prepare_pack}


def prepare(case, seed):
    return _PREPARE[case["family"]](case, seed)


def run(s):
    fam = s["case"]["family"]
    if fam == "step":
        L.lsa_decode_step(s["p"], s["qe"], s["E"], s["q"], s["k"], s["v"], 0.0, s["out"], s["lse"], s["sel"], s["cnt"],
                          s["ws"], s["ws_bytes"])
    elif fam == "recall":
        L.lsa_recall_step(s["p"], s["ix"], s["iq"], s["iw"], s["ik"], s["q"], s["k"], s["v"], 0.0, s["out"], s["lse"],
                          s["sel"], s["cnt"], s["ws"], s["ws_bytes"])
    elif fam == "twolevel":
        L.lsa_two_level_step(s["p"], s["ix"], s["tl"], s["iq"], s["iw"], s["ik"], s["nq"], s["nw"], s["nk"], s["q"],
                             s["k"], s["v"], 0.0, s["out"], s["lse"], s["sel"], s["cnt"], s["ws"], s["ws_bytes"])
    elif fam == "tier":
        L.lsa_tier_step(s["p"], s["tr"], s["ix"], s["core"], s["nq"], s["nw"], s["nk"], s["kept"], s["kept_cnt"],
                        s["slot"], s["q"], s["k"], s["v"], 0.0, s["out"], s["lse"], s["sel"], s["cnt"], s["ws"],
                        s["ws_bytes"])
    elif fam == "golden":
        L.lsa_golden_labels(s["gl"], s["logits"], s["labels"], s["count"], s["nucleus"], s["golden"], s["ws"],
                            s["ws_bytes"])
        return s["labels"], s["count"], s["nucleus"], s["golden"]
    else:
        L.lsa_kv_pack(s["p"], s["kt"], s["vt"], s["offs"], s["k"], s["v"])
        return s["k"].view(torch.int16), s["v"].view(torch.int16)
    return s["out"], s["lse"], s["sel"], s["cnt"]


# ---- the same outputs in float64, by the definitions


def _token_order(C):
    """Element of a K and of a V block that holds (token, dimension)."""
    t, e = torch.arange(C, device="cuda")[:, None], torch.arange(HEAD_DIM, device="cuda")[None, :]
    k = ((((t // 32 * 2 + t // 4 % 2) * 4 + e // 32) * 4 + e // 8 % 4) * 16 + t % 32 // 8 * 4 + t % 4) * 8 + e % 8
    v = (((t // 32 * 8 + e // 16) * 4 + t % 32 // 8) * 16 + e % 16) * 8 + t % 8
    return k, v


def _top(scores, k):
    """Ascending ids of the k largest, the lower id first among equals."""
    order = torch.sort(scores, descending=True, stable=True)[1]
    return torch.sort(order[:k])[0]


def _index_scores(q, w, keys):
    return w.double() @ torch.relu(q.double() @ keys.double().t())


def _recalled(x, k):
    """Ids whose largest layer score reaches 0, the k largest of them at most."""
    r = x.max(0)[0]
    return _top(r, min(k, int((r >= 0).sum())))


def exact(case, seed):
    fam = case["family"]
    if fam in ("golden", "pack"):
        return None  # whole numbers and bytes
    s = prepare(case, seed)
    ns, keep, ctx, C, G = _chunks(case), _keep(case), _ctx(case), case["chunk"], case["q_heads"] // case["kv_heads"]
    ko, vo = _token_order(C)
    out, lse = torch.zeros_like(s["out"], dtype=torch.float64), torch.zeros_like(s["lse"], dtype=torch.float64)
    off = slot_off = 0
    for b, n in enumerate(ns):
        if fam == "step":
            x = s["qe"][b].double() @ s["E"][off:off + n].double().t()
            ids = torch.unique(torch.cat([_top(x[j], keep[b]) for j in range(x.shape[0])]))
        elif fam == "recall":
            x = torch.stack([_index_scores(s["iq"][b, l], s["iw"][b, l], s["ik"][l, off:off + n])
                             for l in range(case["layers"])])
            ids = _recalled(x, keep[b])
        elif fam == "twolevel":
            h = _history(case)[b]
            x = torch.stack([_index_scores(s["iq"][b, l], s["iw"][b, l], s["ik"][l, off:off + h])
                             for l in range(case["layers"])])
            rec = _recalled(x, keep[b])
            nat = _index_scores(s["nq"][b], s["nw"][b], s["nk"][off:off + h])[rec]
            ids = torch.cat([rec[_top(nat, case["core"])], torch.arange(h, n, device="cuda")])
        else:
            kept = s["kept"][b, :keep[b]].long()
            nat = _index_scores(s["nq"][b], s["nw"][b], s["nk"][off:off + n])[kept]
            ids = s["slot"][b, :keep[b]].long()[_top(nat, case["core"])]
        block0 = slot_off if fam == "tier" else off
        tokens = ids.numel() * C
        if fam == "twolevel" and int(ids[-1]) == n - 1:
            tokens -= n * C - ctx[b]
        for g in range(case["kv_heads"]):
            K = s["k"][block0 + ids, g][:, ko].reshape(-1, HEAD_DIM)[:tokens].double()
            V = s["v"][block0 + ids, g][:, vo].reshape(-1, HEAD_DIM)[:tokens].double()
            q = s["q"][b, :, g * G:(g + 1) * G].reshape(-1, HEAD_DIM).double()
            x = q @ K.t() / math.sqrt(HEAD_DIM)
            lse[b, :, g * G:(g + 1) * G] = torch.logsumexp(x, -1).view(case["qtok"], G)
            out[b, :, g * G:(g + 1) * G] = (torch.softmax(x, -1) @ V).view(case["qtok"], G, HEAD_DIM)
        off += n
        slot_off += 2 * keep[b]
    return out, lse, None, None
