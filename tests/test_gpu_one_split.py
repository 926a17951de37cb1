"""Attention over short kept lists (at most 10 to 24 tiles of 32 tokens per
sequence, by the number of sequences and KV heads), which one workgroup per (sequence, KV head) takes whole and writes itself: from
no kept chunk to just past the limit, one to 16 query rows, ragged batches and
a partial last chunk, token by token against the oracle.
"""
from __future__ import annotations

import numpy as np
import pytest

import lsa_synth as synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk,counts", [(64, [8, 1, 5]), (64, [0, 8]), (64, [9, 2]), (128, [4, 3, 1]), (128, [5]),
                                          (64, [2] * 12), (64, [5]), (64, [6]), (64, [6] * 3), (64, [7] * 3),
                                          (64, [8] * 16), (64, [9] * 16)])
@pytest.mark.parametrize("hq,hkv,tq", [(8, 8, 1), (12, 4, 5), (8, 1, 2)])
def test_one_split(chunk, counts, hq, hkv, tq):
    import torch
    import oracle
    import parity
    import paper_2606_09079_amd as L
    rng = np.random.default_rng(sum(counts) * 100 + hq)
    B, G = len(counts), hq // hkv
    ctx = [chunk * int(rng.integers(10, 40)) + int(rng.integers(1, chunk)) for _ in counts]
    prob = synth.Problem("one_split", ctx, chunk, [1] * B, hq, hkv, n_qtok=tq)
    host = synth.host_inputs(prob, 41)
    dev = synth.device_inputs(prob, 41, host=host)
    keep = [max(c, 1) for c in counts]
    kept = []
    for c, n in zip(counts, prob.n_chunks):
        ids = np.sort(rng.choice(n - 1, size=max(c - 1, 0), replace=False))
        kept.append(np.concatenate([ids, [n - 1]]).astype(np.int32) if c else np.zeros(0, np.int32))
    P = L.Problem(ctx, chunk, keep, hq, hkv, n_qtok=tq)
    ws_bytes = L.lsa_workspace_size(L.Problem([chunk * n for n in prob.n_chunks], chunk, keep, hq, hkv, n_qtok=tq))
    ws = torch.zeros(ws_bytes, dtype=torch.uint8, device="cuda")
    sel_h = np.zeros((B, max(keep)), dtype=np.int32)
    for b, k in enumerate(kept):
        sel_h[b, :len(k)] = k
    sel, cnt = torch.from_numpy(sel_h).cuda(), torch.tensor(counts, dtype=torch.int32, device="cuda")
    out = torch.full((B, tq, hq, 128), float("nan"), device="cuda")
    lse = torch.full((B, tq, hq), float("nan"), device="cuda")
    L.lsa_sparse_decode_attn(P, dev["q"], dev["k"], dev["v"], sel, cnt, 0.0, out, lse, ws, ws_bytes)
    torch.cuda.synchronize()
    g_out, g_lse = out.cpu().numpy(), lse.cpu().numpy()
    for b in range(B):
        if counts[b] == 0:
            assert np.all(g_out[b] == 0) and np.all(np.isneginf(g_lse[b]))
            continue
        toks = oracle.kept_tokens(kept[b], chunk, ctx[b])
        for g in range(hkv):
            Kh = synth.kv_head_sparse(prob, 41, "k", b, g, kept[b])
            Vh = synth.kv_head_sparse(prob, 41, "v", b, g, kept[b])
            rows = [(t, g * G + j) for t in range(tq) for j in range(G)]
            qr = np.stack([host["q"][b, t, h] for (t, h) in rows])
            r_out, r_lse = oracle.attention_tokens(qr, Kh, Vh, toks)
            parity.check_attention(np.stack([g_out[b, t, h] for (t, h) in rows]), [g_lse[b, t, h] for (t, h) in rows],
                                   r_out, r_lse, f"C={chunk}, counts {counts}, sequence {b}, KV head {g}")
