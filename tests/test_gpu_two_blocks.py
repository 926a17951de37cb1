"""17 to 32 query rows per KV head with kept lists just below and above the work
from which the split kernel takes them as two blocks of rows (the many-rows
kernel serves them below), and on each side a list that holds everything, one
that ends with the partial last chunk and that chunk alone, against the oracle.
"""
from __future__ import annotations

import numpy as np
import pytest

import lsa_synth as synth

pytestmark = pytest.mark.gpu

HKV = 16
LIMIT = 32 * 512 // HKV  # tiles per KV head


@pytest.mark.parametrize("chunk", [64, 128])
@pytest.mark.parametrize("hq,tq", [(17 * HKV, 1), (8 * HKV, 3), (8 * HKV, 4), (9 * HKV, 2)])
def test_two_blocks(chunk, hq, tq):
    import torch
    import oracle
    import parity
    import paper_2606_09079_amd as L
    n = LIMIT // (chunk // 32) + 1
    tail = 1 + (hq * 7 + chunk) % (chunk - 1)
    prob = synth.Problem("two_blocks", [chunk * (n - 1) + tail], chunk, [8], hq, HKV, n_qtok=tq)
    host = synth.host_inputs(prob, 37)
    dev = synth.device_inputs(prob, 37, host=host)
    G = hq // HKV
    lists = (np.arange(n, dtype=np.int32), np.array([0, 7, 40, n - 2, n - 1], dtype=np.int32),
             np.array([n - 1], dtype=np.int32))
    for keep in (n - 2, n):  # one chunk below the limit, and at it
        P = L.Problem(prob.ctx_tokens, chunk, [keep], hq, HKV, n_qtok=tq)
        ws_bytes = L.lsa_workspace_size(L.Problem([chunk * n], chunk, [keep], hq, HKV, n_qtok=tq))
        for kept in lists:
            kept = kept[max(0, len(kept) - keep):]
            ws = torch.zeros(ws_bytes, dtype=torch.uint8, device="cuda")
            sel = torch.zeros(1, keep, dtype=torch.int32, device="cuda")
            sel[0, :len(kept)] = torch.from_numpy(kept.copy()).cuda()
            cnt = torch.tensor([len(kept)], dtype=torch.int32, device="cuda")
            out = torch.full((1, tq, hq, 128), float("nan"), device="cuda")
            lse = torch.full((1, tq, hq), float("nan"), device="cuda")
            L.lsa_sparse_decode_attn(P, dev["q"], dev["k"], dev["v"], sel, cnt, 0.0, out, lse, ws, ws_bytes)
            torch.cuda.synchronize()
            g_out, g_lse = out.cpu().numpy(), lse.cpu().numpy()
            toks = oracle.kept_tokens(kept, chunk, prob.ctx_tokens[0])
            for g in (0, HKV - 1):
                Kh = synth.kv_head_sparse(prob, 37, "k", 0, g, kept)
                Vh = synth.kv_head_sparse(prob, 37, "v", 0, g, kept)
                rows = [(t, g * G + j) for t in range(tq) for j in range(G)]
                qr = np.stack([host["q"][0, t, h] for (t, h) in rows])
                r_out, r_lse = oracle.attention_tokens(qr, Kh, Vh, toks)
                parity.check_attention(np.stack([g_out[0, t, h] for (t, h) in rows]),
                                       [g_lse[0, t, h] for (t, h) in rows], r_out, r_lse,
                                       f"{G * tq} rows, C={chunk}, keep {keep}, {len(kept)} kept, KV head {g}")
