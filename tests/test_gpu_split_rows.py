"""The split attention kernel with one and two blocks of 16 query rows per KV
head, at the edges of the blocks and of its dispatch (15 to 33 rows), on a
context that ends inside its last chunk: a long kept list, one that ends with
the partial chunk, and the partial chunk alone, token by token against the
oracle at the attention tolerance of the other tests.
"""
from __future__ import annotations

import numpy as np
import pytest

import lsa_synth as synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", [64, 128])
@pytest.mark.parametrize("hq,hkv,tq", [(15, 1, 1), (16, 2, 2), (17, 1, 1), (12, 2, 4), (31, 1, 1), (16, 2, 4), (11, 1, 3)])
def test_split_rows(chunk, hq, hkv, tq):
    import torch
    import oracle
    import parity
    import paper_2606_09079_amd as L
    tail = 1 + (hq * 7 + chunk) % (chunk - 1)
    prob = synth.Problem("split_rows", [chunk * 90 + tail], chunk, [8], hq, hkv, n_qtok=tq)
    host = synth.host_inputs(prob, 31)
    dev = synth.device_inputs(prob, 31, host=host)
    n, G = prob.n_chunks[0], hq // hkv
    for kept in (np.arange(n - 1, dtype=np.int32), np.array([0, 7, 40, n - 2, n - 1], dtype=np.int32),
                 np.array([n - 1], dtype=np.int32)):
        P = L.Problem(prob.ctx_tokens, chunk, [len(kept)], hq, hkv, n_qtok=tq)
        ws_bytes = L.lsa_workspace_size(L.Problem([chunk * n], chunk, [len(kept)], hq, hkv, n_qtok=tq))
        ws = torch.zeros(ws_bytes, dtype=torch.uint8, device="cuda")
        sel = torch.from_numpy(kept[None, :].copy()).cuda()
        cnt = torch.tensor([len(kept)], dtype=torch.int32, device="cuda")
        out = torch.full((1, tq, hq, 128), float("nan"), device="cuda")
        lse = torch.full((1, tq, hq), float("nan"), device="cuda")
        L.lsa_sparse_decode_attn(P, dev["q"], dev["k"], dev["v"], sel, cnt, 0.0, out, lse, ws, ws_bytes)
        torch.cuda.synchronize()
        g_out, g_lse = out.cpu().numpy(), lse.cpu().numpy()
        toks = oracle.kept_tokens(kept, chunk, prob.ctx_tokens[0])
        for g in range(hkv):
            Kh = synth.kv_head_sparse(prob, 31, "k", 0, g, kept)
            Vh = synth.kv_head_sparse(prob, 31, "v", 0, g, kept)
            rows = [(t, g * G + j) for t in range(tq) for j in range(G)]
            qr = np.stack([host["q"][0, t, h] for (t, h) in rows])
            r_out, r_lse = oracle.attention_tokens(qr, Kh, Vh, toks)
            parity.check_attention(np.stack([g_out[0, t, h] for (t, h) in rows]), [g_lse[0, t, h] for (t, h) in rows],
                                   r_out, r_lse, f"{G * tq} rows, C={chunk}, {len(kept)} kept, KV head {g}")
