"""The fused step's one-launch scoring and selection of short sequences against
the separate calls (lsa_score_chunks, then lsa_topk_chunks): identical kept ids
for every embedding type and width, sequence lengths around the wavefront's 64
entries and the rule's limits, any keep budget, repeated and zero embedding
rows (ties, both zeros) and ragged batches.
"""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _step_and_parts(ns, ks, dtype, D, seed, kind):
    import torch
    import paper_2606_09079_amd as L
    g = torch.Generator().manual_seed(seed)
    B, total, H = len(ns), sum(ns), 1
    if dtype == "i8":
        E = torch.randint(-127, 128, (total, D), generator=g, dtype=torch.int8)
        qe = torch.randint(-127, 128, (B, 1, D), generator=g, dtype=torch.int8)
    else:
        dt = torch.float32 if dtype == "f32" else torch.bfloat16
        E, qe = torch.randn(total, D, generator=g).to(dt), torch.randn(B, 1, D, generator=g).to(dt)
    if kind == "ties":
        E[::3] = E[0].clone()
        E[1::5] = 0
    E, qe = E.cuda(), qe.cuda()
    P = L.Problem([64 * n for n in ns], 64, ks, H, H, emb_dim=D, emb_dtype=dtype)
    k = torch.randn(total, H, 64 * 128, device="cuda").to(torch.bfloat16)
    q = torch.randn(B, 1, H, 128, device="cuda").to(torch.bfloat16)
    out = torch.zeros(B, 1, H, 128, device="cuda")
    wsb = L.lsa_workspace_size(P)
    ws = torch.full((wsb,), 0xA5, dtype=torch.uint8, device="cuda")
    sel = torch.full((B, L.lsa_max_sel(P)), -1, dtype=torch.int32, device="cuda")
    cnt = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    L.lsa_decode_step(P, qe, E, q, k, k, 0.0, out, None, sel, cnt, ws, wsb)
    scores = torch.zeros(total, dtype=torch.int32 if dtype == "i8" else torch.float32, device="cuda")
    sel2, cnt2 = torch.full_like(sel, -1), torch.full_like(cnt, -1)
    L.lsa_score_chunks(P, qe, E, scores)
    L.lsa_topk_chunks(P, scores, sel2, cnt2)
    torch.cuda.synchronize()
    return sel.cpu().numpy(), cnt.cpu().numpy(), sel2.cpu().numpy(), cnt2.cpu().numpy()


@pytest.mark.parametrize("kind", ["plain", "ties"])
@pytest.mark.parametrize("dtype,D", [(t, d) for t in ("f32", "bf16", "i8") for d in (64, 128, 256, 512)])
def test_score_select_equals_parts(dtype, D, kind):
    row = D * {"f32": 4, "bf16": 2, "i8": 1}[dtype]
    most = min(512, (128 << 10) // row)  # the rule's limits, and one past them
    for n in sorted({1, 2, 63, 64, 65, 127, 129, 200, 257, most - 1, most, most + 1}):
        for k in sorted({1, max(1, n // 8), max(1, n - 1), n}):
            a, ca, b, cb = _step_and_parts([n], [k], dtype, D, n * 1000 + k, kind)
            assert np.array_equal(ca, cb) and np.array_equal(a, b), (dtype, D, kind, n, k)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i8"])
def test_score_select_ragged(dtype):
    ns = [64, 1, 100, 33, 128, 65, 5, 90, 77, 120, 2]
    ks = [8, 1, 100, 5, 13, 64, 2, 1, 30, 119, 1]
    a, ca, b, cb = _step_and_parts(ns, ks, dtype, 256, 3, "ties")
    assert np.array_equal(ca, cb)
    for i, c in enumerate(ca):
        assert np.array_equal(a[i, :c], b[i, :c]), i
