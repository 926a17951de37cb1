"""Top-k over 16,385 to 65,536 chunks (the register-held selection of long
contexts) at the edges of its variants, against a stable sort of identical scores:
bit-exact kept sets, with ties, signed zeros, all-equal scores (a threshold bin
too large to pack), one chunk kept and all chunks kept, several queries, and
the extremes of int32 scores.
"""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _topk(scores, k, dtype, Q=1):
    import torch
    import paper_2606_09079_amd as L
    n = scores.shape[-1]
    P = L.Problem([64 * n], 64, [k], 8, 8, emb_dim=64, n_lookahead=Q, emb_dtype=dtype)
    sel = torch.full((1, L.lsa_max_sel(P)), -1, dtype=torch.int32, device="cuda")
    cnt = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    pq = torch.full((1, Q, k), -1, dtype=torch.int32, device="cuda")
    L.lsa_topk_chunks(P, torch.from_numpy(np.ascontiguousarray(scores)).cuda(), sel, cnt, pq)
    torch.cuda.synchronize()
    return pq.cpu().numpy()[0], sel.cpu().numpy()[0, :int(cnt.item())]


def _want(row, k):
    order = np.lexsort((np.arange(len(row)), -row.astype(np.float64) + 0.0))
    return np.sort(order[:k])


@pytest.mark.parametrize("n", [16385, 24576, 24577, 40003, 40960, 40961, 65535, 65536])
@pytest.mark.parametrize("kind", ["normal", "grid", "equal"])
def test_topk_wide_f32(n, kind):
    rng = np.random.default_rng(n)
    x = rng.standard_normal((2, n)).astype(np.float32)
    if kind == "grid":  # ties and both zeros
        x = np.round(x * 2.0).astype(np.float32) / np.float32(2.0)
        x[:, ::7] = np.float32(-0.0)
    elif kind == "equal":
        x[:] = np.float32(0.25)
    for k in (1, n // 10, n):
        per_query, union = _topk(x, k, "f32", Q=2)
        for j in range(2):
            assert np.array_equal(per_query[j], _want(x[j], k)), (n, kind, k, j)
        assert np.array_equal(union, np.union1d(_want(x[0], k), _want(x[1], k)))


@pytest.mark.parametrize("n", [16500, 30000, 50000])
def test_topk_wide_i32(n):
    rng = np.random.default_rng(n)
    for lo, hi in ((-2 ** 31, 2 ** 31 - 1), (-5, 5), (-2 ** 31, -2 ** 31 + 2)):
        x = rng.integers(lo, hi, size=(1, n), endpoint=True, dtype=np.int64).astype(np.int32)
        x[0, :3] = [-2 ** 31, 2 ** 31 - 1, 0]
        for k in (1, 700, n):
            _, sel = _topk(x, k, "i8")
            assert np.array_equal(sel, _want(x[0], k)), (n, lo, k)


@pytest.mark.parametrize("n", [16385, 33000, 65000])
def test_recall_wide(n):
    """The recall's threshold, maximum over layers and bound on a long context."""
    import torch
    import paper_2606_09079_amd as L
    rng = np.random.default_rng(n + 1)
    x = (rng.standard_normal((3, n)) - 1.5).astype(np.float32)
    x[0, :5] = np.float32(-0.0)
    r = x.max(0)
    for k in (1, 900, n):
        for shift in (0.0, -10.0):  # the second: nothing recalled but the zeros of layer 0
            y = np.where(x == 0, x, x + np.float32(shift)).astype(np.float32)
            r = y.max(0)
            P, ix = L.Problem([64 * n], 64, [k], 8, 8), L.Indexer(3, 16, 64)
            sel = torch.full((1, L.lsa_max_sel(P)), -1, dtype=torch.int32, device="cuda")
            cnt = torch.full((1,), -1, dtype=torch.int32, device="cuda")
            L.lsa_recall_select(P, ix, torch.from_numpy(y).cuda(), sel, cnt)
            torch.cuda.synchronize()
            want = _want(r, min(k, int((r >= 0).sum())))
            assert np.array_equal(sel.cpu().numpy()[0, :int(cnt.item())], want), (n, k, shift)
