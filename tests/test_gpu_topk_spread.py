"""Top-k up to 16,384 chunks where one histogram over the scores' range settles
the selection and where it must hand over to the radix passes: outliers that
squeeze the other scores into one bin or a few, masked scores, many equal scores
at the boundary (a threshold bin of 65 to 256 keys), two clusters, subnormal and huge ranges, all-equal scores, at the edges of the
kernel's variants.  Kept sets equal a stable sort of the same scores.
"""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_topk_wide import _topk, _want

pytestmark = pytest.mark.gpu


def _scores(rng, n, kind):
    x = rng.standard_normal((2, n)).astype(np.float32)
    if kind == "outlier":
        x[0, n // 2] = np.float32(1e30)
        x[1, n // 3] = np.float32(-1e30)
    elif kind == "squeezed":  # one that leaves the others 20 bins each standard deviation
        x[:, n // 2] = np.float32(200.0)
    elif kind == "masked":  # half at the type's lowest value
        x[:, n // 2:] = np.finfo(np.float32).min
    elif kind == "boundary":  # 70 equal scores where the set ends
        x = np.sort(x, axis=1)[:, ::-1].copy()
        at = max(0, n // 10 - 35)
        x[:, at:at + 70] = x[:, at:at + 1]
        x = x[:, rng.permutation(n)]
    elif kind == "clusters":
        x[:, ::2] = x[:, ::2] * np.float32(1e-6) + np.float32(5.0)
    elif kind == "subnormal":
        x = (x * np.float32(1e-40)).astype(np.float32)
    elif kind == "huge":
        x = (np.sign(x) * np.float32(3e38) * rng.random((2, n)).astype(np.float32)).astype(np.float32)
    elif kind == "equal":
        x[:] = np.float32(-0.0)
        x[:, 1::2] = np.float32(0.0)
    return x


@pytest.mark.parametrize("kind", ["normal", "outlier", "squeezed", "masked", "boundary", "clusters", "subnormal", "huge",
                                  "equal"])
@pytest.mark.parametrize("n", [1, 2, 64, 65, 1023, 2048, 2049, 4097, 8192, 8193, 16384])
def test_topk_spread(n, kind):
    rng = np.random.default_rng(n + len(kind))
    x = _scores(rng, n, kind)
    for k in sorted({1, max(1, n // 10), max(1, n - 1), n}):
        per_query, union = _topk(x, k, "f32", Q=2)
        for j in range(2):
            assert np.array_equal(per_query[j], _want(x[j], k)), (n, kind, k, j)
        assert np.array_equal(union, np.union1d(_want(x[0], k), _want(x[1], k)))


@pytest.mark.parametrize("n", [500, 4000, 16384])
def test_recall_spread(n):
    import torch
    import paper_2606_09079_amd as L
    rng = np.random.default_rng(n)
    for kind in ("normal", "outlier", "squeezed", "masked", "huge", "equal"):
        x = _scores(rng, n, kind)
        r = x.max(0)
        for k in (1, max(1, n // 8), n):
            P, ix = L.Problem([64 * n], 64, [k], 8, 8), L.Indexer(2, 16, 64)
            sel = torch.full((1, L.lsa_max_sel(P)), -1, dtype=torch.int32, device="cuda")
            cnt = torch.full((1,), -1, dtype=torch.int32, device="cuda")
            L.lsa_recall_select(P, ix, torch.from_numpy(np.ascontiguousarray(x)).cuda(), sel, cnt)
            torch.cuda.synchronize()
            want = _want(r, min(k, int((r >= 0).sum())))
            assert np.array_equal(sel.cpu().numpy()[0, :int(cnt.item())], want), (n, kind, k)


@pytest.mark.parametrize("n", [64, 500, 2048, 4097, 8192, 16384])
@pytest.mark.parametrize("share", [2, 16])
def test_unset_scores(n, share):
    """Scores with every bit set (memory that was never written) are NaN and map
    to key 0: below every other score, in entry order among themselves, whether
    or not the kept set reaches them."""
    rng = np.random.default_rng(n * share)
    x = rng.standard_normal((2, n)).astype(np.float32)
    order = x.copy()
    for j in range(2):
        at = rng.permutation(n)[:n - n // share]
        x[j].view(np.uint32)[at] = np.uint32(0xFFFFFFFF)
        order[j, at] = -np.inf
    for k in sorted({1, n // share, n // share + 1, n - 1, n}):
        per_query, _ = _topk(x, k, "f32", Q=2)
        for j in range(2):
            assert np.array_equal(per_query[j], _want(order[j], k)), (n, share, k, j)
