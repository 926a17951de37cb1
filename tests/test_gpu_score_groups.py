"""Scores of several lookahead queries over bf16 embeddings, at the numbers of
chunks where the matrix kernel changes how many 16-chunk groups a wave takes
(one, two or four), for one sequence and for a ragged batch of the same total,
against float64: a dot product of D bf16 values in float32 is off by at most
D 2^-24 times the sum of the products' sizes."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,Q", [(64, 16), (128, 8), (256, 4), (256, 16), (512, 4), (512, 16)])
@pytest.mark.parametrize("total", [16384, 16385, 32768, 32769, 49153, 65536, 65537, 131073])
def test_score_groups(D, Q, total):
    import torch
    import paper_2606_09079_amd as L
    g = torch.Generator(device="cuda")
    g.manual_seed(total + D + Q)
    E = torch.randn(total, D, generator=g, device="cuda").to(torch.bfloat16)
    for ns in ([total], [1, 63, total // 3, total - 64 - total // 3]):
        B = len(ns)
        qe = torch.randn(B, Q, D, generator=g, device="cuda").to(torch.bfloat16)
        p = L.Problem([64 * n for n in ns], 64, [1] * B, 8, 8, emb_dim=D, n_lookahead=Q)
        scores = torch.full((Q * total,), float("nan"), device="cuda")
        L.lsa_score_chunks(p, qe, E, scores)
        off = 0
        for b, n in enumerate(ns):
            got = scores[Q * off:Q * (off + n)].view(Q, n).double()
            e, q = E[off:off + n].double(), qe[b].double()
            err = (got - q @ e.t().contiguous()).abs()
            assert bool((err <= D * 2.0 ** -24 * (q.abs() @ e.abs().t().contiguous()) + 1e-30).all()), (D, Q, ns, b)
            off += n
