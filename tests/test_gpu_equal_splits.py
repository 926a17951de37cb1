"""Attention of batches at the edges of the equal-split rule (just below and
above its least work, nine sequences, a sequence at the split limit, an even
batch), through the fused step and the
separate calls, against the oracle."""
from __future__ import annotations

import pytest

import lsa_synth as synth
from gpu_case import run_case

pytestmark = pytest.mark.gpu

RAGGED = [400 + 331 * i % 1900 for i in range(9)]


def _keep(chunks):
    return [max(1, n * chunks // sum(RAGGED)) for n in RAGGED]


@pytest.mark.parametrize("name,ctx,keep,hq,hkv", [
    ("below", RAGGED, _keep(765), 32, 16),
    ("above", RAGGED, _keep(780), 32, 16),
    ("capped", [13000] + [64] * 8, [12500] + [6] * 8, 2, 1),
    ("even", [900] * 16, [110] * 16, 16, 8),
])
def test_equal_split_edges(name, ctx, keep, hq, hkv):
    prob = synth.Problem("equal_" + name, [64 * n for n in ctx], 64, keep, hq, hkv)
    run_case(prob, 3, seqs=[0, len(ctx) // 2, len(ctx) - 1], rows=[(0, 0), (0, hq - 1)])
