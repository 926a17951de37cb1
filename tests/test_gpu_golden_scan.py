"""Golden-label rows at the sizes where the kernels change what they do: rows
held in registers (up to 16,384 entries), rows scanned in slices, a slice
boundary, rows that start inside a float4 (odd lengths), the largest entries in
one slice, slices masked with the type's lowest value, many equal logits, and
flat rows that the exact kernel decides after the scan.
Same oracle, band and exact follow-ups as the other golden-label tests.
"""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_golden import run_golden

pytestmark = pytest.mark.gpu


def _row(rng, shape, kind):
    x = rng.standard_normal(shape).astype(np.float32)
    n = shape[2]
    if kind == "peaked":  # 1 in 256 entries far above
        x[:, :, rng.choice(n, size=max(1, n // 256), replace=False)] += np.float32(8.0)
    elif kind == "clustered":  # all of them in one run
        at = int(rng.integers(0, max(1, n - n // 256)))
        x[:, :, at:at + max(1, n // 256)] += np.float32(8.0)
    elif kind == "masked":  # the second half masked out
        x[:, :, :max(1, n // 512)] += np.float32(9.0)
        x[:, :, n // 2:] = np.finfo(np.float32).min
    elif kind == "grid":  # many equal logits at the boundary, few levels
        x = (np.round(x * 2.0) / 2.0).astype(np.float32)
    elif kind == "offset":  # large values: the sums' error bound grows with them
        x = (x * 4.0 + np.float32(1000.0)).astype(np.float32)
    return x  # "flat": as drawn


@pytest.mark.parametrize("n", [2047, 2048, 2049, 4096, 16383, 16384, 16385, 32771, 65537])
@pytest.mark.parametrize("kind", ["peaked", "clustered", "masked", "grid", "offset", "flat"])
def test_golden_scanned_rows(n, kind):
    rng = np.random.default_rng(n * 11 + len(kind))
    run_golden([_row(rng, (1, 3, n), kind)], 1, 3, 2, 3, 5)


@pytest.mark.parametrize("p", [(1, 1000), (9, 10), (999, 1000), (1, 1)])
def test_golden_scanned_rows_p(p):
    rng = np.random.default_rng(p[0])
    # a short row first, so that the scanned rows after it start anywhere
    xs = [_row(rng, (2, 3, n), "peaked") for n in (333, 40001, 2050, 131074)]
    run_golden(xs, 2, 3, 2, p[0], p[1])
