"""Which rows the golden-label scan settles: a row whose set lies among the listed
entries must not be left open (it would be read twice more), and a row whose set
reaches below them must.  The sets themselves are compared elsewhere.
"""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_golden_exact import _row

pytestmark = pytest.mark.gpu

# peaked and masked rows: about 64 entries of 16,384 carry the set; flat ones: nearly half of all
OPEN = {"peaked": 0, "masked_peaks": 0, "flat": 32}


@pytest.mark.parametrize("n", [16385, 32769, 40003, 65536, 131071])
@pytest.mark.parametrize("kind", sorted(OPEN))
def test_golden_open_rows(n, kind):
    import torch
    import golden_open
    so = golden_open.lib()
    rng = np.random.default_rng(n + len(kind))
    rows = _row(rng, 32, n, "flat" if kind == "flat" else "peaked")
    if kind == "masked_peaks":  # the second half at the type's lowest value
        rows[:, n // 2:] = np.finfo(np.float32).min
    words = (n + 31) // 32
    x = torch.from_numpy(np.ascontiguousarray(rows).reshape(-1)).cuda()
    bits = torch.zeros(32 * words, dtype=torch.int32, device="cuda")
    rc = so.golden_scan_and_rows(x.data_ptr(), n, 32, 3, 5, bits.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    marks = bits.cpu().numpy().view(np.uint32).reshape(32, words)[:, so.golden_open_word()]
    assert int((marks == np.uint32(so.golden_open_mark())).sum()) == OPEN[kind], (n, kind)
