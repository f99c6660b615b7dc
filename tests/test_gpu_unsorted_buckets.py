"""Sorted conversion of strips with unsorted rows that one wave holds, from height
16 on: strips of up to the wave's 512 entries bucketed by the wave that loaded them,
listed ones of up to 1024 by the list kernel's waves; uniform columns, equal words
(ties keep CSR order), columns bunched at two places far apart (a bitonic network),
sorted and unsorted strips side by side, at the edges of slots and capacities."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("height", [8, 16, 21, 32])
@pytest.mark.parametrize("kind", ["uniform", "ties", "bunched", "one column", "mixed"])
def test_unsorted_strips_of_one_wave(kind, height, dtype):
    from paper_1203_2946_amd import cmrs
    rng = np.random.default_rng(height)
    totals = [0, 1, 2, 63, 64, 65, 255, 256, 257, 260, 300, 448, 500, 511, 512, 513, 700, 1000, 1023, 1024, 1025, 2047]
    totals = rng.permutation(np.concatenate([totals, np.full(90, 200)]))
    k = np.concatenate([np.diff(np.sort(np.concatenate([[0, n], rng.integers(0, n + 1, height - 1)]))) for n in totals])
    cols = 90_000
    n = int(k.sum())
    if kind == "bunched":
        ci = np.where(rng.random(n) < 0.5, rng.integers(0, 5, n), cols - 1 - rng.integers(0, 5, n))
    elif kind == "one column":
        ci = np.full(n, 77)
    else:
        ci = rng.integers(0, 200 if kind == "ties" else cols, n)
    if kind == "mixed":  # every second strip's rows ascend
        row = np.repeat(np.arange(k.size), k)
        up = ci[np.lexsort((ci, row))]
        ci = np.where((row // height) % 2 == 0, up, ci)
    rp = np.concatenate([[0], np.cumsum(k)]).astype(np.int32)
    assert rp[-1] / totals.size < 320 and 2.5 * rp[-1] / totals.size > 256
    ci, val = ci.astype(np.int32), rng.normal(size=n).astype(dtype)
    M = cmrs.from_csr(*(torch.from_numpy(a).cuda() for a in (rp, ci, val)), cols, height, sort=True)
    sp, w, v = oracle.csr_to_cmrs(rp, ci, val, cols, height, sorted_=True)
    assert np.array_equal(M.strip_ptr.cpu().numpy(), sp)
    assert np.array_equal(M.col_word.cpu().numpy().view(np.uint32), w)
    assert np.array_equal(M.val.cpu().numpy().view(np.uint8), v.view(np.uint8))
