"""Sorted conversion of tall strips on both sides of the strip count that takes
wider workgroups, with columns that bucket well, columns bunched at a few places
far apart (bucketing given up for the merge) and strips of both kinds."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("strips", [1, 40, 1024, 1025])
@pytest.mark.parametrize("mean", [460, 905])
@pytest.mark.parametrize("height", [24, 32])
@pytest.mark.parametrize("kind", ["uniform", "bunched", "both"])
def test_tall_strips_by_count_and_columns(kind, height, mean, strips):
    from paper_1203_2946_amd import cmrs
    rng = np.random.default_rng(strips + mean)
    rows, cols = strips * height - (height // 2 if strips > 1 else 0), 200_000
    k = rng.integers(mean // height - 3, mean // height + 6, rows)
    rp = np.concatenate([[0], np.cumsum(k)]).astype(np.int32)
    row = np.repeat(np.arange(rows), k)
    c = rng.integers(0, cols, rp[-1])
    near = (rng.integers(0, 7, rp[-1]) * 30_000 + rng.integers(0, 60, rp[-1]))
    pick = {"uniform": np.zeros(rows, bool), "bunched": np.ones(rows, bool), "both": (np.arange(rows) // height) % 2 == 1}
    c = np.where(pick[kind][row], near, c)
    ci = c[np.lexsort((c, row))].astype(np.int32)
    val = rng.normal(size=ci.size)
    M = cmrs.from_csr(*(torch.from_numpy(a).cuda() for a in (rp, ci, val)), cols, height, sort=True)
    sp, w, v = oracle.csr_to_cmrs(rp, ci, val, cols, height, sorted_=True)
    assert np.array_equal(M.strip_ptr.cpu().numpy(), sp)
    assert np.array_equal(M.col_word.cpu().numpy().view(np.uint32), w)
    assert np.array_equal(M.val.cpu().numpy().view(np.uint64), v.view(np.uint64))
