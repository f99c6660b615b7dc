"""Sorted conversion of many tall strips on both sides of each line of its dispatch
(workgroups of 128, 256 and 512 threads, the group kernel below; strips that are all
resident at once), with strips past the workgroup's capacity: spread columns, a band,
columns bunched at a few places (full buckets: merged), unsorted rows, and unsorted
rows bunched at the two ends (the bitonic network); heights below and from the one
where sorted rows are bucketed, every value size."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["spread", "band", "clusters", "unsorted", "ends"])
@pytest.mark.parametrize("height", [4, 13, 16, 32])
@pytest.mark.parametrize("mean,strips", [(325, 3072), (325, 3073), (446, 3072), (455, 1025), (896, 1025), (905, 1025),
                                         (1845, 1025), (1856, 1025)])
def test_many_tall_strips(kind, height, mean, strips):
    from paper_1203_2946_amd import cmrs
    rng = np.random.default_rng(mean + height)
    rows, cols = strips * height - height // 2, 150_000
    order = rng.permutation(rows)
    k = np.zeros(rows, np.int64)                      # an eighth of the rows stays empty
    k[rng.permutation(strips - 1)[: max(2, strips // 300)] * height] = 2 * mean
    some = order[rows // 8:]
    left = mean * strips - int(k.sum())
    k[some] += left // some.size
    k[some[: left % some.size]] += 1
    assert int(k.sum()) == mean * strips
    row = np.repeat(np.arange(rows), k)
    n = row.size
    if kind == "band":
        c = np.clip(row * cols // rows + rng.integers(-60, 61, n), 0, cols - 1)
    elif kind == "clusters":
        c = rng.integers(0, 5, n) * 30_000 + rng.integers(0, 9, n)
    elif kind == "ends":
        c = np.where(rng.random(n) < 0.5, rng.integers(0, 6, n), cols - 1 - rng.integers(0, 6, n))
    else:
        c = rng.integers(0, cols, n)
    if kind in ("spread", "band", "clusters"):
        c = c[np.lexsort((c, row))]
    rp, ci = np.concatenate([[0], np.cumsum(k)]).astype(np.int32), c.astype(np.int32)
    val = rng.normal(size=n).astype({4: np.float32, 13: np.float64, 16: np.float64, 32: np.float32}[height])
    bits = torch.from_numpy(val).cuda()
    if height == 4:
        bits = bits.to(torch.bfloat16)
        val = bits.cpu().view(torch.int16).numpy().view(np.uint16)
    M = cmrs.from_csr(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), bits, cols, height, sort=True)
    sp, w, v = oracle.csr_to_cmrs(rp, ci, val, cols, height, sorted_=True)
    assert np.array_equal(M.strip_ptr.cpu().numpy(), sp)
    assert np.array_equal(M.col_word.cpu().numpy().view(np.uint32), w)
    assert np.array_equal(M.val.cpu().view(torch.uint8).numpy(), v.view(np.uint8))
