"""Sorted conversion at the edges of the row-run merge: strips of every slot
count and remainder a wave takes, runs around powers of two (the merge's search
steps), one long row at either end of a strip, empty rows between."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _lengths(kind, height, rng):
    if kind == "powers":  # every run length 2^k - 1, 2^k, 2^k + 1 up to 33
        k = np.array([0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33])
        return rng.permutation(np.resize(k, 40 * height))
    if kind == "ends":  # the long row first or last of its strip, the others empty or single
        out = []
        for n in (1, 63, 64, 65, 127, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 1500):
            for at in (0, height - 1):
                strip = rng.integers(0, 2, height)
                strip[at] = n
                out.append(strip)
        return np.concatenate(out)
    # "slots": strips whose total steps through the slots of a wave, ragged last strip
    out = []
    for total in range(1, 8 * 64 + 2, 29):
        cut = np.sort(rng.integers(0, total + 1, height - 1)) if height > 1 else np.zeros(0, np.int64)
        out.append(np.diff(np.concatenate([[0], cut, [total]])))
    return np.concatenate(out)[:-1] if height > 1 else np.concatenate(out)


@pytest.mark.parametrize("height", [1, 2, 3, 4, 7, 8, 16, 21, 32])
@pytest.mark.parametrize("kind", ["powers", "ends", "slots"])
def test_sorted_conversion_at_the_edges(kind, height):
    from paper_1203_2946_amd import cmrs
    rng = np.random.default_rng(height)
    k = _lengths(kind, height, rng)
    cols = 1600
    rp = np.concatenate([[0], np.cumsum(k)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(cols, n, replace=False)) for n in k]).astype(np.int32)
    val = rng.normal(size=ci.size)
    M = cmrs.from_csr(*(torch.from_numpy(a).cuda() for a in (rp, ci, val)), cols, height, sort=True)
    sp, w, v = oracle.csr_to_cmrs(rp, ci, val, cols, height, sorted_=True)
    assert np.array_equal(M.strip_ptr.cpu().numpy(), sp)
    assert np.array_equal(M.col_word.cpu().numpy().view(np.uint32), w)
    assert np.array_equal(M.val.cpu().numpy().view(np.uint64), v.view(np.uint64))


def _check(rp, ci, cols, height, dtype=np.float64):
    from paper_1203_2946_amd import cmrs
    val = np.random.default_rng(1).normal(size=ci.size).astype(dtype)
    M = cmrs.from_csr(*(torch.from_numpy(a).cuda() for a in (rp, ci, val)), cols, height, sort=True)
    sp, w, v = oracle.csr_to_cmrs(rp, ci, val, cols, height, sorted_=True)
    assert np.array_equal(M.strip_ptr.cpu().numpy(), sp)
    assert np.array_equal(M.col_word.cpu().numpy().view(np.uint32), w)
    assert np.array_equal(M.val.cpu().numpy().view(np.uint8), v.view(np.uint8))


@pytest.mark.parametrize("height", [1, 8, 32])
@pytest.mark.parametrize("mean", [449, 451, 899, 901, 1024, 1849, 2050, 3799])
@pytest.mark.parametrize("kind", ["spread", "band", "unsorted", "bunched"])
def test_one_workgroup_per_strip(kind, mean, height):
    """Mean strips on both sides of every shape's limit, strips below and above
    its capacity: spread columns, a band, unsorted rows, and unsorted rows whose
    columns bunch at the two ends (no bucketing)."""
    rng = np.random.default_rng(mean + height)
    strips = 9
    total = rng.permutation(np.linspace(0.1, 1.9, strips) * mean).astype(int)
    k = np.concatenate([np.diff(np.sort(np.concatenate([[0, n], rng.integers(0, n + 1, height - 1)]))) for n in total])
    cols = 100_000 if kind == "spread" else 8_000
    rows = []
    for i, n in enumerate(k):
        if kind == "bunched":
            c = np.where(rng.random(n) < 0.5, rng.integers(0, 6, n), cols - 1 - rng.integers(0, 6, n))
        elif kind == "band":
            c = np.sort(rng.choice(min(cols, max(2 * n, 60)), n, replace=False))
        else:
            c = rng.choice(cols, n, replace=False)
        rows.append(np.sort(c) if kind == "spread" else c)
    rp = np.concatenate([[0], np.cumsum(k)]).astype(np.int32)
    _check(rp, np.concatenate(rows).astype(np.int32), cols, height, np.float32 if height == 8 else np.float64)


@pytest.mark.parametrize("lengths", [
    [600] * 16, [3000, 0, 2900, 5] + [1] * 12, [1100, 1100] + [64] * 14, [9000] + [65, 64] * 7 + [3], [700] * 15 + [5000],
    [64] * 15 + [4000], [2000, 2000, 2000] + [2] * 13])
@pytest.mark.parametrize("descents", [0, 1])
def test_listed_long_strips(lengths, descents):
    """Strips past every list's capacity among many single-entry rows: one, two
    and more long rows, many equal rows, light rows at their limit; with one
    descending pair too (the output is then written again)."""
    rng = np.random.default_rng(len(lengths) + lengths[0])
    k = np.concatenate([np.ones(16 * 800, np.int64), lengths, np.ones(16 * 40, np.int64), lengths])
    cols = 60_000
    rp = np.concatenate([[0], np.cumsum(k)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(cols, n, replace=False)) for n in k]).astype(np.int32)
    if descents:
        r = 16 * 800 + int(np.argmax(lengths))
        at = rp[r] + 63
        ci[at], ci[at + 1] = ci[at + 1], ci[at]
    _check(rp, ci, cols, 16)
