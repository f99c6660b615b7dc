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
