"""The kernel for listed strips of a sorted conversion, against the oracle, with the
lists' lengths read from the head of the workspace (so that the strips meant to be
listed are): more short strips than the launch has waves together with long ones, and
long strips at the limits of what a workgroup of 512 and of 1024 threads merges in LDS,
rows sorted, with one descent, and unsorted."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _check(k, height, dtype, cols, descents=(), shuffle=False, seed=0):
    """Convert rows of k distinct ascending columns; returns the two list lengths."""
    from paper_1203_2946_amd import cmrs
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(k)]).astype(np.int32)
    row = np.repeat(np.arange(k.size), k)
    c = rng.integers(0, cols, row.size)
    if not shuffle:
        c = c[np.lexsort((c, row))]
    ci = c.astype(np.int32)
    for at in descents:
        ci[at], ci[at + 1] = 9, 7
    val = rng.normal(size=ci.size).astype(dtype)
    rows = k.size
    ws = torch.zeros(cmrs.from_csr_workspace_bytes(rows, ci.size, height, True), dtype=torch.uint8, device="cuda")
    M = cmrs.from_csr(*(torch.from_numpy(a).cuda() for a in (rp, ci, val)), cols, height, sort=True, workspace=ws)
    sp, w, v = oracle.csr_to_cmrs(rp, ci, val, cols, height, sorted_=True)
    assert np.array_equal(M.strip_ptr.cpu().numpy(), sp)
    assert np.array_equal(M.col_word.cpu().numpy().view(np.uint32), w)
    assert np.array_equal(M.val.cpu().numpy().view(np.uint8), v.view(np.uint8))
    return ws[:8].view(torch.int32).tolist()


def _rows(total, height, shape, rng):
    """`height` row lengths that add up to total."""
    if shape == "equal":
        k = np.full(height, total // height)
        k[0] += total - int(k.sum())
    elif shape == "one":  # one long row
        k = rng.integers(0, 12, height)
        k[rng.integers(height)] += total - int(k.sum())
    else:  # two, three or four long rows
        k = rng.integers(0, 6, height)
        k[: int(shape)] += (total - int(k.sum())) // int(shape)
        k[0] += total - int(k.sum())
    return k


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shuffle", [False, True])
@pytest.mark.parametrize("height", [4, 8, 16])
def test_more_short_strips_than_waves(height, shuffle, dtype):
    rng = np.random.default_rng(height)
    short, ends = 512 * 8 + 300, [1025, 3000, 8192, 8193, 16384, 16385]
    strips = [rng.multinomial(n, np.full(height, 1 / height)) for n in rng.integers(530, 1025, short)]
    for n in ends:
        strips.insert(int(rng.integers(len(strips))), _rows(n, height, "one", rng))
    k = np.concatenate(strips + [np.ones(60_000 * height // 4, np.int64)])
    assert k.sum() * height / k.size < 320
    assert _check(k, height, dtype, 1 << 18, shuffle=shuffle) == [short, len(ends)]


@pytest.mark.parametrize("kind", ["sorted", "descent", "unsorted"])
@pytest.mark.parametrize("among", ["short strips", "long strips"])
@pytest.mark.parametrize("height,shape", [(1, "one"), (2, "equal"), (3, "2"), (4, "equal"), (8, "equal"), (8, "3"),
                                          (16, "2"), (32, "4"), (32, "equal"), (32, "one")])
def test_limits_of_a_workgroup(height, shape, among, kind):
    rng = np.random.default_rng(height)
    totals = [8191, 8192, 8193, 16383, 16384, 16385, 17000, 2100, 4097]
    strips = [_rows(n, height, shape, rng) for n in totals]
    if among == "short strips":  # 512 threads
        strips += [np.full(height, 2)] * 9000
    k = np.concatenate(strips)
    mean = k.sum() * height / k.size
    assert mean < 320 if among == "short strips" else 3800 <= mean < 15000
    rp = np.concatenate([[0], np.cumsum(k)])
    descents = []
    if kind == "descent":  # inside the longest row of every long strip
        for s in range(len(totals)):
            r = s * height + int(np.argmax(k[s * height:(s + 1) * height]))
            descents.append(int(rp[r]) + [0, 62, 63, 511, 1022, 1023][s % 6] % (int(k[r]) - 1))
    counts = _check(k, height, np.float32 if height == 8 else np.float64, 1 << 18, descents, kind == "unsorted", height)
    assert counts[1] == len(totals)
