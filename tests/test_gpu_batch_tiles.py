"""The batched product's tiles: the same bits from the default tile size and
explicit ones, with one tile, fewer tiles than waves and several tiles per
wave, on the first launch and on later ones of the same plan (the queue
counters are reset by the launch itself)."""
import pytest
import torch

import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("height", [1, 4, 16])
@pytest.mark.parametrize("rows,count", [(5, 1), (2_000, 3), (21_000, 3), (60_000, 7)])
def test_default_tiles_give_the_explicit_bits(dtype, height, rows, count):
    from paper_1203_2946_amd import cmrs
    mats, Xs = [], []
    for k in range(count):
        A = synth.random_csr(rows + k, rows, max_row=12, seed=k, canonical=True)
        rp, ci, v, _ = G.upload(A, dtype)
        mats.append(cmrs.from_csr(rp, ci, v, A.cols, height, sort=True))
        X = synth.uniform_vector(A.cols * (1 + k), seed=k).reshape(A.cols, 1 + k)
        Xs.append(torch.as_tensor(X, device="cuda").to(v.dtype).contiguous())
    want = [cmrs.spmm(M, X) for M, X in zip(mats, Xs)]
    tiles = []
    for tile_nnz in (0, 1, 500, 32768):
        Ys = [torch.empty_like(w) for w in want]
        plan = cmrs.spmm_plan(mats, Xs, Ys, tile_nnz=tile_nnz)
        tiles.append(plan.tiles)
        first = None
        for _ in range(3):
            for Y in Ys:
                Y.fill_(float("nan"))
            cmrs.spmm_batched(plan)
            if first is None:
                first = [Y.clone() for Y in Ys]
            assert all(torch.equal(a, b) for a, b in zip(first, Ys))
        if tile_nnz == 0:
            default = first
        assert all(torch.equal(a, b) for a, b in zip(first, default))
    # The single product may take another group width: sums of at most 16 * 12
    # entries in another order, two roundings each.
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    for w, d, M, X in zip(want, default, mats, Xs):
        assert torch.all((w - d).abs() <= 2 * 12 * u * cmrs.spmm(cmrs.from_csr(*_absolute(M)), X.abs()) + 1e-300)
    nnz = sum(int(M.nnz) for M in mats)
    assert (tiles[0] == tiles[3]) == (nnz < 262144)


def _absolute(M):
    from paper_1203_2946_amd import cmrs
    rp, ci, v = cmrs.to_csr(M)
    return rp, ci, v.abs(), M.cols, M.height


def test_default_plan_in_a_buffer_of_coarse_tiles():
    """A buffer sized for tiles of 32768 entries takes the default tuning too;
    one byte less is refused with either."""
    import ctypes
    from paper_1203_2946_amd import cmrs
    A = synth.random_csr(60_000, 60_000, max_row=12, seed=3, canonical=True)
    rp, ci, v, _ = G.upload(A, "f64")
    M = cmrs.from_csr(rp, ci, v, A.cols, 4, sort=True)
    X = torch.as_tensor(synth.uniform_vector(A.cols, seed=1).reshape(A.cols, 1), device="cuda")
    assert int(M.nnz) >= 262144
    descs, one = (cmrs.CmrsMatDesc * 1)(M.desc()), (ctypes.c_int32 * 1)(1)
    least = int(cmrs.lib.cmrs_spmm_plan_bytes(1, descs, one, ctypes.byref(cmrs.SpmmTuning(32768, 0, 0, 0))))
    assert least < int(cmrs.lib.cmrs_spmm_plan_bytes(1, descs, one, None))
    Y = torch.full_like(X, float("nan"))
    xp, yp = (ctypes.c_void_p * 1)(X.data_ptr()), (ctypes.c_void_p * 1)(Y.data_ptr())
    buf = torch.empty(least, dtype=torch.uint8, device="cuda")
    for tuning in (None, ctypes.byref(cmrs.SpmmTuning(32768, 0, 0, 0))):
        plan = cmrs.SpmmPlanStruct()
        args = (1, descs, one, xp, one, yp, one, 0, tuning, buf.data_ptr())
        assert cmrs.lib.cmrs_spmm_plan(*args, least - 1, ctypes.byref(plan), cmrs._stream()) == cmrs.CMRS_ERR_WORKSPACE
        assert cmrs.lib.cmrs_spmm_plan(*args, least, ctypes.byref(plan), cmrs._stream()) == cmrs.CMRS_OK
        Y.fill_(float("nan"))
        assert cmrs.lib.cmrs_spmm_batched(ctypes.byref(plan), cmrs._stream()) == cmrs.CMRS_OK
        assert torch.equal(Y, cmrs.spmm(M, X))
