"""The strip-group product's choice of stream loads and of loads per step: the
same bits from the automatic choice and both explicit ones, on both sides of
every group width and of the fp64 four-load step, within the bound of the
path against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("height", [1, 4, 8, 12, 32])
@pytest.mark.parametrize("per_row", [1, 3, 7, 14, 29, 57])
def test_automatic_choice_gives_the_explicit_bits(dtype, height, per_row):
    from paper_1203_2946_amd import cmrs
    A = synth.random_csr(701, 900, max_row=2 * per_row, seed=per_row, canonical=True)
    rp, ci, v, hv = G.upload(A, dtype)
    M = cmrs.from_csr(rp, ci, v, A.cols, height, sort=True)
    x, x64 = G.xy_vector(synth.uniform_vector(A.cols, seed=2), dtype)
    y = [cmrs.spmv(M, x, variant=k) for k in ("auto", "group", "group_nt")]
    assert torch.equal(y[0], y[1]) and torch.equal(y[0], y[2])
    hv64 = G.vals_as_f64(hv, dtype)
    ref = oracle.csr_spmv(A.row_ptr, A.col_ind, hv64, x64)
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    bound = oracle.spmv_bound(A.row_ptr, A.col_ind, hv64, x64, u, factor=4.0)
    # One more rounding where the result is stored narrower than its exact value.
    assert np.all(np.abs(y[0].cpu().numpy().astype(np.float64) - ref) <= bound + u * np.abs(ref))
