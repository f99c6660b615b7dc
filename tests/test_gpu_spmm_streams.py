"""Single products on both sides of the line between cached and non-temporal
stream loads (16 and 32 lanes per strip), for strips that end inside a vector
of entries, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("nrhs", [1, 2])
@pytest.mark.parametrize("group", [1, 16, 32, 64])
@pytest.mark.parametrize("per_row", [1, 9, 33])
def test_small_products_by_group_width(dtype, nrhs, group, per_row):
    from paper_1203_2946_amd import cmrs
    A = synth.random_csr(517, 640, max_row=2 * per_row, seed=per_row, canonical=True)
    rp, ci, v, hv = G.upload(A, dtype)
    M = cmrs.from_csr(rp, ci, v, A.cols, 4, sort=True)
    xdt = torch.float64 if dtype == "f64" else torch.float32
    X = torch.as_tensor(synth.uniform_vector(A.cols * nrhs, seed=7).reshape(A.cols, nrhs)).to(xdt)
    Y = cmrs.spmm(M, X.cuda(), group=group).cpu().numpy().astype(np.float64)
    hv64 = G.vals_as_f64(hv, dtype)
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    for k in range(nrhs):
        x64 = np.ascontiguousarray(X[:, k].numpy().astype(np.float64))
        ref = oracle.csr_spmv(A.row_ptr, A.col_ind, hv64, x64)
        bound = oracle.spmv_bound(A.row_ptr, A.col_ind, hv64, x64, u, factor=4.0)
        assert np.all(np.abs(Y[:, k] - ref) <= bound + u * np.abs(ref))
