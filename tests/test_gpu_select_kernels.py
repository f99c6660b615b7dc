"""Edges of the selector kernels: batches around the rows a workgroup and a
wave of the network take, structures around the rows and entries a wave of the
feature count takes."""
import numpy as np
import pytest
import torch

from oracle import selector_ref as R

pytestmark = pytest.mark.gpu


def _sel():
    from paper_1203_2946_amd import selector
    return selector


@pytest.mark.parametrize("batch", [1, 3, 8, 9, 64, 67, 511, 513, 2000])
def test_fused_gradients_equal_the_separate_calls(batch):
    """cmrs_mlp_grads runs forward, loss gradient and backward exactly as the
    three calls do: the same bits, and gradients within the error of a batch
    sum of fp32 products of the fp64 reference, from the kernel's own dY and
    activations (so only the last sum's rounding counts)."""
    S = _sel()
    g = np.random.default_rng(batch)
    X = torch.from_numpy(g.uniform(0, 1, (batch, 40)).astype(np.float32)).cuda()
    T = torch.from_numpy(g.normal(0, 1, (batch, 24)).astype(np.float32)).cuda()
    m = S.Mlp(S.init_params(batch, "cuda"))
    Y, grads = m.grads(X, T)
    H1, H2, Y3 = m.forward(X)
    dY, dH2, dH1 = torch.empty_like(Y3), torch.empty_like(H2), torch.empty_like(H1)
    g3 = torch.full_like(m.params, float("nan"))
    p = [t.data_ptr() for t in (X, m.params, H1, H2, dY, dH2, dH1, g3)]
    assert S._L.cmrs_mse_grad(Y3.numel(), Y3.data_ptr(), T.data_ptr(), dY.data_ptr(), 2.0 / Y3.numel(), S._s()) == 0
    assert S._L.cmrs_mlp_backward(batch, *p, S._s()) == 0
    torch.cuda.synchronize()
    assert torch.equal(Y, Y3) and torch.equal(grads, g3)
    ref, scale = [], []
    for a, d in ((X, dH1), (H1, dH2), (H2, dY)):
        a, d = a.double(), d.double()
        ref += [(a.T @ d).reshape(-1), d.sum(0)]
        scale += [(a.abs().T @ d.abs()).reshape(-1), d.abs().sum(0)]
    err = (grads.double() - torch.cat(ref)).abs()
    assert bool((err <= (batch + 2) * 2.0 ** -24 * torch.cat(scale) + 1e-30).all())


@pytest.mark.parametrize("rows,cols,lengths", [
    (1, 7, [7]), (63, 40, [3]), (64, 64, [1]), (65, 9000, [0, 5]), (129, 100, [0, 0, 0, 4]), (64, 600, [8]),
    (513, 513, [1, 2, 3]), (200, 70_000, [0, 600, 1]), (5000, 31, [0, 7, 31]), (70_000, 70_000, [2, 0, 1])])
def test_features_at_the_edges_of_a_wave(rows, cols, lengths):
    """Rows around 64, empty rows in front, between and behind, runs that end
    inside a 4-entry load, rectangular shapes: the same counts as the
    reference."""
    S = _sel()
    k = np.resize(np.array(lengths), rows)
    rp = np.concatenate([[0], np.cumsum(k)])
    g = np.random.default_rng(rows)
    ci = np.concatenate([np.sort(g.choice(cols, n, replace=False)) for n in k] + [np.zeros(0, np.int64)])
    got = S.features(torch.from_numpy(rp.astype(np.int32)).cuda(), torch.from_numpy(ci.astype(np.int32)).cuda(),
                     cols).cpu().numpy()
    ref = R.features(rp, ci.astype(np.int64), cols)
    np.testing.assert_array_equal(got[:36], ref[:36])
    np.testing.assert_allclose(got[36:], ref[36:], rtol=8 * 2.0 ** -24, atol=0)
