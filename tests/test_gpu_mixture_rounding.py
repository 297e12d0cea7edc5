"""Roundings of single terms of the mixture fit's gradients, at one point and one component per problem, restated in
numpy's binary32 operation by operation.  The exponential is the device's own: a Gaussian component of weight 0 against the
target -1/2 has residual 1/2, and its gradient by the weight is exp(-d^2 / (2 s^2 + eps)) itself."""
import numpy as np
import pytest
import torch

from paper_2402_10128_amd import ges as G

pytestmark = pytest.mark.gpu
F = np.float32
GMM, DOG, LOG = (G.MIX_MODELS[k] for k in ("gmm", "dog", "log"))


def _gradients(model, w, d, s):
    """Gradients (by weight, centre, scale) of components of weight w and scale s at distance d, residual 1/2."""
    P = len(d)
    problems = np.zeros((P, 4), np.int32)
    problems[:, 0], problems[:, 1] = model, 1
    params = np.zeros((P, 128, 4), F)
    params[:, 0, 0], params[:, 0, 1], params[:, 0, 2], params[:, 0, 3] = w, -d, s, 2.0
    grad = torch.zeros((P, 128, 4), device="cuda:0")
    G.ges_mix_fit(torch.from_numpy(problems).cuda(), torch.full((1, 1), -0.5, device="cuda:0"), 0.0, 1.0,
                  torch.from_numpy(params).cuda(), 1, 0.0, grad_out=grad)
    return grad.cpu().numpy()[:, 0, :3]


def test_quotient_of_the_laplacian_next_to_a_tie():
    """2 d^2 / s^3 is one division by s in the definition.  Scales just below a power of two: the quotients of the first
    three pairs lie next to a tie between two numbers."""
    below = np.nextafter(F(1), F(0))
    d = F([0.4999999701976776, 0.2499999850988388, 1.4142135381698608])
    s = np.full(3, below, F)
    rng = np.random.default_rng(1)
    d = np.concatenate([d, rng.uniform(0.1, 3.0, 4000).astype(F)])
    s = np.concatenate([s, np.where(rng.random(4000) < 0.5, below, rng.uniform(0.3, 3.0, 4000).astype(F))]).astype(F)
    E = _gradients(GMM, F(0), d, s)[:, 0]
    w = F(2.0) ** -40   # the residual stays 1/2, the gradient by s is 2^-40 times the derivative
    d2, is2 = d * d, F(1) / (s * s)
    inv1 = F(1) / (F(2) * s * s + F(1e-8))
    base = (F(1) - d2 * is2) * E
    want = (F(2) * d2 * is2 / s) * E + base * d2 * (F(4) * s) * inv1 * inv1
    assert want.dtype == F
    got = _gradients(LOG, w, d, s)[:, 2] / w
    assert np.array_equal(got, want), (np.nonzero(got != want)[0][:5], int((got != want).sum()))


@pytest.mark.parametrize("model", [GMM, DOG, LOG], ids=["gmm", "dog", "log"])
def test_a_gradient_below_the_normal_numbers(model):
    """The derivative by the centre of components of weight 2^-130: subnormal, so that a factor of two left for later
    would cost its last bit."""
    rng = np.random.default_rng(2)
    n = 2000
    d, s = rng.uniform(0.1, 3.0, n).astype(F), rng.uniform(0.5, 1.5, n).astype(F)
    w = F(2.0) ** -130
    E1 = _gradients(GMM, F(0), d, s)[:, 0]
    d2, inv1 = d * d, F(1) / (F(2) * s * s + F(1e-8))
    if model == GMM:
        by_mu = E1 * F(2) * d * inv1
    elif model == DOG:
        E2 = E1 - _gradients(DOG, F(0), d, s)[:, 0]   # E1 - (E1 - E2): exact within a factor of two of each other
        inv2 = F(1) / (F(2) * s * s / F(4) + F(1e-8))
        by_mu = E1 * F(2) * d * inv1 - E2 * F(2) * d * inv2
    else:
        is2 = F(1) / (s * s)
        by_mu = F(2) * d * is2 * E1 + (F(1) - d2 * is2) * E1 * F(2) * d * inv1
    want = F(2) * (F(0.5) * (w * by_mu))   # residual 1/2, mean over one point: 2 / 1
    got = _gradients(model, w, d, s)[:, 1]
    exact = np.ones(n, bool) if model != DOG else (E2 >= E1 / 2)
    assert exact.sum() > 100 and np.abs(want[exact]).max() < np.finfo(F).tiny
    assert np.array_equal(got[exact], want[exact]), int((got != want)[exact].sum())
