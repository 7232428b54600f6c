"""The SIE's ray trace where its closed form would serve (|eps| >= 0.1): as exact as that form next
to the source's centre."""
import numpy as np
import pytest

import oracle
import synth
from helpers import oracle_model

pytestmark = pytest.mark.gpu


def _land(th, x, y):
    """Source position of the image position (x, y) for SIE + shear vectors, in 64 bits."""
    t_e, e1, e2, xc, yc, g1, g2 = th[:, :7].T.astype(np.float64)
    eps, z = e1 + 1j * e2, (x - xc) + 1j * (y - yc)
    w = z - eps * z.conj()
    s = np.sqrt(eps.conj() * w * w / abs(w) ** 2)
    a = t_e * np.sqrt(1 - abs(eps) ** 2) / abs(w) * w * np.arctan(s) / s
    return np.stack([x - a.real - g1 * x - g2 * y, y - a.imag - g2 * x + g1 * y], -1)


def _vectors(spec, n, seed):
    th = synth.draw_particles(spec, synth.draw_truth(spec, 5), n, seed=seed).astype(np.float32)
    rng = np.random.default_rng(seed)
    eps, a = np.exp(rng.uniform(np.log(0.1001), np.log(0.59), n)), rng.uniform(0, 2 * np.pi, n)
    th[:, 1], th[:, 2] = eps * np.cos(a), eps * np.sin(a)
    th[:, 9:11] = 0.0  # a round source
    return th, rng


def _spec(N):
    spec = synth.spec_custom(1, 1, False, False, -1, K=1)
    spec.H = spec.W = N
    return spec


def test_gradient_next_to_the_source_centre():
    """One ray lands 2e-6 arcsec from the centre of a steep profile (n = 8), whose gradient there
    dominates the derivatives in the centre's coordinates (~1 / r). They turn with the offset, so
    an error of the deflection of 1e-11 arcsec shows as 5e-6. Bound: an offset rounded to FP32 and
    some thirty FP32 operations, 30 x 6e-8."""
    import torch
    import paper_2202_07663_amd as G
    n, N = 512, 20
    spec = _spec(N)
    th, rng = _vectors(spec, n, 7)
    th[:, 7], th[:, 8], th[:, 13] = 0.25, 8.0, 10.0
    th[:, 9:11] = 1e-6  # the oracle has no derivative at 0
    i, j = rng.integers(2, N - 2, (2, n))
    pix = float(np.float32(spec.pix))
    at = _land(th, (j - (N - 1) / 2) * pix, (i - (N - 1) / 2) * pix)
    ph = rng.uniform(0, 2 * np.pi, n)
    th[:, 11:13] = at + 2e-6 * np.stack([np.cos(ph), np.sin(ph)], 1)
    obs = np.zeros((N, N), np.float32)
    _, ref = oracle.loglik_grad(oracle_model(spec), th.astype(np.float64), obs)
    m = G.Model.from_spec(spec, obs)
    g = m.loglik_grad(torch.from_numpy(th).cuda())[1].cpu().numpy()
    err = np.linalg.norm((g - ref)[:, 11:13], axis=1) / np.linalg.norm(ref[:, 11:13], axis=1)
    print("max", err.max(), "median", np.median(err), flush=True)
    assert err.max() <= 30 * 6e-8
