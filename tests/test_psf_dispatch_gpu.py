"""The edges of the PSF pass's dispatch, and the ray trace over its ellipticities, against the
oracle.

Tolerances: gradients as everywhere (helpers); log L is a sum of H W pixel terms of order one, so
its error is taken relative to |log L| + H W / 2; model images 2e-5 of their largest pixel.
"""
import numpy as np
import pytest

import oracle
import synth
from helpers import GRAD_RTOL, LOGL_RTOL, assert_grad_close, oracle_model

pytestmark = pytest.mark.gpu


def _check(spec, P, seed, strong=False):
    import torch
    import paper_2202_07663_amd as G
    truth = synth.draw_truth(spec, seed)
    om = oracle_model(spec)
    obs = synth.add_noise(oracle.simulate(om, truth)[0], seed, spec.sigma_bkg, spec.t_exp)
    theta = synth.draw_particles(spec, truth, P, seed=seed + 1)
    if strong:
        i, ang, r = spec.names.index("e1"), np.linspace(0.1, 6.0, P), np.linspace(1e-3, 0.6, P)
        theta[:, i], theta[:, i + 1] = r * np.cos(ang), r * np.sin(ang)
    m = G.Model.from_spec(spec, obs)
    th = torch.from_numpy(theta).cuda()
    ll, g = (t.cpu().numpy() for t in m.loglik_grad(th))
    img = m.simulate(th).cpu().numpy()
    idx = np.unique([0, P // 3, P // 2, P - 1])
    ll_ref, g_ref = oracle.loglik_grad(om, theta[idx], obs)
    err = np.abs(ll[idx] - ll_ref) / (np.abs(ll_ref) + spec.H * spec.W / 2)
    print(spec.H, spec.W, P, m.plan(P), "logl", err.max(), flush=True)
    assert err.max() <= LOGL_RTOL
    assert_grad_close(g[idx], g_ref, rtol=GRAD_RTOL, names=spec.names)
    ref = oracle.simulate(om, theta[idx])
    assert (np.abs(img[idx] - ref) / np.abs(ref).max(axis=(1, 2), keepdims=True)).max() < 2e-5


@pytest.mark.parametrize("H,W,K,P", [
    # matrix cores: 256, 512 and 1024 threads by LDS, batch and tiles
    (60, 60, 21, 512), (60, 60, 21, 1025), (33, 45, 21, 513), (100, 100, 21, 515), (16, 12, 21, 2049),
    # banded: the adjoint half on the VALU and, from 2e8 products, on matrix cores
    (33, 41, 21, 335), (33, 41, 21, 336), (61, 47, 19, 511), (128, 128, 21, 511),
    # banded: heights, widths and PSFs at the ends of their ranges; split columns; one vector
    (100, 3, 31, 1), (9, 128, 31, 5), (127, 40, 25, 130), (65, 33, 1, 3), (128, 128, 31, 7), (57, 60, 3, 70)])
def test_psf_pass_edges(H, W, K, P):
    spec = synth.spec_custom(1, 1, True, True, 1, K=K)
    spec.H, spec.W, spec.psf = H, W, synth.asymmetric_psf(K, seed=K) if K > 1 else spec.psf
    _check(spec, P, 20 + K)


@pytest.mark.parametrize("epl", [False, True])
@pytest.mark.parametrize("P", [9, 520])
def test_ray_trace_up_to_strong_ellipticity(epl, P):
    spec = synth.spec_custom(1, 2, epl, True, 3, K=5)
    spec.H, spec.W = 24, 21
    _check(spec, P, 7, strong=True)
