"""The sampler's own sub-pixel kernels (one leapfrog step's gradient and log p~) against the oracle:
every number of accumulators and shapelet order, with and without the lens light, |eps| on both
sides of the derivative series and of the SIE's closed form, and the lens centre on a sub-pixel. And
its fused per-chain kernel with four waves a chain against one."""
import numpy as np
import pytest

import oracle
import synth
from helpers import LOGL_RTOL, assert_grad_close, oracle_model
from sampler_gradient import sampler_gradient

pytestmark = pytest.mark.gpu


def _system(epl, lens_light, nmax, seed=3):
    import paper_2202_07663_amd as G
    spec = synth.spec_custom(1, 3, epl, lens_light, nmax, K=5)
    spec.H, spec.W = 23, 29
    truth = synth.draw_truth(spec, seed)
    om = oracle_model(spec)
    obs = synth.add_noise(oracle.simulate(om, truth)[0], seed, spec.sigma_bkg, spec.t_exp)
    return spec, truth, om, obs, G.Model.from_spec(spec, obs)


def _check(spec, om, obs, m, th):
    ref_l, ref = oracle.loglik_grad(om, th.astype(np.float64), obs)
    lp, g = sampler_gradient(m, th)
    assert_grad_close(g, ref, names=spec.names)
    assert (np.abs(lp - ref_l) / (np.abs(ref_l) + spec.H * spec.W / 2)).max() <= LOGL_RTOL


@pytest.mark.parametrize("eps", [None, 0.0195, 0.0205, 0.0995, 0.1005, 0.55])
@pytest.mark.parametrize("epl,lens_light,nmax", [(False, False, -1), (True, True, -1), (True, False, 0), (False, True, 1),
                                                 (True, False, 4), (False, True, 5), (True, True, 6), (False, False, 6),
                                                 (True, True, 7), (False, True, 8), (True, True, 8)])
def test_gradient_matches_oracle(epl, lens_light, nmax, eps):
    spec, truth, om, obs, m = _system(epl, lens_light, nmax)
    th = synth.draw_particles(spec, truth, 9, seed=4).astype(np.float32)
    if eps is not None:
        i, ang = spec.names.index("e1"), np.linspace(0.1, 6.0, len(th))
        th[:, i], th[:, i + 1] = eps * np.cos(ang), eps * np.sin(ang)
    _check(spec, om, obs, m, th)


@pytest.mark.parametrize("epl,nmax", [(False, -1), (True, -1), (True, 3), (False, 8)])
def test_lens_centre_on_a_sub_pixel(epl, nmax):
    """The centre on a sub-pixel centre, and off it by less than the floor of the radius."""
    spec, truth, om, obs, m = _system(epl, True, nmax)
    th = synth.draw_particles(spec, truth, 6, seed=5).astype(np.float32)
    i, pitch = spec.names.index("x"), float(np.float32(spec.pix)) / spec.k
    th[:, i], th[:, i + 1] = 0.0, 0.0  # odd image, odd k: a sub-pixel centre
    th[3:, i] += np.float32(2e-7)
    th[2, i] = pitch
    th[:, i - 2:i] = 0.2, 0.1
    _check(spec, om, obs, m, th)


@pytest.mark.parametrize("epl,nmax", [(True, 8), (False, -1)])
def test_chains_of_768_and_769_agree(epl, nmax):
    """Trajectories of about a unit of the mass matrix in each coordinate: positions, momenta
    and log p~ are the same bits with four waves a chain (up to 768) and with one."""
    import torch
    import paper_2202_07663_amd as G
    spec = synth.spec_custom(1, 2, epl, True, nmax, K=5)
    spec.H, spec.W = 12, 11
    truth = synth.draw_truth(spec, 3)
    om = oracle_model(spec)
    obs = synth.add_noise(oracle.simulate(om, truth)[0], 3, spec.sigma_bkg, spec.t_exp)
    m = G.Model.from_spec(spec, obs)
    rng = np.random.default_rng(2)
    priors = [{"family": 0, "mu": float(t), "sigma": 1.0, "lo": 0.0, "hi": 0.0} for t in truth]
    width = 1e-5 * np.maximum(np.abs(truth), 0.05)  # not above the posterior's
    z0 = truth + rng.normal(size=(769, m.d)) * width
    p0 = (rng.normal(size=z0.shape) / width).astype(np.float32)
    got = []
    for C in (768, 769):
        z, p = torch.from_numpy(z0[:C]).cuda(), torch.from_numpy(p0[:C]).cuda()
        h = G.HMC(m, C, 3, 0, 0, priors, step_size=0.3, z0=z, mass_chol=np.diag(width))
        got.append([t.cpu().numpy()[:768] for t in h.leapfrog(z, p, 3, 0.3)])
        h.close()
    ok = np.isfinite(got[0][2])
    print("finite", ok.mean(), "moved, in widths", np.median(np.abs(got[0][0] - z0[:768]) / width))
    assert ok.mean() > 0.9 and np.median(np.abs(got[0][0] - z0[:768]) / width) > 0.3
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
