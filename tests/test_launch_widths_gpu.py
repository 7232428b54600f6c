"""The per-particle kernels on both sides of the batch size where they go from four waves a
particle to one, and the fit step fused with the next one's prologue. Both forms do the same
arithmetic: log L, gradients and fit states are compared bit for bit; positions of a leapfrog
trajectory, rounded to FP32 at each step, to 4 units of that rounding."""
import numpy as np
import pytest

import oracle
import synth
from helpers import oracle_model

pytestmark = pytest.mark.gpu


def _model(epl, nmax):
    import paper_2202_07663_amd as G
    spec = synth.spec_custom(1, 2, epl, True, nmax, K=5)
    spec.H, spec.W = 12, 11
    truth = synth.draw_truth(spec, 3)
    obs = synth.add_noise(oracle.simulate(oracle_model(spec), truth)[0], 3, spec.sigma_bkg, spec.t_exp)
    return G, spec, truth, G.Model.from_spec(spec, obs)


@pytest.mark.parametrize("epl,nmax", [(True, 8), (False, -1)])
def test_batches_of_768_and_769_agree(epl, nmax):
    import torch
    G, spec, truth, m = _model(epl, nmax)
    th = torch.from_numpy(synth.draw_particles(spec, truth, 769, seed=5)).cuda()
    (la, ga), (lb, gb) = m.loglik_grad(th[:768]), m.loglik_grad(th)
    np.testing.assert_array_equal(la.cpu().numpy(), lb.cpu().numpy()[:768])
    np.testing.assert_array_equal(ga.cpu().numpy(), gb.cpu().numpy()[:768])
    # two leapfrog steps
    rng = np.random.default_rng(2)
    priors, chol = synth.fit_priors(spec), 1e-6 * np.eye(m.d)
    z0 = G.FitState(m, 769, 10, priors, seed=4).store()[0].cpu().numpy().astype(np.float64)
    p0 = (rng.normal(size=z0.shape) * 1e6).astype(np.float32)
    got = []
    for C in (768, 769):
        z, p = torch.from_numpy(z0[:C]).cuda(), torch.from_numpy(p0[:C]).cuda()
        h = G.HMC(m, C, 2, 0, 0, priors, step_size=0.1, z0=z, mass_chol=chol)
        got.append([t.cpu().numpy()[:768].astype(np.float64) for t in h.leapfrog(z, p, 2, 0.1)])
    (za, _, lpa), (zb, _, lpb) = got
    np.testing.assert_array_equal(np.isfinite(lpa), np.isfinite(lpb))
    assert np.all(np.abs(za - zb) <= 4 * np.spacing(np.abs(za).astype(np.float32)))


@pytest.mark.parametrize("P", [1, 7, 768, 769])
def test_fit_steps_in_one_call_equal_single_steps(P):
    G, spec, truth, m = _model(True, 3)
    priors = synth.fit_priors(spec)
    one, each = (G.FitState(m, P, 20, priors, seed=6) for _ in range(2))
    one.step(3)
    for _ in range(3):
        each.step(1)
    for a, b in zip(one.store(), each.store()):
        a, b = (np.asarray(t.cpu() if hasattr(t, "cpu") else t) for t in (a, b))
        np.testing.assert_array_equal(a, b)
