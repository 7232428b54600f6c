"""Errors of gradient components that are differences of sums: the batched calls' against the
sampler's, whose kernels take every component sub-pixel by sub-pixel. 2304 vectors have one tile
each, whose lanes add some 57 sub-pixels in FP32. Compared: the geometric means of |g - g_64| / |g_64|
over a few hundred vectors and components, whose ratio scatters by about 0.05."""
import numpy as np
import pytest

import oracle
import synth
from helpers import oracle_model
from sampler_gradient import sampler_gradient

pytestmark = pytest.mark.gpu


def _ratio(cases, names, n=64, P=2304):
    """Geometric mean of the batched calls' relative errors over that of the sampler's."""
    import torch
    import paper_2202_07663_amd as G
    logs = []
    for k, (epl, nmax, eps) in enumerate(cases):
        spec = synth.spec_custom(60, 2, epl, True, nmax)
        rng = np.random.default_rng(k)
        i, (a0, *a) = spec.names.index("e1"), rng.uniform(0, 2 * np.pi, n + 1)
        truth = synth.draw_truth(spec, 30 + k)
        truth[i], truth[i + 1] = eps * np.cos(a0), eps * np.sin(a0)
        om = oracle_model(spec)
        obs = synth.add_noise(oracle.simulate(om, truth)[0], k, spec.sigma_bkg, spec.t_exp)
        th = synth.draw_particles(spec, truth, n, seed=k).astype(np.float32)
        th[:, i], th[:, i + 1] = eps * np.cos(a), eps * np.sin(a)
        _, ref = oracle.loglik_grad(om, th.astype(np.float64), obs)
        m = G.Model.from_spec(spec, obs)
        full = np.resize(th, (P, th.shape[1]))
        g = m.loglik_grad(torch.from_numpy(full).cuda())[1].cpu().numpy()[:n]
        s = sampler_gradient(m, full)[1][:n]
        j = [spec.names.index(x) for x in names]
        ea, eb = (np.abs(x[:, j] - ref[:, j]) / np.abs(ref[:, j]) + 1e-10 for x in (s, g))
        logs.append(np.log(eb / ea).ravel())
        print(epl, nmax, eps, "sampler", np.exp(np.log(ea).mean()), "ratio", np.exp(logs[-1].mean()), flush=True)
    return float(np.exp(np.concatenate(logs).mean()))


def test_mass_ellipticity():
    cases = [(epl, nmax, eps) for epl, nmax in ((True, -1), (False, -1), (True, 3)) for eps in (0.0205, 0.05, 0.1)]
    r = _ratio(cases, ["e1", "e2"])
    print("ratio", r)
    assert r <= 1.2


def test_sersic_index():
    cases = [(epl, nmax, 0.1) for epl, nmax in ((True, -1), (False, -1), (True, 3), (False, 2))]
    r = _ratio(cases, ["l_n", "s_n"], n=192)
    print("ratio", r)
    assert r <= 1.1
