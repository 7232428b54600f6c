"""The sub-pixel adjoint at the edges of its instances: every number of accumulators around the
sizes of its wave sums, with and without the lens light, an image that is no multiple of a tile,
|eps| on both sides of the derivative series, and a batch of one."""
import numpy as np
import pytest

import oracle
import synth
from helpers import assert_grad_close, oracle_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [None, 0.0195, 0.0205])
@pytest.mark.parametrize("epl,lens_light,nmax", [(False, False, -1), (True, True, -1), (True, False, 0),
                                                 (False, True, 1), (True, True, 6), (False, False, 6),
                                                 (True, True, 7), (False, True, 8), (True, True, 8)])
def test_gradient_matches_oracle(epl, lens_light, nmax, eps):
    import torch
    import paper_2202_07663_amd as G
    spec = synth.spec_custom(1, 3, epl, lens_light, nmax, K=5)
    spec.H, spec.W = 23, 29
    truth = synth.draw_truth(spec, 3)
    om = oracle_model(spec)
    obs = synth.add_noise(oracle.simulate(om, truth)[0], 3, spec.sigma_bkg, spec.t_exp)
    theta = synth.draw_particles(spec, truth, 9, seed=4)
    if eps is not None:
        i = spec.names.index("e1")
        ang = np.linspace(0.1, 6.0, len(theta))
        theta[:, i], theta[:, i + 1] = eps * np.cos(ang), eps * np.sin(ang)
    _, ref = oracle.loglik_grad(om, theta, obs)
    m = G.Model.from_spec(spec, obs)
    for th, rg in ((theta, ref), (theta[:1], ref[:1])):
        _, g = m.loglik_grad(torch.from_numpy(th).cuda())
        assert_grad_close(g.cpu().numpy(), rg, names=spec.names)
