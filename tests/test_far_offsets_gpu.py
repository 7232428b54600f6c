"""Source offsets of tens of thousands of shapelet scales, where the Gaussian is zero and the
polynomials are near the end of the FP32 range: wherever log L is finite, so is its gradient."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nmax,most", [(8, 6.3e4), (7, 3.0e5), (6, 2.5e6), (5, 4.9e7), (3, 6.5e12)])
def test_gradient_is_finite_where_log_l_is(nmax, most):
    import torch
    import paper_2202_07663_amd as G
    # no lensing to speak of: the offsets from the source are those in the image, +-0.3575 arcsec
    spec = synth.spec_custom(12, 1, False, False, nmax, K=1)
    i = {n: k for k, n in enumerate(spec.names)}
    th = np.zeros((5, spec.d), np.float32)
    th[:, i["theta_E"]] = 1e-4
    th[:, i["e1"]], th[:, i["x"]] = 0.05, 3.0
    th[:, i["s_R"]], th[:, i["s_n"]], th[:, i["s_e1"]], th[:, i["s_I"]] = 0.2, 1.0, 0.1, 5.0
    # the largest |u|, |v| as shares of `most`, where g_n of the forward pass is last finite
    th[:, i["beta"]] = 0.36 / (most * np.array([0.5, 0.7, 0.8, 0.9, 0.98]))
    th[:, i["beta"] + 1:] = 1e-7 * th[:, i["beta"], None]
    m = G.Model.from_spec(spec, np.ones((12, 12), np.float32))
    t = torch.from_numpy(th).cuda()
    ll = m.loglik(t).cpu().numpy()
    assert np.all(np.isfinite(ll))
    lg, g = m.loglik_grad(t)
    np.testing.assert_allclose(lg.cpu().numpy(), ll, rtol=1e-12)
    g = g.cpu().numpy()
    assert np.all(g[:, i["beta"]:] == 0.0)  # no sub-pixel sees the shapelets
    th[:, i["beta"]] = 0.01  # nor at a scale of its own but for the sub-pixels near the centre
    th[:, i["beta"] + 1:] = 0.0
    _, ref = m.loglik_grad(torch.from_numpy(th).cuda())
    k = i["beta"]
    np.testing.assert_allclose(g[:, :k], ref.cpu().numpy()[:, :k], rtol=1e-4, atol=1e-3)
