"""The likelihood sums do not depend on the launch: a served system's log posterior and chi^2 are
the same bits alone and in one launch with others of its kernel configuration (whose PSF pass then
takes the block size of them all), and so is a vector's log L at any batch of the matrix-core and
the whole-image VALU pass."""
import numpy as np
import pytest

import oracle
import synth
from helpers import oracle_model

pytestmark = pytest.mark.gpu


def _system(H, W, K, seed, nmax=-1, k=1):
    spec = synth.spec_custom(1, k, True, False, nmax, K=K)
    spec.H, spec.W = H, W
    truth = synth.draw_truth(spec, seed)
    om = oracle_model(spec)
    return spec, truth, synth.add_noise(oracle.simulate(om, truth)[0], seed, spec.sigma_bkg, spec.t_exp)


@pytest.mark.parametrize("systems", [
    # (H, W, K, P): matrix cores, 512 threads alone and 256 together
    [(60, 60, 21, 512), (60, 60, 21, 512), (56, 60, 21, 700)],
    # banded, bands of different sizes and block sizes; one of them at two lanes a strip
    [(32, 32, 21, 64), (40, 40, 21, 300), (57, 44, 21, 130)],
    # the whole-image VALU pass alone; the banded kernels beside a banded system
    [(48, 48, 25, 512), (64, 64, 25, 100), (7, 30, 25, 40)]])
def test_served_sums_do_not_depend_on_partners(systems):
    import paper_2202_07663_amd as G
    # three requests of each system: nine sums that could come out differently
    reqs = [(_system(H, W, K, 40 + i), P, s) for i, (H, W, K, P) in enumerate(systems) for s in range(3)]

    def submit(srv, req):
        (spec, _, obs), P, seed = req
        return srv.submit(spec, obs, P, 2, synth.fit_priors(spec), seed=seed)

    alone = []
    srv = G.Server(max_systems=1)
    for req in reqs:
        alone.append(srv.wait(submit(srv, req)))
    srv.close()
    # a first system fills the server until all the others wait, which then start in one tick
    srv = G.Server(max_systems=16, fill_subpixels=4e7)
    big = _system(100, 100, 21, 50, k=2)
    first = srv.submit(big[0], big[2], 1100, 200, synth.fit_priors(big[0]), seed=1)
    tickets = [submit(srv, r) for r in reqs]
    srv.wait(first)
    together = [srv.wait(t) for t in tickets]
    srv.close()
    for a, b in zip(alone, together):
        assert a["status"] == 0 and b["status"] == 0
        assert (a["best"], a["logpost_best"], a["chi2nu"]) == (b["best"], b["logpost_best"], b["chi2nu"])
        np.testing.assert_array_equal(a["theta_best"], b["theta_best"])


@pytest.mark.parametrize("H,W,K,path", [(60, 60, 21, "mfma"), (33, 45, 21, "mfma"), (100, 100, 21, "mfma"),
                                        (80, 70, 9, "mfma"), (40, 41, 25, "valu")])
def test_log_likelihood_same_at_any_batch(H, W, K, path):
    import torch
    import paper_2202_07663_amd as G
    spec, truth, obs = _system(H, W, K, 60)
    m = G.Model.from_spec(spec, obs)
    th = torch.from_numpy(synth.draw_particles(spec, truth, 1100, seed=61)).cuda()
    ref = m.loglik(th).cpu().numpy()
    for P in (512, 513, 777, 1024):
        assert m.plan(P)["psf_path"] == path
        np.testing.assert_array_equal(m.loglik(th[:P]).cpu().numpy(), ref[:P])
        np.testing.assert_array_equal(m.loglik_grad(th[:P])[0].cpu().numpy(), ref[:P])
