"""The work space is what its arrays take: two pixel arrays per vector besides the constants, the
partial sums and the kept source positions. The limit of the allocation-free call is where it was,
also for images of a few pixels, whose layout takes more than the limit counts."""
import ctypes

import numpy as np
import pytest

import oracle
import synth
from helpers import oracle_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,k,P", [(60, 2, 4096), (40, 1, 1000), (100, 2, 512)])
def test_work_space_holds_two_pixel_arrays(N, k, P):
    import paper_2202_07663_amd as G
    spec = synth.spec_custom(N, k, True, True, 2)
    m = G.Model.from_spec(spec, np.ones((N, N), np.float32))
    m.reserve(P)
    plan = m.plan(P)
    own = 8 * k * k * N * N + 2 * 4 * N * N  # source positions, pixel arrays
    # constants, band sums, and a row of 72 sums for each of up to 2048 + P tiles
    other = P * (4096 + 128) + (2048 + P) * 72 * 8 + 8 * 256
    for key in ("workspace_bytes", "workspace_reserved"):
        assert P * own < plan[key] <= P * own + other


@pytest.mark.parametrize("N,k,limit", [(1, 1, 27594), (6, 4, 14563), (6, 1, 26214)])
def test_allocation_free_limit_of_small_images(N, k, limit):
    import torch
    import paper_2202_07663_amd as G
    from paper_2202_07663_amd import _lib
    spec = synth.spec_custom(N, k, False, False, -1, K=3)
    truth = synth.draw_truth(spec, 3)
    om = oracle_model(spec)
    obs = synth.add_noise(oracle.simulate(om, truth)[0], 3, spec.sigma_bkg, spec.t_exp)
    m = G.Model.from_spec(spec, obs)
    P = m.plan(1)["noalloc_max_P"]
    assert P == limit
    th = torch.from_numpy(synth.draw_particles(spec, truth, P, seed=4)).cuda()
    ll, g = torch.empty(P, dtype=torch.float64, device="cuda"), torch.empty(P, m.d, device="cuda")
    rc = _lib.lib().gl_loglik_grad_noalloc(m._h, th.data_ptr(), P, ll.data_ptr(), g.data_ptr(),
                                           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    rl, rg = m.loglik_grad(th)
    np.testing.assert_array_equal(ll.cpu().numpy(), rl.cpu().numpy())
    np.testing.assert_array_equal(g.cpu().numpy(), rg.cpu().numpy())
