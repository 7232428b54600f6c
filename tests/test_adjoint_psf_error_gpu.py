"""Error of the PSF pass's adjoint half on matrix cores (batches below 512 vectors) against that of
the vector ALUs, which the sampler's launches keep. With every amplitude zero and unit noise the
pixel seeds are the observed image itself, exactly; a lens light far smaller than a pixel then has
one pixel's correlation of seed and PSF, times a constant, as its derivative in I."""
import numpy as np
import pytest

import synth
from sampler_gradient import sampler_gradient

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,K,P", [(60, 60, 21, 130), (30, 112, 21, 138), (60, 60, 21, 400), (57, 83, 15, 300), (96, 96, 17, 400)])
def test_not_above_the_vector_sums(H, W, K, P):
    import torch
    import paper_2202_07663_amd as G
    rng = np.random.default_rng(K + P)
    errs = {"matrix": [], "vector": []}
    for psf in (synth.moffat_psf(K, 0.15, 2.5), synth.asymmetric_psf(K, seed=K)):
        for obs in rng.normal(size=(2, H, W)).astype(np.float32):
            m = G.Model(H, W, synth.PIX, 1, "sie", False, True, -1, psf, obs, 1.0, 1e30)  # no shot noise
            assert m.plan(P)["psf_path"] == "banded"
            i, j = rng.integers(0, H, P), rng.integers(0, W, P)
            pix = float(np.float32(synth.PIX))
            th = np.zeros((P, m.d), np.float32)
            th[:, :2] = 1.0, 0.1
            th[:, 5:7] = 0.01, 0.5  # lens light: R, n
            th[:, 9], th[:, 10] = (j - (W - 1) / 2) * pix, (i - (H - 1) / 2) * pix
            th[:, 12:14] = 0.2, 1.0
            pad = np.pad(obs.astype(np.float64), (K - 1) // 2)
            ref = np.array([(pad[a:a + K, b:b + K] * psf.astype(np.float64)).sum() for a, b in zip(i, j)])
            g = {"matrix": m.loglik_grad(torch.from_numpy(th).cuda())[1].cpu().numpy(), "vector": sampler_gradient(m, th)[1]}
            for k, x in g.items():
                x = x[:, 11].astype(np.float64)
                scale = (x * ref).sum() / (ref ** 2).sum()  # the profile's value on its pixel
                errs[k].append((x / scale - ref) / np.sqrt((ref ** 2).mean()))
    rms = {k: float(np.sqrt(np.mean(np.square(v)))) for k, v in errs.items()}
    print(H, W, K, P, rms, "ratio", rms["matrix"] / rms["vector"], flush=True)
    assert rms["matrix"] <= rms["vector"]
