"""The work that users of this framework have it do, as measurable cases.

Every case is one pass through the public entry points on one lens system: images of the
model, log L, log L with its gradient (directly and through autograd), one Adam step of a
multi-start fit, one iteration of the variational fit, one short leapfrog trajectory. The
systems are those of this repository's workloads (40 x 40 SIE, 60 x 60 EPL + shapelets,
80 x 80 EPL, the 100 x 100 n_max = 8 system of the serving stream) and a ragged one.

`exact` is the same model written in plain torch in 64 bits (gradients by autograd).
"""
import math

import numpy as np
import torch

import paper_2202_07663_amd as G

PIX = 0.065  # arcsec per pixel

# per system: image, supersampling, PSF size, components, noise
SIE40 = dict(H=40, W=40, k=1, K=11, epl=False, shear=True, lens_light=False, nmax=-1,
             sigma_bkg=0.1, t_exp=1000.0)
EPL60 = dict(H=60, W=60, k=2, K=21, epl=True, shear=True, lens_light=True, nmax=6,
             sigma_bkg=0.1, t_exp=1000.0)
EPL80 = dict(H=80, W=80, k=2, K=21, epl=True, shear=True, lens_light=True, nmax=-1,
             sigma_bkg=0.2, t_exp=100.0)
EPL100 = dict(H=100, W=100, k=2, K=21, epl=True, shear=True, lens_light=True, nmax=8,
              sigma_bkg=0.1, t_exp=1000.0)
RAGGED = dict(H=53, W=37, k=3, K=9, epl=False, shear=True, lens_light=True, nmax=3,
              sigma_bkg=0.1, t_exp=1000.0)


def listed():
    def case(name, op, system, P):
        return dict(name=name, op=op, P=P, **system)

    return [
        # the model image of one parameter vector, looked at interactively: latency
        case("image_sie40_1", "image", SIE40, 1),
        # one vector inside a user's own torch optimiser: forward and backward
        case("autograd_epl60_1", "autograd", EPL60, 1),
        # a leapfrog step's gradient for 64 chains, called from a user's own sampler
        case("grad_epl60_64", "grad", EPL60, 64),
        # 64 chains of the library's sampler, three leapfrog steps
        case("leapfrog_epl60_64", "leapfrog", EPL60, 64),
        # the gradient of 300 starts, the size of the paper's MAP stage
        case("grad_epl80_300", "grad", EPL80, 300),
        # one iteration of the variational fit with 500 samples, the paper's VI stage
        case("vi_epl80_500", "vi", EPL80, 500),
        # posterior-predictive images of 512 draws
        case("image_epl80_512", "image", EPL80, 512),
        # one Adam step of 512 starts, the throughput-budgeted fit
        case("fit_epl60_512", "fit", EPL60, 512),
        # an odd system and batch: H != W, k = 3, a 9 x 9 PSF, SIE + lens light
        case("grad_ragged_777", "grad", RAGGED, 777),
        # log L alone of a full batch: ranking starts, importance weights
        case("loglik_epl60_4096", "loglik", EPL60, 4096),
        # log L and its gradient of a full batch: the MAP stage at 4096 starts
        case("grad_epl60_4096", "grad", EPL60, 4096),
        # the serving stream's largest system
        case("grad_epl100_2048", "grad", EPL100, 2048),
    ]


MOST_SUBPIXELS = 2048 * 100 * 100 * 4  # of the largest listed case


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)) - 0.5 / hi)))))


def draw(rng):
    op = rng.choice(["image", "loglik", "grad", "grad", "grad", "autograd", "fit", "vi", "leapfrog"])
    H = _log_int(rng, 24, 112)
    W = H if rng.random() < 0.5 else _log_int(rng, 24, 112)
    k = rng.choice([1, 2, 2, 2, 3, 4])
    lo, hi = {"image": (1, 2048), "loglik": (1, 4096), "grad": (1, 4096), "autograd": (1, 512),
              "fit": (64, 4096), "vi": (100, 2000), "leapfrog": (8, 512)}[op]
    P = _log_int(rng, lo, hi)
    P = max(1, min(P, MOST_SUBPIXELS // (H * W * k * k)))
    noise = rng.choice([(0.1, 1000.0), (0.2, 100.0)])
    c = dict(op=op, P=P, H=H, W=W, k=k, K=rng.choice([5, 9, 11, 15, 21, 21, 21, 25, 31]),
             epl=rng.random() < 0.7, shear=rng.random() < 0.9, lens_light=rng.random() < 0.7,
             nmax=rng.choice([-1, -1, 2, 3, 4, 5, 6, 7, 8]), sigma_bkg=noise[0], t_exp=noise[1])
    over = work(c)["flops"] / max(work(x)["flops"] for x in listed())
    return dict(c, P=max(1, int(P / over))) if over > 1 else c


# ------------------------------------------------------------------------------------------
# Inputs
# ------------------------------------------------------------------------------------------
def _n_params(c):
    return len(_priors(c))


def _priors(c):
    """Priors of the fit, one per parameter in the library's order."""
    def N(mu, s):
        return {"family": 0, "mu": mu, "sigma": s, "lo": 0.0, "hi": 0.0}

    def LN(m, s):
        return {"family": 1, "mu": math.log(m), "sigma": s, "lo": 0.0, "hi": 0.0}

    def TN(mu, s, lo, hi):
        return {"family": 2, "mu": mu, "sigma": s, "lo": lo, "hi": hi}

    def U(lo, hi):
        return {"family": 3, "mu": 0.0, "sigma": 1.0, "lo": lo, "hi": hi}

    p = [LN(1.25, 0.4)] + ([TN(2.0, 0.5, 1.0, 3.0)] if c["epl"] else [])
    p += [N(0, 0.2), N(0, 0.2), N(0, 0.1), N(0, 0.1)]
    if c["shear"]:
        p += [N(0, 0.1), N(0, 0.1)]
    if c["lens_light"]:
        p += [LN(1.0, 0.5), U(0.5, 8.0), TN(0, 0.1, -0.15, 0.15), TN(0, 0.1, -0.15, 0.15),
              N(0, 0.02), N(0, 0.02), LN(300.0, 0.5)]
    p += [LN(0.25, 0.5), U(0.5, 8.0), TN(0, 0.3, -0.5, 0.5), TN(0, 0.3, -0.5, 0.5),
          N(0, 0.5), N(0, 0.5), LN(12.0, 0.9)]
    if c["nmax"] >= 0:
        p += [U(0.02, 0.4)] + [N(0, 2.0)] * ((c["nmax"] + 1) * (c["nmax"] + 2) // 2)
    return p


def _draw_theta(c, rng, n, broad):
    """Parameter vectors of the systems' distribution (broad = 1: truths) or of one twice as
    wide (broad = 2: where starts come from)."""
    def uni(lo, hi):
        m, h = 0.5 * (lo + hi), 0.5 * (hi - lo) * broad
        return rng.uniform(max(m - h, 0.5 * lo), m + h, n)

    def nor(s, most=None):
        x = rng.normal(0.0, s * broad, n)
        return x if most is None else np.clip(x, -most, most)

    cols = [uni(1.0, 1.5)] + ([uni(1.8, 2.2)] if c["epl"] else [])
    cols += [nor(0.1, 0.3), nor(0.1, 0.3), nor(0.05), nor(0.05)]
    if c["shear"]:
        cols += [nor(0.05), nor(0.05)]
    if c["lens_light"]:
        cols += [uni(0.5, 1.5), uni(2.0, 6.0), nor(0.05, 0.14), nor(0.05, 0.14), nor(0.01),
                 nor(0.01), np.exp(rng.normal(math.log(300.0), 0.3 * broad, n))]
    cols += [uni(0.1, 0.4), uni(1.0, 4.0), nor(0.15, 0.45), nor(0.15, 0.45), nor(0.1), nor(0.1),
             uni(5.0, 20.0)]
    if c["nmax"] >= 0:
        cols += [uni(0.05, 0.2)]
        cols += [nor(1.0) for _ in range((c["nmax"] + 1) * (c["nmax"] + 2) // 2)]
    return np.stack(cols, 1)


def _to_z(theta, priors):
    """Unconstrained coordinates of parameter vectors."""
    z = np.array(theta, np.float64)
    for j, p in enumerate(priors):
        if p["family"] == 1:
            z[:, j] = np.log(z[:, j])
        elif p["family"] >= 2:
            u = np.clip((z[:, j] - p["lo"]) / (p["hi"] - p["lo"]), 1e-3, 1 - 1e-3)
            z[:, j] = np.log(u) - np.log1p(-u)
    return z


def _psf(K):
    """Moffat kernel, FWHM 0.15 arcsec, beta 2.5, unit sum."""
    i = (np.arange(K) - (K - 1) / 2) * PIX
    a = 0.15 / (2.0 * math.sqrt(2.0 ** (1.0 / 2.5) - 1.0))
    p = (1.0 + (i[:, None] ** 2 + i[None, :] ** 2) / a ** 2) ** (-2.5)
    return (p / p.sum()).astype(np.float32)


def _inputs(c, seed):
    """What a pass reads, as numpy arrays made from the seed: the observed image (the truth's,
    with its noise), and the parameter vectors or the state of the fit or sampler."""
    rng = np.random.default_rng(seed)
    truth = _draw_theta(c, rng, 1, 1.0)
    got = {"psf": _psf(c["K"]), "obs": None}
    if c["op"] != "image":
        clean = _images(c, torch.from_numpy(truth.astype(np.float32)).double(), "cpu")[0].numpy()
        shot = rng.poisson(np.maximum(clean, 0.0) * c["t_exp"]) / c["t_exp"]
        got["obs"] = (shot + rng.normal(0.0, c["sigma_bkg"], clean.shape)).astype(np.float32)
    P, priors = c["P"], _priors(c)
    d = len(priors)
    if c["op"] in ("image", "loglik", "grad", "autograd"):
        # half the vectors near the truth, half from the broad distribution
        near = P - P // 2
        scale = 0.01 * np.maximum(np.abs(truth), np.array([p["sigma"] if p["family"] == 0 else 0.1 for p in priors]))
        th = truth + rng.normal(size=(near, d)) * scale
        th = np.concatenate([th, _draw_theta(c, rng, P - near, 2.0)])
        got["theta"] = th.astype(np.float32)
    elif c["op"] == "fit":  # starts from the broad distribution, moments at zero
        got["z"] = _to_z(_draw_theta(c, rng, P, 2.0), priors).astype(np.float32)
    else:  # a surrogate of the posterior about the truth: its mean and lower factor
        got["mu"] = _to_z(truth, priors)[0]
        low = np.tril(rng.normal(0.0, 1e-4, (d, d)), -1)
        got["chol"] = low + np.diag(1e-3 * np.exp(rng.normal(0.0, 0.3, d)))
        if c["op"] == "leapfrog":
            n = rng.normal(size=(2, P, d))
            chol = got["chol"].astype(np.float32).astype(np.float64)
            got["z"] = got["mu"] + n[0] @ chol.T
            got["p"] = np.linalg.solve(chol.T, n[1].T).T.astype(np.float32)
    return got


LEAPFROG_STEPS, LEAPFROG_EPS = 3, 1e-2
FIT_STEPS_IN_ALL = 300
VI_RATE = 1e-3


def prepare(case, seed):
    c = case
    i = _inputs(c, seed)
    m = G.Model(c["H"], c["W"], PIX, c["k"], "epl" if c["epl"] else "sie", c["shear"],
                c["lens_light"], c["nmax"], i["psf"], i["obs"], c["sigma_bkg"], c["t_exp"])
    s = {"op": c["op"], "model": m}
    op = c["op"]
    if op in ("image", "loglik", "grad", "autograd"):
        s["theta"] = torch.from_numpy(i["theta"]).cuda().requires_grad_(op == "autograd")
    elif op == "fit":
        s["fit"] = G.FitState(m, c["P"], FIT_STEPS_IN_ALL, _priors(c), seed=seed)
        s["z"] = torch.from_numpy(i["z"]).cuda()
        s["m"], s["v"] = torch.zeros_like(s["z"]), torch.zeros_like(s["z"])
    elif op == "vi":
        s["vi"] = G.VI(m, c["P"], 1000, _priors(c), i["mu"], lr_max=VI_RATE, lr_warmup=0, seed=seed)
        s["x"] = torch.from_numpy(_pack(i["mu"], i["chol"])).cuda()
        s["m"], s["v"] = torch.zeros_like(s["x"]), torch.zeros_like(s["x"])
    else:
        s["hmc"] = G.HMC(m, c["P"], LEAPFROG_STEPS, 250, 0, _priors(c), step_size=LEAPFROG_EPS,
                         seed=seed, z0=torch.from_numpy(i["z"]).cuda(), mass_chol=i["chol"])
        s["z"], s["p"] = torch.from_numpy(i["z"]).cuda(), torch.from_numpy(i["p"]).cuda()
    return s


def run(state):
    s, op = state, state["op"]
    if op == "image":
        return s["model"].simulate(s["theta"])
    if op == "loglik":
        return s["model"].loglik(s["theta"])
    if op == "grad":
        return s["model"].loglik_grad(s["theta"])
    if op == "autograd":
        logl = G.LogLik.apply(s["theta"], s["model"])
        (g,) = torch.autograd.grad(logl.sum(), s["theta"])
        return logl.detach(), g
    if op == "fit":  # one step from the given state: z, both moments, the step count
        s["fit"].load(s["z"], s["m"], s["v"], 0)
        s["fit"].step(1)
        return s["fit"].store()
    if op == "vi":  # one iteration from the given surrogate: mean, factor, covariance
        s["vi"].set_state(s["x"], s["m"], s["v"], 0)
        s["vi"].step(1)
        return s["vi"].get()
    return s["hmc"].leapfrog(s["z"], s["p"], LEAPFROG_STEPS, LEAPFROG_EPS)


def work(case):
    c = case
    px, sub, d, P = c["H"] * c["W"], c["H"] * c["W"] * c["k"] ** 2, _n_params(c), c["P"]
    grad = c["op"] not in ("image", "loglik")
    M = (c["nmax"] + 1) * (c["nmax"] + 2) // 2 if c["nmax"] >= 0 else 0
    # per sub-pixel: deflection (its series at about 12 terms, two fused multiply-adds each),
    # light profiles, shapelet sum; backward: the Jacobian of each and its accumulation
    fwd = 52 + (48 if c["epl"] else 20) + 18 * (1 + c["lens_light"]) + (3 * M + 4 * c["nmax"] + 8 if M else 0)
    bwd = 142 + (48 if c["epl"] else 0) + 52 * (1 + c["lens_light"]) + (9 * M + 8 * c["nmax"] + 16 if M else 0)
    flops = sub * (fwd + bwd * grad) + px * (2 * c["K"] ** 2 * (1 + grad) + 20)
    evals = P * (LEAPFROG_STEPS + 1 if c["op"] == "leapfrog" else 1)
    fixed = 4 * (px * (c["op"] != "image") + c["K"] ** 2)
    moved = {"image": 4 * (d + px), "loglik": 4 * d + 8, "grad": 8 * d + 8, "autograd": 8 * d + 8,
             "fit": 24 * d, "vi": 0, "leapfrog": 24 * d + 8}[c["op"]] * P
    if c["op"] == "vi":
        moved = 8 * (d + d * (d + 1) // 2) * 3 + 8 * (d + 2 * d * d)
    return {"bytes": fixed + moved, "flops": evals * flops}


# ------------------------------------------------------------------------------------------
# The model in 64 bits
# ------------------------------------------------------------------------------------------
class _Series(torch.autograd.Function):
    """S_t(X) = sum_n c_n(t) (-X)^n, c_n / c_(n-1) = (2n - 2 + t) / (2n + 2 - t), for one t per
    row of X, with its derivatives."""

    @staticmethod
    def forward(ctx, X, t, terms):
        n = torch.arange(1, terms, dtype=t.dtype, device=t.device)
        a, b = 2 * n - 2 + t[:, None], 2 * n + 2 - t[:, None]
        one = torch.ones_like(t)[:, None]
        cn = torch.cat([one, torch.cumprod(a / b, 1)], 1)
        dcn = cn * torch.cat([0 * one, torch.cumsum(1 / a + 1 / b, 1)], 1)
        S, SX, St = torch.zeros_like(X), torch.zeros_like(X), torch.zeros_like(X)
        for q in range(terms - 1, -1, -1):
            SX = -X * SX - S
            S = -X * S + cn[:, q, None]
            St = -X * St + dcn[:, q, None]
        ctx.save_for_backward(SX, St)
        return S

    @staticmethod
    def backward(ctx, g):
        SX, St = ctx.saved_tensors
        return g * SX.conj(), (g.conj() * St).real.sum(1), None


class _Convolve(torch.autograd.Function):
    """img [P, H, W] convolved with psf [K, K] (zero outside)."""

    @staticmethod
    def forward(ctx, img, psf):
        ctx.psf = psf
        return _correlate(img, np.flip(psf, (0, 1)))

    @staticmethod
    def backward(ctx, g):
        return _correlate(g, ctx.psf), None


def _correlate(img, taps):
    K, (H, W) = taps.shape[0], img.shape[1:]
    c = (K - 1) // 2
    pad = torch.nn.functional.pad(img, (c, c, c, c))
    out = torch.zeros_like(img)
    for a in range(K):
        for b in range(K):
            out.add_(pad[:, a:a + H, b:b + W], alpha=float(taps[a, b]))
    return out


def _clamped(e1, e2, most):
    r = torch.sqrt(e1 * e1 + e2 * e2).clamp_min(1e-300)
    s = torch.clamp(most / r, max=1.0)
    return e1 * s, e2 * s


def _sersic(p, x, y):
    """p: columns R, n, e1, e2, x, y, I."""
    R, n, e1, e2, xc, yc, i0 = (q[:, None] for q in p)
    e1, e2 = _clamped(e1, e2, 0.9)
    dx, dy, ee = x - xc, y - yc, e1 * e1 + e2 * e2
    r2 = ((1 + ee - 2 * e1) * dx * dx - 4 * e2 * dx * dy + (1 + ee + 2 * e1) * dy * dy) / (1 - ee)
    r2 = r2.clamp_min(1e-12)
    return i0 * torch.exp(-(1.9992 * n - 0.3271) * ((torch.sqrt(r2) / R) ** (1 / n) - 1))


def _shapelets(c, p, dx, dy):
    """p: columns beta, coefficients by order n = n1 + n2 and, within it, n2 = 0 .. n."""
    beta, N = p[0][:, None], c["nmax"]
    C = torch.zeros(len(p[0]), N + 1, N + 1, dtype=dx.dtype, device=dx.device)
    q, at, values = 1, [], []
    for n in range(N + 1):
        for n2 in range(n + 1):
            at.append((n - n2) * (N + 1) + n2)
            values.append(p[q])
            q += 1
    C = C.reshape(len(beta), -1).index_copy(1, torch.tensor(at, device=dx.device), torch.stack(values, 1))
    C = C.reshape(-1, N + 1, N + 1)

    def phi(u):  # Hermite functions
        h = [math.pi ** -0.25 * torch.exp(-0.5 * u * u)]
        for n in range(N):
            nxt = math.sqrt(2.0 / (n + 1)) * u * h[n]
            h.append(nxt - math.sqrt(n / (n + 1)) * h[n - 1] if n else nxt)
        return torch.stack(h, 2)

    return (torch.bmm(phi(dx / beta), C) * phi(dy / beta)).sum(2) / beta


def _images(c, theta, device):
    """Model images [P, H, W] of theta [P, d] (float64)."""
    H, W, k = c["H"], c["W"], c["k"]
    pix = float(np.float32(PIX))

    def grid(n):
        return ((torch.arange(n * k, dtype=torch.float64, device=device) + 0.5) / k - 0.5 - 0.5 * (n - 1)) * pix

    y, x = torch.meshgrid(grid(H), grid(W), indexing="ij")
    x, y = x.reshape(1, -1), y.reshape(1, -1)
    col = list(theta.unbind(1))
    th_e = col.pop(0)
    t = col.pop(0) - 1 if c["epl"] else torch.ones_like(th_e)
    e1, e2 = _clamped(col.pop(0), col.pop(0), 0.6)
    xc, yc = col.pop(0), col.pop(0)
    g1, g2 = (col.pop(0), col.pop(0)) if c["shear"] else (torch.zeros_like(xc), torch.zeros_like(xc))
    top = max(float(torch.sqrt(e1 * e1 + e2 * e2).detach().max()), 1e-3)
    terms = 2 + math.ceil(math.log(1e-17) / math.log(top))
    eps, z = torch.complex(e1, e2)[:, None], torch.complex(x - xc[:, None], y - yc[:, None])
    w = z - eps * z.conj()
    w2 = (w.real ** 2 + w.imag ** 2).clamp_min(1e-12)
    S = _Series.apply(eps.conj() * w * w / w2, t, terms)
    B = th_e * torch.sqrt(1 - e1 * e1 - e2 * e2)
    alpha = torch.exp(t[:, None] * (torch.log(B)[:, None] - 0.5 * torch.log(w2))) * w * S
    bx = x - alpha.real - g1[:, None] * x - g2[:, None] * y
    by = y - alpha.imag - g2[:, None] * x + g1[:, None] * y
    light = 0.0
    if c["lens_light"]:
        light = _sersic(col[:7], x, y)
        col = col[7:]
    light = light + _sersic(col[:7], bx, by)
    if c["nmax"] >= 0:
        light = light + _shapelets(c, col[7:], bx - col[4][:, None], by - col[5][:, None])
    img = light.reshape(-1, H, k, W, k).mean((2, 4))
    return _Convolve.apply(img, _psf(c["K"]).astype(np.float64))


def _chunks(c, P):
    n = max(1, 1_500_000 // (c["H"] * c["W"] * c["k"] ** 2))
    return [(a, min(P, a + n)) for a in range(0, P, n)]


def _logl_64(c, theta, obs, grad=True):
    """log L [P] and its gradient [P, d] in 64 bits."""
    s2b = float(np.float32(c["sigma_bkg"])) ** 2
    obs = torch.from_numpy(obs).to(theta.device, torch.float64)
    ll, g = torch.empty(len(theta), dtype=torch.float64, device=theta.device), torch.zeros_like(theta)
    for a, b in _chunks(c, len(theta)):
        th = theta[a:b].detach().clone().requires_grad_(grad)
        m = _images(c, th, theta.device)
        s2 = s2b + m.clamp_min(0.0) / c["t_exp"]
        v = -0.5 * ((obs - m) ** 2 / s2 + torch.log(2 * math.pi * s2)).sum((1, 2))
        if grad:
            (g[a:b],) = torch.autograd.grad(v.sum(), th)
        ll[a:b] = v.detach()
    return ll, g


def _logpost_64(c, z, obs):
    """log posterior density of unconstrained z [P, d], its gradient, and log L's part."""
    pri = _priors(c)

    def row(key, f=None):
        return torch.tensor([float(np.float32(p[key])) for p in pri], dtype=torch.float64, device=z.device)

    fam = torch.tensor([p["family"] for p in pri], device=z.device)
    mu, sg, lo, hi = row("mu"), row("sigma"), row("lo"), row("hi")
    sig = torch.sigmoid(z)
    boxed = lo + (hi - lo) * sig
    th = torch.where(fam == 0, z, torch.where(fam == 1, torch.exp(torch.where(fam == 1, z, 0 * z)), boxed))
    dth = torch.where(fam == 0, torch.ones_like(z), torch.where(fam == 1, th, (hi - lo) * sig * (1 - sig)))
    r = (torch.where(fam == 2, th, z) - mu) / sg
    jac = 1 - 2 * sig
    dlp = torch.where(fam == 3, jac, torch.where(fam == 2, -r / sg * dth + jac, -r / sg))
    half = -0.5 * r * r - torch.log(sg) - 0.5 * math.log(2 * math.pi)
    cdf = torch.special.ndtr
    box = torch.log(torch.where(fam >= 2, hi - lo, torch.ones_like(hi)))
    Z = torch.where(fam == 2, cdf((hi - mu) / sg) - cdf((lo - mu) / sg), torch.ones_like(mu))
    ls = torch.nn.functional.logsigmoid(z) + torch.nn.functional.logsigmoid(-z)
    lp = torch.where(fam == 3, ls, torch.where(fam == 2, half + ls + box - torch.log(Z), half))
    ll, g = _logl_64(c, th, obs)
    return ll + lp.sum(1), g * dth + dlp


def _pack(mu, chol):
    """Mean and lower factor as the variational state: the factor's rows, log of its diagonal."""
    low = np.array(chol)
    i = np.arange(len(mu))
    low[i, i] = np.log(low[i, i])
    return np.concatenate([mu, low[np.tril_indices(len(mu))]])


def _philox_normals(seed, n, d, k, tag):
    """Standard normals [n, d] by Philox4x32-10 (Salmon et al. 2011) with counter (sample,
    parameter, iteration, tag), Box-Muller on 52-bit uniforms."""
    u64, low = np.uint64, np.uint64(0xFFFFFFFF)
    c = [np.repeat(np.arange(n, dtype=u64), d), np.tile(np.arange(d, dtype=u64), n),
         np.full(n * d, k, u64), np.full(n * d, tag, u64)]
    key = [u64(seed & 0xFFFFFFFF), u64(seed >> 32)]
    for _ in range(10):
        p, q = u64(0xD2511F53) * c[0], u64(0xCD9E8D57) * c[2]
        c = [(q >> u64(32)) ^ c[1] ^ key[0], q & low, (p >> u64(32)) ^ c[3] ^ key[1], p & low]
        key = [(key[0] + u64(0x9E3779B9)) & low, (key[1] + u64(0xBB67AE85)) & low]
    u = [((c[i] >> u64(6)).astype(np.float64) * 2.0 ** 26 + (c[i + 1] >> u64(6)).astype(np.float64) + 0.5) / 2.0 ** 52
         for i in (0, 2)]
    return (np.sqrt(-2.0 * np.log(u[0])) * np.cos(2.0 * np.pi * u[1])).reshape(n, d)


def exact(case, seed):
    c, op = case, case["op"]
    i = _inputs(c, seed)

    def dev(a):
        return torch.from_numpy(np.asarray(a)).cuda().double()

    if op == "image":
        th = dev(i["theta"])
        return torch.cat([_images(c, th[a:b], th.device) for a, b in _chunks(c, len(th))])
    if op in ("loglik", "grad", "autograd"):
        ll, g = _logl_64(c, dev(i["theta"]), i["obs"], op != "loglik")
        return ll if op == "loglik" else (ll, g)
    if op == "fit":
        z = dev(i["z"])
        _, g = _logpost_64(c, z, i["obs"])
        b1, b2, lr = (float(np.float32(v)) for v in (0.9, 0.999, 1e-2))
        m, v = -(1 - b1) * g, (1 - b2) * g * g
        z = z - lr * (m / (1 - b1)) / (torch.sqrt(v / (1 - b2)) + 1e-8)
        return z, m, v, None
    if op == "vi":
        mu, chol = dev(i["mu"]), dev(i["chol"])
        d = len(mu)
        eps = dev(_philox_normals(seed, c["P"], d, 0, 0x76690000))
        _, g = _logpost_64(c, mu + eps @ chol.T, i["obs"])
        g = -g / c["P"]
        gm, gl = g.sum(0), torch.tril(g.T @ eps)
        diag = torch.diagonal(chol)
        lr, b1, b2 = (float(np.float32(v)) for v in (VI_RATE, 0.9, 0.999))

        def adam(x, q):
            return x - lr * q * ((1 - b1) / (1 - b1)) / (torch.sqrt(q * q * (1 - b2) / (1 - b2)) + 1e-8)

        new = torch.tril(adam(chol, gl), -1) + torch.diag(torch.exp(adam(torch.log(diag), diag * torch.diagonal(gl) - 1)))
        return {"mu": adam(mu, gm), "chol": new, "cov": new @ new.T}
    z, p = dev(i["z"]), dev(i["p"])
    chol = dev(i["chol"].astype(np.float32))
    e = float(np.float32(LEAPFROG_EPS))
    lp, g = _logpost_64(c, z, i["obs"])
    p = p + 0.5 * e * g
    for step in range(LEAPFROG_STEPS):
        z = z + e * (p @ chol) @ chol.T
        lp, g = _logpost_64(c, z, i["obs"])
        p = p + (e if step + 1 < LEAPFROG_STEPS else 0.5 * e) * g
    return z, p, lp
