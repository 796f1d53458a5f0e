"""One Adam step that is linear in the gradient (no moments, eps far above it:
u moves by 2 lr g / eps, g = J^T W r), so that the gradient itself shows: the
light's correlation with the flipped PSF at every PSF-side path, PSFs without
any symmetry, sides with one, two and three tap registers.  g against the
oracle's Jacobian to the adjoint's bar (1e-5 of the sum of magnitudes), chi^2
against the oracle's model at the step's end (1e-6).  test_wrong_psfs_show
checks on the CPU that a PSF that is not flipped, or is shifted or transposed,
in the gradient misses that bar a hundredfold."""
import math

import numpy as np
import pytest

import oracle as O
from paper_2404_07780_amd import synth as S
from tests.oracle_models import single, to_gm

H, W = 43, 70
SERSIC = [35.2, 21.6, 15.0, 6.0, 2.3, 0.6, 35.0, 3.0]
NAMES = ["x0", "y0", "mag", "re", "n", "q", "pa", "sky"]
SIDES = [3, 9, 15, 17, 25, 31, 41]
EPS = 1e12


def _case(k):
    """PSF, data, sigma and start; the gradient g and the sum of magnitudes in the LM variables."""
    r = np.random.default_rng(40 + k)
    yy, xx = np.mgrid[-(k // 2):k // 2 + 1, -(k // 2):k // 2 + 1]
    psf = r.uniform(0.2, 1.0, (k, k)) * np.exp(-np.hypot(yy - 0.1 * k, xx + 0.2 * k) / (0.3 * k))
    psf = (psf / psf.sum()).astype(np.float32)
    om, truth = single(S.SERSIC, sky=True), np.array(SERSIC)
    data = (O.model_image(om, H, W, psf, truth).reshape(H, W) + r.normal(size=(H, W))).astype(np.float32)
    sigma = r.uniform(0.8, 1.6, (H, W)).astype(np.float32)
    start = truth + np.array([0.4, -0.3, 0.1, 0.6, -0.3, 0.08, 6.0, 0.3])
    return om, psf, data, sigma, start


def _du(names, p):
    """d natural / d LM variable at p."""
    return np.array([p[i] if n in ("re", "n") else 180.0 / math.pi if n == "pa" else 1.0
                     for i, n in enumerate(names)])


def _gradient(om, psf, data, sigma, start, light=None):
    """g and sum |.|, with the derivatives convolved with `psf`, the residual's model with `light`."""
    res = data.astype(np.float64) - O.model_image(om, H, W, psf if light is None else light, start).reshape(H, W)
    terms = O.jacobian(om, H, W, psf, start).reshape(-1, H * W) * (res / sigma.astype(np.float64) ** 2).ravel()
    return terms.sum(1) * _du(NAMES, start), np.abs(terms).sum(1) * _du(NAMES, start)


@pytest.mark.parametrize("k", SIDES)
def test_wrong_psfs_show(k):
    om, psf, data, sigma, start = _case(k)
    g, mag = _gradient(om, psf, data, sigma, start)
    # columns whose gradient comes by the correlation (the magnitude's uses the forward light)
    corr = [0, 1, 3, 4, 5, 6]
    for wrong in (psf[::-1, ::-1], psf.T, np.roll(psf, 1, axis=1), np.roll(psf, 1, axis=0)):
        bad, _ = _gradient(om, np.ascontiguousarray(wrong), data, sigma, start, light=psf)
        assert np.max(np.abs(bad - g)[corr] / mag[corr]) > 1e-3


@pytest.mark.gpu
@pytest.mark.parametrize("k", SIDES)
def test_gradient_step(k):
    torch = pytest.importorskip("torch")
    from paper_2404_07780_amd import gmfit as G

    print(f"Adam gradient, PSF side {k}", flush=True)
    om, psf, data, sigma, start = _case(k)
    g, mag = _gradient(om, psf, data, sigma, start)
    lr = 1e-3 * EPS / np.max(np.abs(2 * g))
    b = G.Batch(np.array([H]), np.array([W]), np.array([0]), np.array([k]), np.array([0]), data.ravel(),
                sigma.ravel(), psf.ravel())
    p, chi2 = (t.cpu().numpy() for t in G.gm_fit_adam(to_gm(om), b, start[None], steps=1, lr=lr, beta1=0.0,
                                                      beta2=0.0, eps=EPS)[:2])
    du = np.array([math.log(p[0][i] / start[i]) if n in ("re", "n") else
                   math.radians(p[0][i] - start[i]) if n == "pa" else p[0][i] - start[i] for i, n in enumerate(NAMES)])
    # the step is 2 lr g / (2 |g| + eps); natural values are kept to 2^-52 of their size
    got, slack = du * EPS / (2 * lr), 1e-13 * EPS / lr
    assert np.all(np.abs(got - g) <= 1e-5 * mag + slack), (got, g, mag)
    w = 1.0 / sigma.astype(np.float64) ** 2
    want = np.sum(w * (data - O.model_image(om, H, W, psf, p[0]).reshape(H, W)) ** 2)
    assert abs(chi2[0] - want) <= 1e-6 * want
