"""The convolutions at every remainder of their blocking: PSF sides whose row
segments end inside a four-element group, a 16-tap register or exactly on its
edge, kernels with a compile-time side (15, 25, 41) and the any-side ones,
with an even and an odd number of FP32 planes.  The PSFs are random, so that a
flipped or shifted tap shows.  Model images and Jacobians against the FP64
oracle to the image (1e-5) and Jacobian (1e-5 of a column's peak) bars; two
Adam steps (the correlation with the flipped PSF) to the fit bar (1e-4)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle as O
from paper_2404_07780_amd import gmfit as G
from paper_2404_07780_amd import synth as S
from tests.gpu_helpers import image_parity, param_parity
from tests.oracle_models import single, to_gm

H, W = 43, 37
SIDES = [1, 3, 5, 7, 13, 15, 17, 25, 29, 31, 33, 41, 45]
SERSIC = [18.2, 21.6, 17.0, 6.0, 2.3, 0.6, 35.0, 3.0]
DISK = [18.2, 21.6, 17.0, 4.0, 0.6, 35.0, 3.0]      # five FP32 planes: one without a partner


def _psf(k):
    r = np.random.default_rng(k)
    p = r.uniform(0.2, 1.0, (k, k)) * np.exp(-np.hypot(*np.mgrid[-(k // 2):k // 2 + 1, -(k // 2):k // 2 + 1]) / 3.0)
    return (p / p.sum()).astype(np.float32)


def _batch(psf, data=None, sigma=None):
    k = psf.shape[0]
    one = np.ones(H * W, np.float32)
    return G.Batch(np.array([H]), np.array([W]), np.array([0]), np.array([k]), np.array([0]),
                   one if data is None else data.ravel(), one if sigma is None else sigma.ravel(), psf.ravel())


@pytest.mark.parametrize("type_, p", [(S.SERSIC, SERSIC), (S.EXPDISK, DISK)], ids=["sersic", "expdisk"])
@pytest.mark.parametrize("k", SIDES)
def test_image_and_jacobian(k, type_, p):
    print(f"PSF side {k}, type {type_}", flush=True)
    om = single(type_, sky=True)
    psf, p = _psf(k), np.array([p])
    b = _batch(psf)
    ok, worst = image_parity(G.gm_model_image(to_gm(om), b, p).cpu().numpy().reshape(H, W),
                             O.model_image(om, H, W, psf, p[0]))
    assert ok, worst
    jac = G.gm_jacobian(to_gm(om), b, p).cpu().numpy().reshape(om.p, H, W)
    ref = O.jacobian(om, H, W, psf, p[0]).reshape(om.p, H, W)
    for c in range(om.p):
        assert np.max(np.abs(jac[c] - ref[c])) <= 1e-5 * np.max(np.abs(ref[c])), c


@pytest.mark.parametrize("k", [3, 15, 17, 25, 31])
def test_adam_correlation(k):
    print(f"Adam, PSF side {k}", flush=True)
    om = single(S.SERSIC, sky=True)
    psf, truth = _psf(k), np.array(SERSIC)
    data = (O.model_image(om, H, W, psf, truth).reshape(H, W)
            + np.random.default_rng(1).normal(size=(H, W))).astype(np.float32)
    sigma = np.ones((H, W), np.float32)
    start = truth + np.array([0.3, -0.2, 0.1, 0.5, -0.3, 0.1, 5.0, 0.2])
    gp = G.gm_fit_adam(to_gm(om), _batch(psf, data, sigma), start[None], steps=2)[0].cpu().numpy()[0]
    rp = O.fit_adam(om, data, sigma, psf, start, steps=2)[0]
    ok, worst = param_parity(["x0", "y0", "mag", "re", "n", "q", "pa", "sky"], gp, rp)
    assert ok.all(), worst
