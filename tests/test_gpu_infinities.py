"""A derivative beyond FP32's range at the centre of a bright, compact galaxy
is infinite there and spoils the pixels whose PSF reaches it, and no others:
the Jacobian's non-finite pixels are those within half a PSF side of a
non-finite pixel of the unconvolved Jacobian, and everywhere else the values
are that Jacobian's convolution (numpy, FP64) to the Jacobian bar, 1e-5 of
the column's largest finite value.  Sides with a kernel of
their own and without, an even and an odd number of FP32 planes.

A fit, its errors and the errors kernel use pixels beside such a centre: with
the centre masked as far as the model is above 1e15, a fit of the scale and
the sky (the others fixed) ends where the oracle's does."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle as O
from paper_2404_07780_amd import gmfit as G
from paper_2404_07780_amd import synth as S
from tests.oracle_models import single, to_gm

H, W = 70, 101
# total flux 1e41: 1e39 per pixel at the centre, within FP32's 3.4e38 a few pixels out
SERSIC = [50.3, 34.6, -80.0, 3.0, 1.0, 0.8, 35.0, 3.0]
DISK = [50.3, 34.6, -80.0, 1.8, 0.8, 35.0, 3.0]


def _jacobian(type_, p, psf, convolve):
    om = single(type_, convolve=convolve, sky=True)
    one = np.ones(H * W, np.float32)
    k = psf.shape[0]
    b = G.Batch(np.array([H]), np.array([W]), np.array([0]), np.array([k]), np.array([0]), one, one, psf.ravel())
    return G.gm_jacobian(to_gm(om), b, np.array([p])).cpu().numpy().reshape(om.p, H, W)


def _spread(a, k, fn):
    """fn over the k x k neighbourhood of every pixel (zero outside)."""
    c = k // 2
    z = np.zeros((H + 2 * c, W + 2 * c), a.dtype)
    z[c:c + H, c:c + W] = a
    return fn(np.lib.stride_tricks.sliding_window_view(z, (k, k)))


@pytest.mark.parametrize("type_, p", [(S.SERSIC, SERSIC), (S.EXPDISK, DISK)], ids=["sersic", "expdisk"])
@pytest.mark.parametrize("k", [1, 5, 15, 25, 31, 41])
def test_infinite_derivatives_stay_within_the_psf(k, type_, p):
    print(f"infinities: type {type_}, PSF side {k}", flush=True)
    r = np.random.default_rng(k)
    psf = r.uniform(0.2, 1.0, (k, k))
    psf = (psf / psf.sum()).astype(np.float32)
    raw, jac = _jacobian(type_, p, psf, False), _jacobian(type_, p, psf, True)
    for c in [c for c in range(len(p) - 1) if c != 2]:       # the magnitude's column follows the FP64 light
        bad = ~np.isfinite(raw[c])
        assert bad.any() and bad.sum() < 400, c
        reach = _spread(bad, k, lambda w: w.any(axis=(2, 3)))
        assert np.array_equal(np.isfinite(jac[c]), ~reach), c
        x = np.where(bad, 0.0, raw[c].astype(np.float64))
        flip = psf[::-1, ::-1].astype(np.float64)
        ref = _spread(x, k, lambda w: np.einsum("ijab,ab->ij", w, flip))
        err = np.abs(jac[c].astype(np.float64) - ref)[~reach]
        assert err.max() <= 1e-5 * np.abs(x).max(), c


@pytest.mark.parametrize("team", [1, 2, 4])
@pytest.mark.parametrize("k", [9, 15, 25])
def test_fit_beside_an_infinite_centre(k, team):
    print(f"infinities: fit, PSF side {k}, team {team}", flush=True)
    h, w = 48, 61
    fixed = dict(x0=30.2, y0=24.4, mag=-84.0, n=0.2, q=0.9, pa=20.0)
    om = single(S.SERSIC, sky=True, free=["re"], fixed=fixed)
    psf = np.full((k, k), 1.0 / k ** 2, np.float32)
    truth = np.array([1.5, 1.0])
    jac = O.jacobian(om, h, w, psf, truth).reshape(2, h, w)
    img = O.model_image(om, h, w, psf, truth).reshape(h, w)
    use = (np.abs(jac[0]) < 1e15) & (np.abs(img) < 1e15)
    sigma = np.where(use, 1.0 + 1e-3 * np.abs(img), 1.0).astype(np.float32)
    r = np.random.default_rng(k)
    data = np.where(use, img + sigma * r.normal(size=img.shape), 0.0).astype(np.float32)
    omega = use.astype(np.uint8)
    b = G.Batch(np.array([h]), np.array([w]), np.array([0]), np.array([k]), np.array([0]), data.ravel(),
                sigma.ravel(), psf.ravel(), omega=omega.ravel())
    start = truth * np.array([1.0 + 1e-6, 1.1])
    ctx = G.Context()
    gm = to_gm(om)
    G.gm_set_schedule(gm, k, team=team, team_min_tiles=1 if team == 4 else 1 << 20, ctx=ctx)    # 2: helpers
    err = torch.empty(1, 2, dtype=torch.float64, device=b.device)
    gp, gc, gn, gs = (t.cpu().numpy() for t in G.gm_fit_batch(gm, b, start[None], err_out=err, ctx=ctx))
    rp, rc, rn, rs = O.fit(om, data, sigma, psf, start, omega=omega)
    re = O.param_errors(om, data, sigma, psf, rp, omega=omega)
    assert rs == 0 and int(gs[0]) == 0
    assert np.all(np.abs(gp[0] - rp) <= 1e-3 * re + 1e-9 * np.abs(rp)), (gp[0], rp, re)
    for e in (err, G.gm_param_errors(gm, b, gp, ctx=ctx)):
        assert np.allclose(e.cpu().numpy()[0], re, rtol=1e-3, atol=0), (e, re)
    ctx.close()
