"""Workgroups that find the work queue empty help the fits still running: they
make tiles of the owners' evaluations.  The owner adds every tile's products
itself, in tile order, so a fit gives the same bits however many helpers it
had; gm_fit_batch_noalloc runs without helpers and is the reference (as is
team = 1).  Batches
far smaller than the resident workgroups, so that helpers are there from the
start: cutouts of one to 64 tiles (more tiles than the ring of 16, more than
the 16 tiles between flushes), both PSF-side paths, the two-component model,
masks, a learned fit's refit inside a plan, and waits bounded at a
microsecond."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2404_07780_amd import gmfit as G
from paper_2404_07780_amd import learned as L
from paper_2404_07780_amd import synth as S


def _batch(model, sides, k, seed):
    """Galaxies rendered by the library (the fits are compared with each other), masked at random."""
    r = np.random.default_rng(seed)
    n = len(sides)
    h = np.array([a for a, _ in sides], np.int32)
    w = np.array([b for _, b in sides], np.int32)
    off = np.concatenate([[0], np.cumsum(h.astype(np.int64) * w)[:-1]])
    truth = np.zeros((n, S.MODEL_SPECS[model]["p"]))
    truth[:, 0], truth[:, 1] = w / 2 + r.uniform(-2, 2, n), h / 2 + r.uniform(-2, 2, n)
    truth[:, 2], truth[:, 3], truth[:, 4] = 15.0, r.uniform(2, 9, n), r.uniform(0.6, 5, n)
    truth[:, 5], truth[:, 6], truth[:, -1] = r.uniform(0.3, 1, n), r.uniform(0, 180, n), 1.0
    if model == "bulgedisk":
        truth[:, 7], truth[:, 8], truth[:, 9], truth[:, 10] = 14.5, r.uniform(4, 9, n), r.uniform(0.3, 1, n), 40.0
    psf = np.tile(S.gaussian_psf(2.0, k).astype(np.float32).ravel(), n)
    npix = int((h.astype(np.int64) * w).sum())
    one = np.ones(npix, np.float32)
    gm = G.Model.from_spec(S.MODEL_SPECS[model])
    ks, po = np.full(n, k, np.int32), np.arange(n, dtype=np.int64) * k * k
    img = G.gm_model_image(gm, G.Batch(h, w, off, ks, po, one, one, psf), truth).cpu().numpy()
    data = (img + r.normal(size=npix)).astype(np.float32)
    return gm, G.Batch(h, w, off, ks, po, data, one, psf, omega=(r.uniform(size=npix) > 0.03).astype(np.uint8))


def _reference(gm, b, start, **kw):
    out = [start.clone(), torch.empty(b.n, dtype=torch.float64, device=b.device),
           torch.empty(b.n, dtype=torch.int32, device=b.device), torch.empty(b.n, dtype=torch.int32, device=b.device)]
    G.gm_fit_batch_noalloc(gm, b, *out, **kw)
    return out


SIDES = [(64, 64), (256, 256), (30, 30), (70, 95), (161, 224), (33, 32), (128, 129), (96, 40)]


@pytest.mark.parametrize("model, k", [("sersic", 15), ("sersic", 25), ("sersic", 9), ("bulgedisk", 25)])
@pytest.mark.parametrize("wait_us", [0, 1])
def test_helped_fits_are_the_same_bits(model, k, wait_us):
    print(f"helpers: {model}, PSF side {k}, waits {wait_us or 'default'}", flush=True)
    gm, b = _batch(model, SIDES, k, seed=k + 1)
    ctx = G.Context()
    G.gm_set_schedule(gm, k, team=2, team_min_tiles=1 << 20, team_wait_us=wait_us, ctx=ctx)     # no teams
    start, _ = G.gm_default_guess(gm, b, ctx=ctx)
    ref = _reference(gm, b, start, ctx=ctx, max_iter=12)
    for rep in range(3):
        got = G.gm_fit_batch(gm, b, start, ctx=ctx, max_iter=12)
        for a, c in zip(got, ref):
            assert torch.equal(a, c), rep
    G.gm_set_schedule(gm, k, team=1, ctx=ctx)
    for a, c in zip(G.gm_fit_batch(gm, b, start, ctx=ctx, max_iter=12), ref):
        assert torch.equal(a, c)
    ctx.close()


def test_helped_plan_with_refit():
    """A plan replayed three times (its reset is a graph node) equals the eager call and, where the first fit
    converged, the unhelped fit from the same start."""
    print("helpers: learned plan", flush=True)
    gm, b = _batch("sersic", [(64, 64)] * 6 + [(100, 140)] * 2, 15, seed=5)
    ctx = G.Context()
    G.gm_set_schedule(gm, 15, team=2, team_min_tiles=1 << 20, ctx=ctx)      # no teams
    mlp = L.new_mlp(3, train=False)
    want = G.gm_fit_learned(gm, b, mlp, ctx=ctx, proposal_max_iter=3)
    start, _ = G.gm_default_guess(gm, b, ctx=ctx)
    ref = _reference(gm, b, start, ctx=ctx)
    refitted = want[4] > 0
    assert bool(refitted.any())
    assert torch.equal(want[0][refitted], ref[0][refitted]) and torch.equal(want[1][refitted], ref[1][refitted])
    plan = G.gm_plan_fit_learned(gm, b, mlp, errors=False, proposal_max_iter=3, ctx=ctx)
    for _ in range(3):
        plan.launch()
        torch.cuda.synchronize()
        for a, c in zip((plan.params, plan.chi2, plan.niter, plan.status), want):
            assert torch.equal(a, c)
        G.gm_fit_batch(gm, b, start, ctx=ctx)
    plan.close()
    ctx.close()
