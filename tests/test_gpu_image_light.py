"""The model image evaluates the light plane alone, in LDS sized for that
plane: one and two components, cutouts with a last tile of one row and column,
each compiled PSF side and the any-side kernel, galaxies of different sides in
one batch (the LDS is sized for the largest), and the plane-group counts, on
which an image does not depend (same bits).  Against the FP64 oracle to the
image bar (1e-5)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle as O
from paper_2404_07780_amd import gmfit as G
from paper_2404_07780_amd import synth as S
from tests.gpu_helpers import image_parity
from tests.oracle_models import from_spec

SHAPES = [(32, 32), (33, 65), (40, 31)]
TRUTH = {"sersic": [16.2, 14.6, 17.0, 5.0, 2.3, 0.6, 35.0, 3.0],
         "bulgedisk": [16.2, 14.6, 17.0, 3.0, 3.1, 0.8, 20.0, 16.5, 6.0, 0.5, 40.0, 3.0]}


@pytest.mark.parametrize("sides", [(15, 15, 15), (25, 25, 25), (41, 41, 41), (1, 1, 1), (5, 31, 15)])
@pytest.mark.parametrize("model", ["sersic", "bulgedisk"])
def test_image(model, sides):
    print(f"{model}, PSF sides {sides}", flush=True)
    n = len(SHAPES)
    h = np.array([a for a, _ in SHAPES], np.int32)
    w = np.array([b for _, b in SHAPES], np.int32)
    off = np.concatenate([[0], np.cumsum(h.astype(np.int64) * w)[:-1]])
    r = np.random.default_rng(7)
    psfs = []
    for k in sides:
        p = r.uniform(0.2, 1.0, (k, k))
        psfs.append((p / p.sum()).astype(np.float32))
    ks = np.array(sides, np.int32)
    po = np.concatenate([[0], np.cumsum(ks.astype(np.int64) ** 2)[:-1]])
    one = np.ones(int((h.astype(np.int64) * w).sum()), np.float32)
    b = G.Batch(h, w, off, ks, po, one, one, np.concatenate([p.ravel() for p in psfs]))
    truth = np.tile(np.array(TRUTH[model]), (n, 1))
    gm, om = G.Model.from_spec(S.MODEL_SPECS[model]), from_spec(model)
    img = G.gm_model_image(gm, b, truth)
    got = img.cpu().numpy()
    for g in range(n):
        ref = O.model_image(om, int(h[g]), int(w[g]), psfs[g], truth[g])
        ok, worst = image_parity(got[off[g]:off[g] + h[g] * w[g]].reshape(h[g], w[g]), ref)
        assert ok, (SHAPES[g], sides[g], worst)
    for ng in {"sersic": (1, 2), "bulgedisk": (2, 3)}[model]:
        ctx = G.Context()
        try:
            for k in set(sides):
                G.gm_set_schedule(gm, k, plane_groups=ng, ctx=ctx)
            other = G.gm_model_image(gm, b, truth, ctx=ctx)
        except G.GmError:
            assert max(sides) > 15      # the LDS does not hold that many planes of a wide PSF
            continue
        assert torch.equal(img, other), ng
