"""A model image is the same bits under every plane-group count that fits its
PSF side (the light alone is evaluated, in LDS sized for one plane): every
count that the library offers for the batch's largest side runs, and none is
passed over."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2404_07780_amd import gmfit as G
from paper_2404_07780_amd import synth as S
from tests.test_gpu_image_light import SHAPES, TRUTH


@pytest.mark.parametrize("sides", [(1, 1, 1), (15, 15, 15), (25, 25, 25), (41, 41, 41), (5, 31, 15)])
@pytest.mark.parametrize("model", ["sersic", "bulgedisk"])
def test_image_is_the_same_under_every_plane_group_count(model, sides):
    h, w = (np.array(x, np.int32) for x in zip(*SHAPES))
    off = np.concatenate([[0], np.cumsum(h.astype(np.int64) * w)[:-1]])
    ks = np.array(sides, np.int32)
    po = np.concatenate([[0], np.cumsum(ks.astype(np.int64) ** 2)[:-1]])
    psf = np.concatenate([np.random.default_rng(k).uniform(0.2, 1.0, k * k) / k ** 2 for k in sides])
    one = np.ones(int((h.astype(np.int64) * w).sum()), np.float32)
    b = G.Batch(h, w, off, ks, po, one, one, psf.astype(np.float32))
    gm = G.Model.from_spec(S.MODEL_SPECS[model])
    truth = np.tile(np.array(TRUTH[model]), (len(SHAPES), 1))
    want = G.gm_model_image(gm, b, truth)
    counts = G.gm_schedule_options(gm, max(sides))
    print(f"plane groups: {model}, PSF sides {sides}: {counts}", flush=True)
    assert counts
    for ng in counts:
        ctx = G.Context()
        for k in set(sides):
            G.gm_set_schedule(gm, k, plane_groups=ng, ctx=ctx)
        assert torch.equal(G.gm_model_image(gm, b, truth, ctx=ctx), want), ng
        ctx.close()
