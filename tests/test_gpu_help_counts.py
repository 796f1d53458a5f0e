"""The helpers of a launch, by their counts: they make tiles; with waits
bounded at a microsecond evaluations go on without a tile that is late (the
recovery: the fit's own workgroup makes it and the rest of its evaluations,
the slot is given up), with the same bits; and helpers that the fits still
running have no tiles for leave their compute units."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2404_07780_amd import gmfit as G
from tests.test_gpu_helpers import SIDES, _batch, _reference


def _fit(sides, k, wait_us, seed, **kw):
    gm, b = _batch("sersic", sides, k, seed=seed)
    ctx = G.Context()
    assert not any(G.gm_help_counts(ctx).values())
    G.gm_set_schedule(gm, k, team=2, team_min_tiles=1 << 20, team_wait_us=wait_us, ctx=ctx)      # no teams
    start, _ = G.gm_default_guess(gm, b, ctx=ctx)
    ref = _reference(gm, b, start, ctx=ctx, **kw)
    seen = []
    for _ in range(3):
        for a, c in zip(G.gm_fit_batch(gm, b, start, ctx=ctx, **kw), ref):
            assert torch.equal(a, c)
        seen.append(G.gm_help_counts(ctx))
        assert seen[-1]["idle"] == seen[-1]["turned"] - seen[-1]["left"], seen[-1]
    ctx.close()
    print(seen, flush=True)
    return seen


@pytest.mark.parametrize("k", [15, 9])
def test_helpers_make_tiles(k):
    print(f"help counts: PSF side {k}", flush=True)
    for c in _fit(SIDES, k, 0, 3, max_iter=12):
        assert c["turned"] > 0 and c["tiles"] > 0 and c["lost"] == 0, c


@pytest.mark.parametrize("k", [15, 9])
def test_late_tiles_are_made_by_the_owner(k):
    print(f"help counts: waits of a microsecond, PSF side {k}", flush=True)
    for c in _fit(SIDES, k, 1, 3, max_iter=12):
        assert c["turned"] > 0 and c["lost"] > 0, c


def test_helpers_without_work_leave():
    print("help counts: more helpers than tiles", flush=True)
    for c in _fit([(64, 64)] * 60, 15, 0, 8):
        assert c["tiles"] > 0 and c["left"] > 0, c
