"""Smoothing's paths against each other and the oracle: the one-kernel form,
the two-kernel form (a call in place) and the scalar loops a tile falls back to
around an infinity or a NaN all sum in the same order, so they agree bit for
bit wherever their windows are finite."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402  (test infrastructure)
from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def planner():
    pl = P.Planner(inputs.WORKLOAD_VEHICLE, inputs.BASE_COST, inputs.BASE_INTEG, 8, 8, 700, 700)
    yield pl
    pl.close()


def heights(H, W):
    rng = np.random.default_rng(H * 1009 + W)
    return torch.from_numpy(rng.normal(0.0, 0.4, (H, W)).astype(np.float32)).cuda()


# radii at the ends of both forms (1, 28 | 29, 127), at a whole number of steps
# of four taps and one short of it; sizes at, under and over the tiles
@pytest.mark.parametrize("r", [1, 2, 9, 18, 24, 28, 29, 60, 127])
@pytest.mark.parametrize("H,W", [(1, 1), (64, 64), (63, 65), (129, 257), (16, 300), (500, 31)])
def test_in_place_equals_out_of_place_and_oracle(planner, r, H, W):
    h = heights(H, W)
    out = torch.full((H, W), math.nan, device="cuda")
    planner.smooth_terrain(h, 0.1, 0.1 * r / 3, out)
    same = h.clone()
    planner.smooth_terrain(same, 0.1, 0.1 * r / 3, same)
    assert torch.equal(out, same)
    ref = oracle.smooth_terrain(h.cpu().numpy(), float(np.float32(0.1)), float(np.float32(0.1 * r / 3)))
    # two passes of 2r + 1 taps: (2r + 2) roundings each of the largest height
    tol = 2 * (2 * r + 2) * 2.0 ** -24 * float(h.abs().max())
    assert float(np.abs(out.cpu().numpy() - ref).max()) <= tol


def test_overlapping_buffers(planner):
    """An output that starts a few rows into the heights."""
    buf = torch.zeros(140, 90, device="cuda")
    h, out = buf[:100], buf[37:137]
    buf[:100] = heights(100, 90)
    want = torch.empty(100, 90, device="cuda")
    planner.smooth_terrain(h.clone(), 0.1, 0.6, want)
    planner.smooth_terrain(h, 0.1, 0.6, out)
    assert torch.equal(out, want)


@pytest.mark.parametrize("r", [9, 28, 60])
@pytest.mark.parametrize("value", [math.nan, math.inf, -math.inf])
@pytest.mark.parametrize("in_place", [False, True])
def test_non_finite_heights_stay_in_their_window(planner, r, value, in_place):
    H, W = 200, 330
    h = heights(H, W)
    clean = torch.empty_like(h)
    planner.smooth_terrain(h, 0.1, 0.1 * r / 3, clean)
    for j, i in ((100, 150), (0, 0), (199, 329)):
        bad = h.clone()
        bad[j, i] = value
        out = bad if in_place else torch.empty_like(h)
        planner.smooth_terrain(bad, 0.1, 0.1 * r / 3, out)
        hit = torch.zeros(H, W, dtype=torch.bool, device="cuda")
        hit[max(j - r, 0):j + r + 1, max(i - r, 0):i + r + 1] = True
        assert torch.equal(out[~hit], clean[~hit])
        if math.isnan(value):
            assert bool(torch.isnan(out[hit]).all())
        else:
            assert bool((out[hit] == value).all())
