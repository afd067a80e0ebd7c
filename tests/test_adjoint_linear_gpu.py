"""The backward pass of few candidates, whose steps are linearised in parallel,
against the serial one, which the same candidates get in a launch of many."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu


def planner(K, N, S, costmap):
    w = inputs.c2(K=K, N=N)
    T = w.terrain
    st = np.array(w.state0, np.float32)
    cost = dict(w.cost, sigma=40.0, eps_esm=2000.0)
    # some candidates reach the goal, in different intervals
    cost.update(goal_x=float(st[0] + 0.3 * st[6]), goal_y=float(st[1]), goal_r=0.4)
    pl = P.Planner(w.vehicle, cost, dict(w.integ, substeps=S), K, N, T.W, T.H)
    cm = None
    if costmap:
        rng = np.random.default_rng(3)
        cm = torch.from_numpy(rng.uniform(0, 3, T.height.shape).astype(np.float32)).cuda()
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res, cm)
    u = np.ascontiguousarray(w.controls)
    u[: max(N // 3, 1), 0, 5] = 9.0      # clamped
    u[0, 1, 6] = np.nan                  # scores +inf
    u[:, 1, 7] = -4.0
    return pl, st, u


def grad(pl, st, u, C, weight=None):
    N, _, K = u.shape
    J = torch.full((K,), -7.0, device="cuda")
    g = torch.full((N, 2, K), -7.0, device="cuda")
    w = None if weight is None else torch.from_numpy(weight).cuda()
    pl.rollout_grad(st, torch.from_numpy(np.ascontiguousarray(u)).cuda(), J, g, w, C)
    torch.cuda.synchronize()
    return J.cpu().numpy(), g.cpu().numpy()


def many():
    """More candidates than the parallel pass takes."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return 24 * torch.cuda.get_device_properties(0).multi_processor_count + 8


# horizons at, under and over a batch of sixteen steps and the 160 whose states
# fit on chip; segments of one step, of some, of all; candidate counts that do
# not fill a workgroup's four
@pytest.mark.parametrize("costmap", [False, True])
@pytest.mark.parametrize("N,S,C", [(1, 1, 1), (15, 1, 4), (16, 1, 16), (17, 1, 1), (40, 4, 7),
                                   (41, 4, 41), (9, 17, 2), (200, 1, 200), (200, 1, 14),
                                   (3, 100, 1)])
def test_equals_serial_pass(N, S, C, costmap):
    Kw = many()
    pl, st, u = planner(Kw, N, S, costmap)
    weight = np.linspace(-1.0, 2.0, Kw).astype(np.float32)
    Jw, gw = grad(pl, st, u, C, weight)
    assert np.isinf(Jw[6]) and not gw[:, :, 6].any()
    # two float32 evaluations of the same products: 64 roundings a step, each
    # of the candidate's largest entry
    tol = 64 * N * S * 2.0 ** -24
    for K in (9, 64, 262):
        J, g = grad(pl, st, u[:, :, :K], C, weight[:K])
        np.testing.assert_array_equal(J, Jw[:K])
        r = gw[:, :, :K]
        scale = np.abs(r).max(axis=(0, 1))
        assert np.array_equal(g == 0, r == 0)
        assert (np.abs(g - r).max(axis=(0, 1)) <= tol * scale).all()
    pl.close()


@pytest.mark.parametrize("N", [1, 2, 3, 12])
def test_blown_up_candidates_equal_serial_pass_bitwise(N):
    """States outside any vehicle's range go through the serial steps (a roll
    rate of 3e8 rad/s, beyond the kernel's 1e8; the cost is finite in the first
    step)."""
    Kw = many()
    pl, st, u = planner(Kw, N, 1, False)
    st = st.copy()
    st[9] = 3e8
    Jw, gw = grad(pl, st, u, 5)
    J, g = grad(pl, st, u[:, :, :33], 5)
    np.testing.assert_array_equal(J, Jw[:33])
    np.testing.assert_array_equal(g, gw[:, :, :33])
    if N == 1:
        assert np.isfinite(J).any() and g.any()
    pl.close()
