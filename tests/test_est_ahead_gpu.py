"""The EST rollout's kernels against each other: launches of up to one wave per
SIMD request slopes and wheel costs a step ahead, wider ones with a costmap at
the step, and a candidate's results are the same bits in either. The horizons
are at, under and over the four intervals whose controls are requested
together; some candidates reach the goal, in different intervals."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402  (test infrastructure)
from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402
from tests.parity import assert_rollout_parity  # noqa: E402

pytestmark = pytest.mark.gpu


def run(pl, st, u):
    N, _, K = u.shape
    J = torch.full((K,), -7.0, device="cuda")
    fs = torch.full((7, K), -7.0, device="cuda")
    pl.rollout_est(st, torch.from_numpy(np.ascontiguousarray(u)).cuda(), J, fs)
    torch.cuda.synchronize()
    return J.cpu().numpy(), fs.cpu().numpy()


@pytest.mark.parametrize("costmap", [False, True])
@pytest.mark.parametrize("N,S", [(1, 1), (3, 1), (4, 1), (5, 1), (18, 1), (1, 7), (3, 6)])
def test_narrow_launch_equals_wide_one(N, S, costmap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    Kw = 64 * simds + 100
    w = inputs.c2(K=Kw, N=N)
    T = w.terrain
    s = np.asarray(w.state0, np.float32)
    st = np.array([s[0], s[1], s[5], 0, 0, 0, s[6]], np.float32)
    cost = dict(w.cost, goal_x=float(s[0] + 0.1 * s[6]), goal_y=float(s[1]), goal_r=0.2)
    integ = dict(w.integ, substeps=S)
    u = np.ascontiguousarray(w.controls).copy()
    u[N // 2, 0, 3] = np.nan
    cm = None
    if costmap:
        cm = np.random.default_rng(2).uniform(0, 3, T.height.shape).astype(np.float32)
    pl = P.Planner(w.vehicle, cost, integ, Kw, N, T.W, T.H)
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res,
                   None if cm is None else torch.from_numpy(cm).cuda())
    Jw, fw = run(pl, st, u)
    for K in (5, 64, 1000):
        J, fs = run(pl, st, u[:, :, :K])
        np.testing.assert_array_equal(J, Jw[:K])
        np.testing.assert_array_equal(fs, fw[:, :K])
    o = oracle.Oracle(w.vehicle, cost, integ)
    o.set_terrain(T.height, T.x0, T.y0, T.res, cm)
    Jo, fo, _ = o.est_rollout(st, u[:, :, :200])
    assert_rollout_parity(Jw[:200], fw[:, :200], Jo, fo, f"N={N} S={S}")
    pl.close()


@pytest.mark.parametrize("vy", [11.0, 15.0, 40.0, -40.0])
def test_sliding_candidates_narrow_equals_wide(vy):
    """Slip ratios around and beyond 1, where wide launches leave the short
    form of the arctangent, wave by wave."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    Kw, N = 64 * simds + 64, 12
    w = inputs.c2(K=Kw, N=N)
    T = w.terrain
    s = np.asarray(w.state0, np.float32)
    st = np.array([s[0], s[1], s[3], vy, 0, 0, s[6]], np.float32)
    pl = P.Planner(w.vehicle, w.cost, w.integ, Kw, N, T.W, T.H)
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res)
    u = np.ascontiguousarray(w.controls)
    Jw, fw = run(pl, st, u)
    J, fs = run(pl, st, u[:, :, :700])
    np.testing.assert_array_equal(J, Jw[:700])
    np.testing.assert_array_equal(fs, fw[:, :700])
    pl.close()
