"""The EST rollout's kernels against each other: launches of up to one wave per
SIMD request slopes and wheel costs a step ahead, wider ones with a costmap at
the step, and a candidate's results are the same bits in either. The horizons
are at, under and over the four intervals whose controls are requested
together; some candidates reach the goal, in different intervals. Launches of some waves per SIMD and a remainder share
their steps equally between the waves, cutting candidates' horizons anywhere."""
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


def many(rounds, rest, N, S, capacity=None):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    K = 64 * (rounds * simds + rest) - 3
    T = inputs.c2(K=8, N=N)
    w, t = T, T.terrain
    s = np.asarray(w.state0, np.float32)
    st = np.array([s[0], s[1], s[3], 0, 0, 0, s[6]], np.float32)
    cost = dict(w.cost, goal_x=float(s[0] + 0.2 * s[6]), goal_y=float(s[1]), goal_r=0.3)
    g = torch.Generator(device="cuda")
    g.manual_seed(K + N)
    u = 0.8 * torch.randn(N, 2, K, generator=g, device="cuda")
    pl = P.Planner(w.vehicle, cost, dict(w.integ, substeps=S), K, N, t.W, t.H)
    pl.set_terrain(torch.from_numpy(t.height).cuda(), t.x0, t.y0, t.res)
    return pl, st, u, K, simds


def narrow(pl, st, u, simds):
    """The launches of one wave per SIMD that together hold the candidates."""
    J, fs = [], []
    for a in range(0, u.shape[2], 64 * simds):
        part = u[:, :, a:a + 64 * simds].contiguous()
        Jp = torch.empty(part.shape[2], device="cuda")
        fp = torch.empty(7, part.shape[2], device="cuda")
        pl.rollout_est(st, part, Jp, fp)
        J.append(Jp)
        fs.append(fp)
    return torch.cat(J), torch.cat(fs, 1)


# remainders of one group, of most of a quarter, a half and three quarters of a
# round (the shared form ends there), with horizons shorter than a trip of
# controls, of one step, and of several substeps
@pytest.mark.parametrize("rounds,rest", [(1, 1), (1, 250), (1, 300), (2, 3), (2, 760), (2, 800),
                                         (3, 121), (4, 500), (6, 40), (7, 1)])
@pytest.mark.parametrize("N,S", [(1, 1), (5, 1), (30, 1), (4, 9)])
def test_equal_shares_equal_narrow_launches(rounds, rest, N, S):
    pl, st, u, K, simds = many(rounds, rest, N, S)
    want = narrow(pl, st, u, simds)
    J, fs = torch.empty(K, device="cuda"), torch.empty(7, K, device="cuda")
    for _ in range(3):
        J.fill_(-7.0)
        fs.fill_(-7.0)
        pl.rollout_est(st, u, J, fs)
        assert torch.equal(J, want[0]) and torch.equal(fs, want[1])
    pl.close()


@pytest.mark.parametrize("shares_on_side", [False, True])
def test_equal_shares_other_streams_and_graphs(shares_on_side):
    """Another stream and a captured graph take the form without shared state."""
    pl, st, u, K, simds = many(3, 121, 6, 1)
    want = narrow(pl, st, u, simds)  # on the default stream, unshared
    outs = [(torch.empty(K, device="cuda"), torch.empty(7, K, device="cuda")) for _ in range(3)]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    if not shares_on_side:
        pl.rollout_est(st, u, *outs[0])
    P.plan_set_stream(pl.ctx, side.cuda_stream)
    pl.rollout_est(st, u, *outs[1])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        pl.rollout_est(st, u, *outs[2])
    for _ in range(3):
        outs[2][0].fill_(-7.0)
        torch.cuda.synchronize()
        graph.replay()
        P.plan_set_stream(pl.ctx, 0)
        pl.rollout_est(st, u, *outs[0])
        torch.cuda.synchronize()
        for J, fs in outs:
            assert torch.equal(J, want[0]) and torch.equal(fs, want[1])
    pl.close()
