"""Launches of at most one wave per SIMD over two or four lanes per candidate
take the loop that requests cells and controls ahead, in trips of four
intervals, and give a drawn interval's pair to a group from the lane that drew
it. Every candidate's results must equal, bit for bit, those it has in a launch
too wide for that loop, which takes the general one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu
N_MAX = 21


@pytest.fixture(scope="module", params=[False, True], ids=["no_costmap", "costmap"])
def case(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    K = 32 * simds + 64  # more than one wave per SIMD at two and at four lanes
    w = inputs.c2(K=K, N=N_MAX)
    T = w.terrain
    cost = dict(w.cost)
    integ = dict(w.integ, dt=0.05)
    # a goal that some candidates reach, in different intervals
    st = w.state0
    cost.update(goal_x=float(st[0] + 0.35 * st[6] * np.cos(st[5])),
                goal_y=float(st[1] + 0.35 * st[6] * np.sin(st[5])), goal_r=0.3)
    u = np.ascontiguousarray(w.controls).copy()
    u[7, 0, 3] = np.nan
    u[4, 1, 40] = np.nan
    u[0, 1, 17] = np.inf
    pl = P.Planner(w.vehicle, cost, integ, K, N_MAX, T.W, T.H)
    cm = None
    if request.param:
        rng = np.random.default_rng(5)
        cm = torch.from_numpy(rng.uniform(0, 3, T.height.shape).astype(np.float32)).cuda()
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res, cm)
    pl.set_order(P.PLAN_ORDER_OFF)
    yield pl, np.asarray(st), u, K
    pl.close()


def run(pl, st, u, K, N, spec, lanes, block):
    pl.set_launch(lanes, block)
    J = torch.full((K,), -7.0, device="cuda")
    fs = torch.full((13, K), -7.0, device="cuda")
    if spec is None:
        pl.rollout(st, torch.from_numpy(np.ascontiguousarray(u[:N, :, :K])).cuda(), J, fs)
    else:
        pl.rollout_sampled(st, spec, N, J, fs)
    torch.cuda.synchronize()
    pl.set_launch(0, 0)
    return J.cpu().numpy(), fs.cpu().numpy()


def same(a, b, msg):
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y, err_msg=msg)


# horizons at, under and over a trip, and those at which a lane group's draws
# (sixteen intervals at four lanes) end; candidate counts that fill a wave, a
# compute unit's waves, and neither
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 7, 8, 15, 16, 17, 21])
@pytest.mark.parametrize("draws", ["given", "uniform", "gauss"])
def test_equals_general_loop(case, N, draws):
    pl, st, u, Kw = case
    spec = None
    if draws == "uniform":
        spec = P.sample_spec(P.PLAN_SAMPLE_UNIFORM, 11, 3, (1.5, 1.2))
    elif draws == "gauss":
        nominal = torch.from_numpy(np.linspace(-0.3, 0.4, 2 * N).reshape(N, 2)
                                   .astype(np.float32)).cuda()
        spec = P.sample_spec(P.PLAN_SAMPLE_GAUSSIAN, 11, 3, (0.6, 0.4), nominal=nominal,
                             keep_nominal=True, N=N)
    wide = {lanes: run(pl, st, u, Kw, N, spec, lanes, 64) for lanes in (2, 4)}
    same(wide[2], wide[4], "general loop")
    if N == N_MAX and draws == "given":
        assert np.isinf(wide[4][0]).any() and np.isfinite(wide[4][0]).any()
        moved = np.unique(wide[4][1][0]).size
        assert moved > Kw // 2
    for K in (1, 63, 64, 700):
        for lanes, block in ((2, 64), (2, 256), (4, 64), (4, 256), (0, 0)):
            got = run(pl, st, u, K, N, spec, lanes, block)
            same(got, (wide[4][0][:K], wide[4][1][:, :K]), f"K={K} lanes={lanes} block={block}")


@pytest.mark.parametrize("lanes", [2, 4])
def test_chunks_and_goal_at_the_start(case, lanes):
    """Chunks that start at any interval, and a start that is at the goal."""
    pl, st, u, Kw = case
    K, N = 300, N_MAX
    ud = torch.from_numpy(np.ascontiguousarray(u[:, :, :K])).cuda()
    want = run(pl, st, u, Kw, N, None, lanes, 64)
    pl.set_launch(lanes, 64)
    J, fs = torch.empty(K, device="cuda"), torch.empty(13, K, device="cuda")
    pl.init_state(st, fs, J)
    for n0, n1 in ((0, 3), (3, 3), (3, 10), (10, 11), (11, N)):
        pl.rollout_chunk(fs, J, ud, n0, n1, n1 == N)
    torch.cuda.synchronize()
    pl.set_launch(0, 0)
    same((J.cpu().numpy(), fs.cpu().numpy()), (want[0][:K], want[1][:, :K]), "chunks")
    at_goal = st.copy()
    at_goal[0] += 0.35 * st[6] * np.cos(st[5])
    at_goal[1] += 0.35 * st[6] * np.sin(st[5])
    J, fs = run(pl, at_goal, u, K, N, None, lanes, 64)
    assert (fs == at_goal.astype(np.float32)[:, None]).all() and np.unique(J).size == 1


# checkpoints at, between and past the ends of trips, and at the horizon's end
@pytest.mark.parametrize("C", [1, 3, 4, 7, 20, 21])
@pytest.mark.parametrize("N", [3, 20, 21])
def test_checkpoints_equal_general_loop(case, N, C):
    """Costs and gradients of launches whose backward pass is the serial one
    either way: it starts every segment from a checkpoint."""
    pl, st, u, Kw = case
    res = []
    for K in (Kw, (Kw - 64) // 4 + 3):  # 8 candidates per SIMD: one wave, serial backward
        ud = torch.from_numpy(np.ascontiguousarray(u[:N, :, :K])).cuda()
        pl.set_launch(4, 64)
        J, g = torch.empty(K, device="cuda"), torch.empty(N, 2, K, device="cuda")
        pl.rollout_grad(st, ud, J, g, None, C)
        torch.cuda.synchronize()
        pl.set_launch(0, 0)
        res.append((J.cpu().numpy(), g.cpu().numpy(), K))
    (Jw, gw, _), (J, g, K) = res
    same((J, g), (Jw[:K], gw[:, :, :K]), f"N={N} C={C}")


@pytest.mark.parametrize("N,S", [(1, 1), (2, 1), (7, 1), (3, 4)])
@pytest.mark.parametrize("costmap", [False, True])
def test_runge_kutta_equals_general_loop(N, S, costmap):
    """Runge-Kutta's stages requested ahead (up to one wave per SIMD over two
    or four lanes) against the step that requests each stage's cells at it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    Kw = 32 * simds + 64
    w = inputs.c2(K=Kw, N=N)
    T = w.terrain
    st = np.asarray(w.state0)
    # arrivals in the second step, and a start at the goal below
    cost = dict(w.cost, goal_x=float(st[0] + 0.05 * st[6]), goal_y=float(st[1]), goal_r=0.3)
    u = np.ascontiguousarray(w.controls).copy()
    u[0, 0, 3] = np.nan
    pl = P.Planner(w.vehicle, cost, dict(w.integ, dt=0.04, substeps=S, method=P.PLAN_RK4), Kw, N,
                   T.W, T.H)
    cm = None
    if costmap:
        cm = torch.from_numpy(np.random.default_rng(8).uniform(0, 3, T.height.shape)
                              .astype(np.float32)).cuda()
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res, cm)
    for start in (st, np.concatenate([[cost["goal_x"], cost["goal_y"]], st[2:]])):
        wide = run(pl, start, u, Kw, N, None, 4, 64)
        same(run(pl, start, u, Kw, N, None, 2, 256), wide, "general step")
        for K in (5, 64, 1500):
            for lanes, block in ((2, 64), (2, 256), (4, 64), (4, 256), (0, 0)):
                got = run(pl, start, u, K, N, None, lanes, block)
                same(got, (wide[0][:K], wide[1][:, :K]), f"K={K} lanes={lanes} block={block}")
    # chunks
    K = 200
    ud = torch.from_numpy(np.ascontiguousarray(u[:, :, :K])).cuda()
    wide = run(pl, st, u, Kw, N, None, 4, 64)
    J, fs = torch.empty(K, device="cuda"), torch.empty(13, K, device="cuda")
    pl.init_state(st, fs, J)
    for n0, n1 in ((0, N // 2), (N // 2, N)):
        pl.rollout_chunk(fs, J, ud, n0, n1, n1 == N)
    torch.cuda.synchronize()
    same((J.cpu().numpy(), fs.cpu().numpy()), (wide[0][:K], wide[1][:, :K]), "chunks")
    pl.close()
