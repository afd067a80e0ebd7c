"""Launches of four lanes per candidate with more waves than compute units take
one of two kernels by the size of their controls: the results around that size,
in one piece and in chunks, against one and two lanes set by hand."""
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("costmap", [False, True])
@pytest.mark.parametrize("K,N", [(4097, 85), (4097, 86), (9001, 38), (9001, 39), (16384, 21),
                                 (16384, 22), (16384, 1)])
def test_given_controls(K, N, costmap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = inputs.c2(K=8, N=8)
    T = w.terrain
    g = torch.Generator(device="cuda")
    g.manual_seed(K + N)
    # some candidates reach the goal
    s0 = w.state0
    cost = dict(w.cost, goal_x=float(s0[0] + 0.2 * s0[6]), goal_y=float(s0[1]), goal_r=0.3)
    pl = P.Planner(w.vehicle, cost, w.integ, K, N, T.W, T.H)
    cm = torch.rand(T.H, T.W, generator=g, device="cuda") if costmap else None
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res, cm)
    u = 0.3 * torch.randn(N, 2, K, generator=g, device="cuda")
    u[0, 1, 5] = float("nan")

    def outputs():
        J, fs = torch.full((K,), -7.0, device="cuda"), torch.full((13, K), -7.0, device="cuda")
        pl.rollout(s0, u, J, fs)
        Ja, plan = torch.full((K,), -7.0, device="cuda"), torch.full((N, 2), -7.0, device="cuda")
        best = pl.rollout_argmin(s0, u, Ja, plan)
        Jc, st = torch.empty(K, device="cuda"), torch.empty(13, K, device="cuda")
        pl.init_state(s0, st, Jc)
        for n in range(0, N, 17):
            pl.rollout_chunk(st, Jc, u, n, min(n + 17, N), n + 17 >= N)
        assert torch.equal(J, Ja) and torch.equal(J, Jc)
        assert torch.equal(torch.nan_to_num(fs), torch.nan_to_num(st))
        return best, J, torch.nan_to_num(fs), plan

    first = outputs()
    assert pl.get_launch()[0] == 4 and torch.isfinite(first[1]).any() and torch.isinf(first[1][5])
    for lanes in (1, 2):
        pl.set_launch(lanes, 0)
        other = outputs()
        assert other[0] == first[0]
        assert all(torch.equal(p, q) for p, q in zip(first[1:], other[1:]))
    pl.close()
