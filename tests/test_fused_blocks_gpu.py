"""Workgroup sizes of launches that also select: one wave a workgroup where the
steps earn back the selection's cost per workgroup, and the same results in
either."""
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("drawn", [False, True])
@pytest.mark.parametrize("K,N,costmap,block", [
    (4096, 5, False, 256), (4096, 42, False, 256), (4096, 43, False, 64), (2048, 21, False, 256),
    (2048, 22, False, 64), (96, 1, False, 64), (4096, 100, True, 256), (1600, 99, True, 256),
    (1600, 100, True, 64), (4097, 300, False, 256)])
def test_workgroup_by_candidates_and_steps(K, N, costmap, block, drawn):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = inputs.c2(K=8, N=8)
    T = w.terrain
    g = torch.Generator(device="cuda")
    g.manual_seed(K + N)
    pl = P.Planner(w.vehicle, w.cost, w.integ, K, N, T.W, T.H)
    cm = torch.rand(T.H, T.W, generator=g, device="cuda") if costmap else None
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res, cm)
    u = 0.3 * torch.randn(N, 2, K, generator=g, device="cuda")
    spec = P.sample_spec(P.PLAN_SAMPLE_GAUSSIAN, 3, 1, (0.3, 0.3), None, False, N)

    def run():
        J, plan = torch.full((K,), -7.0, device="cuda"), torch.full((N, 2), -7.0, device="cuda")
        best = (pl.rollout_sampled_argmin(w.state0, spec, N, J, plan) if drawn
                else pl.rollout_argmin(w.state0, u, J, plan))
        return best, J, plan

    best, J, plan = run()
    assert pl.get_launch() == (4, block)
    for hand in (64, 256):
        pl.set_launch(4, hand)
        bh, Jh, ph = run()
        assert bh == best and torch.equal(Jh, J) and torch.equal(ph, plan)
    pl.close()
