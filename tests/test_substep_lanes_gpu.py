"""Lanes that launches of several substeps an interval take between the sizes at
which one lane gives every SIMD a wave and 65 536 candidates, and their results
against one and two lanes set by hand."""
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("costmap", [False, True])
@pytest.mark.parametrize("K,S,lanes", [(32768, 5, 2), (32769, 1, 1), (32769, 2, 2),
                                       (32769, 3, 2), (40003, 5, 2), (65535, 4, 2),
                                       (65536, 4, 1)])
def test_given_controls(K, S, lanes, costmap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    N = 3
    w = inputs.c2(K=8, N=8)
    T = w.terrain
    g = torch.Generator(device="cuda")
    g.manual_seed(K + S)
    pl = P.Planner(w.vehicle, w.cost, dict(w.integ, substeps=S), K, N, T.W, T.H)
    cm = torch.rand(T.H, T.W, generator=g, device="cuda") if costmap else None
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res, cm)
    u = 0.3 * torch.randn(N, 2, K, generator=g, device="cuda")

    def run():
        J, fs = torch.full((K,), -7.0, device="cuda"), torch.full((13, K), -7.0, device="cuda")
        pl.rollout(w.state0, u, J, fs)
        return J, fs

    J, fs = run()
    assert pl.get_launch()[0] == lanes
    assert torch.isfinite(J).any()
    for hand in (1, 2):
        pl.set_launch(hand, 0)
        Jh, fh = run()
        assert torch.equal(J, Jh) and torch.equal(fs, fh)
    pl.close()


@pytest.mark.parametrize("K,S,lanes", [(32769, 1, 2), (32769, 2, 2), (32769, 3, 2), (65535, 1, 2),
                                       (65535, 8, 2), (65536, 1, 1), (65536, 8, 1)])
def test_gradient(K, S, lanes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    N = 4
    w = inputs.c2(K=8, N=8)
    T = w.terrain
    g = torch.Generator(device="cuda")
    g.manual_seed(K + S)
    pl = P.Planner(w.vehicle, w.cost, dict(w.integ, substeps=S), K, N, T.W, T.H)
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res)
    u = 0.3 * torch.randn(N, 2, K, generator=g, device="cuda")

    def run():
        J, gr = torch.full((K,), -7.0, device="cuda"), torch.full((N, 2, K), -7.0, device="cuda")
        pl.rollout_grad(w.state0, u, J, gr, None, 3)
        return J, gr

    J, gr = run()
    assert pl.get_launch()[0] == lanes and gr.any()
    for hand in (1, 2):
        pl.set_launch(hand, 0)
        Jh, gh = run()
        assert torch.equal(J, Jh) and torch.equal(gr, gh)
    pl.close()


@pytest.mark.parametrize("costmap", [False, True])
@pytest.mark.parametrize("K,S,lanes", [(32769, 1, 1), (32769, 2, None), (41313, 10, 2),
                                       (57280, 3, 2), (57281, 3, 1), (65535, 3, 1)])
def test_other_forms(K, S, lanes, costmap):
    """Selection, chunks and drawn controls: two lanes below seven eighths of a
    wave per SIMD of one lane each (57 344 candidates on 1 024 of them), except
    two substeps without a costmap."""
    lanes = lanes or (2 if costmap else 1)
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    N = 3
    w = inputs.c2(K=8, N=8)
    T = w.terrain
    g = torch.Generator(device="cuda")
    g.manual_seed(K + S)
    pl = P.Planner(w.vehicle, w.cost, dict(w.integ, substeps=S), K, N, T.W, T.H)
    cm = torch.rand(T.H, T.W, generator=g, device="cuda") if costmap else None
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res, cm)
    pl.set_order(P.PLAN_ORDER_OFF)
    u = 0.3 * torch.randn(N, 2, K, generator=g, device="cuda")
    spec = P.sample_spec(P.PLAN_SAMPLE_GAUSSIAN, 5, 6, (0.3, 0.3), None, False, N)

    def run(expect=None):
        out = []
        J = torch.full((K,), -7.0, device="cuda")
        plan = torch.full((N, 2), -7.0, device="cuda")
        best = pl.rollout_argmin(w.state0, u, J, plan)
        out += [J, plan, torch.tensor(best, dtype=torch.float64)]
        assert expect is None or pl.get_launch()[0] == expect
        J = torch.full((K,), -7.0, device="cuda")
        pl.rollout_sampled(w.state0, spec, N, J)
        out.append(J)
        assert expect is None or pl.get_launch()[0] == expect
        x, J = torch.empty(13, K, device="cuda"), torch.empty(K, device="cuda")
        pl.init_state(w.state0, x, J)
        pl.rollout_chunk(x, J, u, 0, 2, False)
        pl.rollout_chunk(x, J, u, 2, N, True)
        assert expect is None or pl.get_launch()[0] == expect
        return out + [x, J]

    got = run(lanes)
    assert torch.isfinite(got[0]).any()
    for hand in (1, 2):
        pl.set_launch(hand, 0)
        for a, b in zip(got, run()):
            assert torch.equal(a, b)
    pl.close()


@pytest.mark.parametrize("K,N,costmap,plain,fused",
                         [(32769, 99, False, (1, 64), (1, 256)), (32769, 100, True, (1, 64), (1, 64)),
                          (49152, 128, True, (1, 64), (1, 64)), (49153, 127, True, (1, 64), (1, 64)),
                          (49153, 128, True, (2, 64), (2, 64)), (49153, 128, False, (1, 64), (1, 64)),
                          (57280, 128, True, (2, 64), (2, 64)), (57281, 128, True, (1, 256), (1, 256)),
                          (65536, 3, False, (1, 256), (1, 256))])
def test_one_substep(K, N, costmap, plain, fused):
    """Lanes and threads of one substep an interval, in one launch, with selection
    and in chunks (as without selection, but never two lanes), on 1 024 SIMDs."""
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

    def run(expect=None):
        J, fs = torch.full((K,), -7.0, device="cuda"), torch.full((13, K), -7.0, device="cuda")
        pl.rollout(w.state0, u, J, fs)
        assert expect is None or pl.get_launch() == plain
        Ja, plan = torch.full((K,), -7.0, device="cuda"), torch.full((N, 2), -7.0, device="cuda")
        best = pl.rollout_argmin(w.state0, u, Ja, plan)
        assert expect is None or pl.get_launch() == fused
        x, Jc = torch.empty(13, K, device="cuda"), torch.empty(K, device="cuda")
        pl.init_state(w.state0, x, Jc)
        for n in range(0, N, 50):
            pl.rollout_chunk(x, Jc, u, n, min(N, n + 50), n + 50 >= N)
        assert expect is None or pl.get_launch() == (1, plain[1])
        return J, fs, Ja, plan, torch.tensor(best, dtype=torch.float64), x, Jc

    got = run(True)
    assert torch.isfinite(got[0]).any()
    for hand in ((1, 64), (1, 256), (2, 64)):
        pl.set_launch(*hand)
        for a, b in zip(got, run()):
            assert torch.allclose(a, b, rtol=0.0, atol=0.0, equal_nan=True)
    pl.close()
