"""Gradients of candidates that reach the goal early: the parallel backward pass
ends with the last step that one of a workgroup's four takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def grads(N, S, reach, sizes, C=10):
    """Of the same candidates in launches of several sizes; the goal is about
    `reach` intervals away, and the last quarter of them brakes."""
    w = inputs.c2(K=8, N=8)
    T = w.terrain
    s0 = np.array(w.state0, np.float32)
    dt = 0.02 * S
    ahead = float(s0[6]) * dt * reach + 0.05
    goal_r = 0.3 if reach else 0.2
    cost = dict(w.cost, goal_x=float(s0[0]) + ahead * np.cos(float(s0[3])),
                goal_y=float(s0[1]) + ahead * np.sin(float(s0[3])), goal_r=goal_r)
    Kw = max(sizes)
    pl = P.Planner(w.vehicle, cost, dict(w.integ, substeps=S, dt=dt), Kw, N, T.W, T.H)
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res)
    g = torch.Generator(device="cuda")
    g.manual_seed(N + S)
    u = 0.05 * torch.randn(N, 2, Kw, generator=g, device="cuda")
    u[:, 1, 3::4] = -0.5
    out = []
    for K in sizes:
        # what workgroups that take every step leave on the chip is not read
        pl.set_cost(dict(cost, goal_x=1e6))
        n = 4 * torch.cuda.get_device_properties(0).multi_processor_count
        pl.rollout_grad(s0, u[:, :, :n].contiguous(), torch.empty(n, device="cuda"),
                        torch.empty(N, 2, n, device="cuda"), None, C)
        pl.set_cost(cost)
        J, G = torch.full((K,), -7.0, device="cuda"), torch.full((N, 2, K), -7.0, device="cuda")
        pl.rollout_grad(s0, u[:, :, :K].contiguous(), J, G, None, C)
        out.append((J.cpu().numpy(), G.cpu().numpy()))
    pl.close()
    return out


# arrivals at once, inside, at and after a batch of sixteen steps, and horizons
# of one window of recomputed states and of several, some without a step
@pytest.mark.parametrize("N,S,reach", [(40, 1, 0), (40, 1, 5), (40, 1, 16), (60, 1, 31),
                                       (20, 3, 6), (20, 3, 9), (9, 17, 2), (4, 160, 1),
                                       (400, 1, 0), (400, 1, 12), (400, 1, 60)])
def test_equals_the_serial_pass(N, S, reach):
    units = torch.cuda.get_device_properties(0).multi_processor_count
    sizes = [24 * units + 8, 4 * units - 3, 9]
    (Jw, Gw), *few = grads(N, S, reach, sizes)
    assert np.isfinite(Jw).any()
    frozen = (Gw[-1] == 0).all(axis=0)
    assert frozen.any() and (reach > 0) == Gw.any()
    # two float32 evaluations of the same products: 64 roundings a step, each of
    # the candidate's largest entry
    tol = 64 * N * S * 2.0 ** -24
    for (J, G), K in zip(few, sizes[1:]):
        r = Gw[:, :, :K]
        np.testing.assert_array_equal(J, Jw[:K])
        assert np.array_equal(G == 0, r == 0)
        assert (np.abs(G - r).max(axis=(0, 1)) <= tol * np.abs(r).max(axis=(0, 1))).all()



@pytest.mark.parametrize("N,S", [(1, 1), (17, 1), (40, 1), (9, 17), (400, 1)])
def test_candidates_without_a_finite_cost(N, S):
    """Whole workgroups of them, some with one that has, and some without: zeros,
    and the others' gradients as if they were not there."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    w = inputs.c2(K=8, N=8)
    T = w.terrain
    Kw = 24 * units + 8
    pl = P.Planner(w.vehicle, w.cost, dict(w.integ, substeps=S, dt=0.01 * S), Kw, N, T.W, T.H)
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res)
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    u = 0.05 * torch.randn(N, 2, Kw, generator=g, device="cuda")
    bad = torch.zeros(Kw, dtype=torch.bool, device="cuda")
    bad[:20] = True
    bad[20:40:4] = True
    bad[41:60] = True

    def grad(u, K):
        J, G = torch.full((K,), -7.0, device="cuda"), torch.full((N, 2, K), -7.0, device="cuda")
        pl.rollout_grad(w.state0, u[:, :, :K].contiguous(), J, G, None, 10)
        return J, G

    ub = u.clone()
    ub[N // 2, 1, bad] = float("nan")
    for K in (19, 41, 4 * units - 1, Kw):
        J, G = grad(u, K)
        Jb, Gb = grad(ub, K)
        b = bad[:K]
        assert torch.isfinite(J).all() and G.any()
        assert torch.isinf(Jb[b]).all() and not Gb[:, :, b].any()
        assert torch.equal(Jb[~b], J[~b]) and torch.equal(Gb[:, :, ~b], G[:, :, ~b])
    pl.close()

# (rounds of one workgroup a compute unit, intervals, substeps)
@pytest.mark.parametrize("rounds,N,S", [(2, 12, 1), (3, 24, 1), (4, 32, 1), (6, 60, 1),
                                        (4, 10, 3), (6, 8, 10)])
def test_short_horizons_of_many_take_the_serial_pass(rounds, N, S):
    """Where the serial pass skips most of few steps, several rounds of the
    parallel one lose: those launches have the serial pass's bits."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    sizes = [24 * units + 8, 4 * units * rounds]
    (Jw, Gw), (J, G) = grads(N, S, 4 if S < 4 else 1, sizes)
    assert Gw.any()
    np.testing.assert_array_equal(J, Jw[:sizes[1]])
    np.testing.assert_array_equal(G, Gw[:, :, :sizes[1]])
