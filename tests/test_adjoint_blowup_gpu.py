"""Gradients of candidates whose motion or adjoint comes near the end of float's
range, which the parallel backward pass hands to the serial steps: those that the
final state tells, which the first workgroups of the launch take, and those that
only the adjoint tells, pulled back again at the end. Either has the bits of the
serial pass, which the same candidates get in a launch of many."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu

WILD = 1e18  # rates from which a final state counts as blown up


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


class Problem:
    def __init__(self, component, value, N, S, dt, costmap=False, rough=None):
        self.many = 24 * torch.cuda.get_device_properties(0).multi_processor_count + 56
        w = inputs.c2(K=8, N=8)
        T = w.terrain
        self.pl = P.Planner(w.vehicle, w.cost, dict(w.integ, substeps=S, dt=dt), self.many, N,
                            T.W, T.H)
        g = torch.Generator(device="cuda")
        g.manual_seed(N)
        self.u = 0.3 * torch.randn(N, 2, self.many, generator=g, device="cuda")
        cm = torch.rand(T.H, T.W, generator=g, device="cuda") if costmap else None
        self.s0 = np.array(w.state0, np.float32)
        if rough is None:
            self.pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res, cm)
        else:
            h = rough * torch.rand(T.H, T.W, generator=g, device="cuda")
            self.pl.set_terrain(h, 0.0, 0.0, 0.1)
            self.s0[:] = [25, 25, 0.9, 0.3, 0, 0, 8] + [0] * 6
        self.s0[component] = value

    def grad(self, u, weight=None, every=7):
        J, g = torch.empty(u.shape[2], device="cuda"), torch.full_like(u, -7.0)
        self.pl.rollout_grad(self.s0, u, J, g, weight, every)
        return J, g


def bits(t):
    return torch.nan_to_num(t, nan=12345.0, posinf=3e38, neginf=-3e38)


# horizons within one window of states and over two; a start that spins or
# pitches so that some candidates blow up
@pytest.mark.parametrize("costmap", [False, True])
@pytest.mark.parametrize("component,value,N,S,dt", [(10, 30.0, 40, 1, 0.02),
                                                    (9, 20.0, 170, 1, 0.01),
                                                    (9, 20.0, 90, 2, 0.04)])
def test_blown_up_by_the_final_state(component, value, N, S, dt, costmap):
    p = Problem(component, value, N, S, dt, costmap)
    J, fs = torch.empty(p.many, device="cuda"), torch.empty(13, p.many, device="cuda")
    p.pl.rollout(p.s0, p.u, J, fs)
    wild = torch.isfinite(J) & ~(fs[6:12].abs().amax(0) < WILD)
    w, rest = torch.nonzero(wild).flatten(), torch.nonzero(~wild).flatten()
    assert len(w) > 4  # more than one workgroup of the front pulls back at a time
    Jm, gm = p.grad(p.u)
    assert torch.equal(Jm, J)
    # many in a row (several times four in one workgroup's 32), alone, at the end
    order = torch.cat([rest[:3], w[:37], rest[3:60], w[-2:], rest[60:61], w[:1]])
    for K in (len(order), len(order) - 1, 41):
        k = order[:K]
        Jk, gk = p.grad(p.u[:, :, k].contiguous())
        assert torch.equal(Jk, J[k])
        is_wild = wild[k]
        assert torch.equal(bits(gk[:, :, is_wild]), bits(gm[:, :, k][:, :, is_wild]))
        # the others: rounding may grow without bound, their infinities and NaN not
        assert torch.equal(torch.isfinite(gk), torch.isfinite(gm[:, :, k]))
        g = gk[:, :, is_wild]
        assert bool((torch.isfinite(g) & (g != 0)).any())
    p.pl.close()


@pytest.mark.parametrize("N,S", [(40, 1), (200, 1), (20, 9), (400, 2)])
def test_blown_up_by_the_adjoint(N, S):
    """Calm motion whose seeds take the adjoint beyond 1e28."""
    p = Problem(6, 12.0, N, S, min(0.01 * S, 3.0 / N))
    weight = torch.ones(p.many, device="cuda")
    weight[1::3] = 1e30
    weight[5] = float("nan")
    weight[8] = float("inf")
    Jm, gm = p.grad(p.u, weight)
    for K in (3, 33):
        J, g = p.grad(p.u[:, :, :K].contiguous(), weight[:K].contiguous())
        assert torch.equal(J, Jm[:K])
        again = ~(weight[:K] < 1e28)
        assert torch.isfinite(g[:, :, 1]).all() and bool(g[:, :, 1].abs().max() > 1e28)
        assert torch.equal(bits(g[:, :, again]), bits(gm[:, :, :K][:, :, again]))
        # two float32 evaluations of the same products: 64 roundings a step, each
        # of the candidate's largest entry
        ref = gm[:, :, :K][:, :, ~again]
        err = (g[:, :, ~again] - ref).abs().amax((0, 1))
        assert bool((err <= 64 * N * S * 2.0 ** -24 * ref.abs().amax((0, 1))).all())
    p.pl.close()


@pytest.mark.parametrize("vy", [1e4, 1e6, 9e7])
def test_fast_candidates_stay_with_the_parallel_pass(vy):
    """Rates far from any vehicle's but also from the end of float's range."""
    N = 40
    p = Problem(7, vy, N, 1, 0.02, rough=0.1)
    Jm, gm = p.grad(p.u)
    J, g = p.grad(p.u[:, :, :262].contiguous())
    assert torch.equal(J, Jm[:262]) and torch.isfinite(J).all()
    ref = gm[:, :, :262]
    assert torch.isfinite(g).all() and g.any()
    err = (g - ref).abs().amax((0, 1))
    assert bool((err <= 64 * N * 2.0 ** -24 * ref.abs().amax((0, 1))).all())
    p.pl.close()
