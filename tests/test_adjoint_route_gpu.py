"""Which backward pass a gradient takes depends on the candidates, the intervals
and the substeps alone: the caller's checkpoint interval changes no bit of it,
also near the longest horizons whose segments still fit on chip."""
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


def planner(K, N, S, dt):
    w = inputs.c2(K=K, N=8)
    T = w.terrain
    pl = P.Planner(w.vehicle, w.cost, dict(w.integ, substeps=S, dt=dt), K, N, T.W, T.H)
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res)
    g = torch.Generator(device="cuda")
    g.manual_seed(N + S)
    return pl, w.state0, 0.2 * torch.randn(N, 2, K, generator=g, device="cuda")


def grad(pl, s0, u, C):
    N, _, K = u.shape
    J, g = torch.empty(K, device="cuda"), torch.full((N, 2, K), -7.0, device="cuda")
    pl.rollout_grad(s0, u, J, g, None, C)
    return J, g


# both sides of 4.3 substeps an interval (where only one interval fits the 160
# steps of a segment) and of 110 277 steps, substeps that leave a segment short,
# and more than fit one
@pytest.mark.parametrize("N,S", [(1, 160), (6, 160), (689, 160), (690, 160), (500, 100),
                                 (430, 100), (431, 100), (5000, 50), (3000, 53), (40, 161),
                                 (20000, 2), (700, 3)])
def test_checkpoint_interval_changes_no_bit(N, S):
    pl, s0, u = planner(16, N, S, 2.0 / N)
    J, g = grad(pl, s0, u, 1)
    assert torch.isfinite(J).all() and torch.isfinite(g).all() and g.any()
    for C in (2, 3, 5, 40, N):
        Jc, gc = grad(pl, s0, u, C)
        assert torch.equal(Jc, J) and torch.equal(gc, g), C
    pl.close()


# a few steps of many candidates, few but long segments
@pytest.mark.parametrize("N,S", [(1, 1), (4, 1), (5, 1), (20, 1), (2, 160), (5, 100)])
def test_sizes_the_parallel_pass_is_slow_at_take_the_serial_one(N, S):
    """Their gradients are the bits of a launch of more candidates, which always
    takes the serial pass."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    pl, s0, u = planner(24 * units + 8, N, S, 0.02)
    want = grad(pl, s0, u, 10)
    for K in (24 * units, 16 * units + 1):
        J, g = grad(pl, s0, u[:, :, :K].contiguous(), 10)
        assert torch.equal(J, want[0][:K]) and torch.equal(g, want[1][:, :, :K])
    assert want[1].any()
    pl.close()
