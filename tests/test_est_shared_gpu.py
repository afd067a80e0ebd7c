"""Sliding candidates in a launch whose steps the waves share: slip ratios around
and beyond 1, where each wave leaves the short form of the arctangent by itself,
against launches of one wave per SIMD, which always take the long one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402
from tests.test_est_ahead_gpu import narrow  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vy", [11.0, 15.0, -40.0])
@pytest.mark.parametrize("N,S", [(30, 1), (6, 5)])
def test_sliding_candidates_shared_equals_narrow(vy, N, S):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    K = 64 * (simds + 5) - 7
    w = inputs.c2(K=8, N=8)
    T = w.terrain
    s = np.asarray(w.state0, np.float32)
    st = np.array([s[0], s[1], s[3], vy, 0, 0, s[6]], np.float32)
    pl = P.Planner(w.vehicle, w.cost, dict(w.integ, substeps=S), K, N, T.W, T.H)
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res)
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    u = 0.8 * torch.randn(N, 2, K, generator=g, device="cuda")
    u[N // 2, 0, 3] = float("nan")
    want = narrow(pl, st, u, simds)
    J, fs = torch.empty(K, device="cuda"), torch.empty(7, K, device="cuda")
    for _ in range(2):
        J.fill_(-7.0)
        fs.fill_(-7.0)
        pl.rollout_est(st, u, J, fs)
        assert torch.equal(J, want[0])
        assert torch.equal(torch.nan_to_num(fs), torch.nan_to_num(want[1]))
    assert torch.isinf(J[3]) and torch.isfinite(J).any()
    pl.close()
