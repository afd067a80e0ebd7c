"""The softmin's three forms (one, two and four plan entries a workgroup, chosen
by the horizon) against float64, at the horizons where the choice changes and at
candidate counts at, under and over a pass of 8 192."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 127, 128, 129, 256, 257, 300])
@pytest.mark.parametrize("K", [1, 63, 1025, 8192, 8193, 20000])
def test_weighted_mean(N, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(K * 1000 + N)
    pl = P.Planner(inputs.WORKLOAD_VEHICLE, inputs.BASE_COST, inputs.BASE_INTEG, K, N, 8, 8)
    u = rng.normal(0, 0.3, (N, 2, K)).astype(np.float32)
    J = rng.uniform(50, 60, K).astype(np.float32)
    if K > 8:
        J[3], J[K // 2] = np.inf, np.nan
    lam = 2.0
    plan = torch.full((N, 2), -7.0, device="cuda")
    k, jb = pl.select(torch.from_numpy(u).cuda(), torch.from_numpy(J).cuda(), plan,
                      P.PLAN_SOFTMIN, lam)
    ok = np.isfinite(J)
    best = int(np.flatnonzero(ok)[np.argmin(J[ok])])
    assert (k, np.float32(jb)) == (best, J[best])
    w = np.where(ok, np.exp(-(np.where(ok, J, np.inf).astype(np.float64) - J[best]) / lam), 0.0)
    lim = np.array([inputs.WORKLOAD_VEHICLE["delta_rate_max"], 1.0])[None, :, None]
    c = np.clip(u.astype(np.float64), -lim, lim)
    want = (c * w).sum(2) / w.sum()
    # a thread's chain, its wave's tree and sixteen waves: (K / 1024 + 6 + 16)
    # roundings of sums of |w c|, twice (numerator, denominator), and the
    # exponential's few ulps
    tol = (2 * (K / 1024 + 22) + 8) * 2.0 ** -23 * ((np.abs(c) * w).sum(2) / w.sum())
    assert (np.abs(plan.cpu().numpy() - want) <= tol).all()
    pl.close()
