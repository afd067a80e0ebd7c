"""Ticks of several rounds of workgroups: the entries run longest first and
every second round in reverse, and each request's result is still the plain
path's, bit for bit, with and without costmaps among them (ticks without any
take kernels that leave the cost channel out)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu


# workgroups of the tick: under one round, one and a part, two and a part, four
# (reversed rounds are whole ones only)
@pytest.mark.parametrize("n_req,K", [(3, 500), (18, 4096), (40, 4096), (64, 4100)])
@pytest.mark.parametrize("costmaps", [0, 1, 2])  # none, every third, all
def test_results_identical_to_plain_path(n_req, K, costmaps):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = inputs.c2(K=K, N=24)
    T = w.terrain
    h = torch.from_numpy(T.height).cuda()
    rng = np.random.default_rng(n_req)
    cm = torch.from_numpy(rng.uniform(0, 2, T.height.shape).astype(np.float32)).cuda()
    u = torch.from_numpy(np.ascontiguousarray(w.controls)).cuda()
    pl = P.Planner(w.vehicle, w.cost, w.integ, K, w.N, T.W, T.H)
    srv = P.Server(w.vehicle, n_req, K, w.N, T.W, T.H, 1 << 36, 16)
    want, got = [], []
    for i in range(n_req):
        N = int(rng.integers(1, w.N + 1))
        c = cm if costmaps == 2 or (costmaps == 1 and i % 3 == 0) else None
        ui = (u[:N] * (1.0 - 0.01 * i)).contiguous()
        J, plan = torch.empty(K, device="cuda"), torch.empty(N, 2, device="cuda")
        pl.set_terrain(h, T.x0, T.y0, T.res, c)
        want.append((pl.rollout_argmin(w.state0, ui, J, plan), J, plan))
        Js, out = torch.empty(K, device="cuda"), torch.zeros(N, 2, device="cuda")
        got.append((srv.submit(h, T.x0, T.y0, T.res, w.state0, ui, w.cost, w.integ, out, c, Js),
                    Js, out))
    srv.drain()
    torch.cuda.synchronize()
    for ((k, jb), J, plan), (rid, Js, out) in zip(want, got):
        res = srv.result(rid)
        assert res["status"] == 1 and res["best_k"] == k
        assert np.float32(res["best_cost"]) == np.float32(jb)
        assert torch.equal(Js, J) and torch.equal(out, plan)
    srv.close()
    pl.close()
