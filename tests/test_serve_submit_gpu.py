"""Server.submit packs the request in one call where that reproduces the
struct's own conversions, and goes field by field where it does not."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ready():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = inputs.c2(K=100, N=5)
    T = w.terrain
    srv = P.Server(w.vehicle, 4, 100, 5, T.W, T.H, 1 << 30)
    h = torch.from_numpy(T.height).cuda()
    u = torch.from_numpy(np.ascontiguousarray(w.controls)).cuda()
    yield w, srv, h, u
    srv.close()


def submit(ready, **kw):
    w, srv, h, u = ready
    T = w.terrain
    a = dict(height=h, x0=T.x0, y0=T.y0, res=T.res, state0=w.state0, controls=u, cost=w.cost,
             integ=w.integ, plan=torch.zeros(5, 2, device="cuda"))
    a.update(kw)
    rid = srv.submit(**a)
    srv.drain()
    return srv.result(rid)


@pytest.mark.parametrize("convert", [list, tuple, np.asarray, lambda s: [np.float32(v) for v in s]])
def test_state_types_give_one_result(ready, convert):
    want = submit(ready)
    got = submit(ready, state0=convert(ready[0].state0))
    assert want["status"] == 1
    assert (got["best_k"], got["best_cost"]) == (want["best_k"], want["best_cost"])
    assert set(got) == {"status", "best_k", "best_cost", "slot", "t_submit", "t_admit", "t_done"}


def test_refused_as_by_fields(ready):
    with pytest.raises(P.PlanError):  # beyond float32: infinite, refused by the library
        submit(ready, x0=1e39)
    with pytest.raises(P.PlanError):
        submit(ready, state0=[float("nan")] * 13)
    with pytest.raises(ValueError):
        submit(ready, state0=[0.0] * 12)
    with pytest.raises(ValueError):
        submit(ready, plan=torch.zeros(4, 2, device="cuda"))
    with pytest.raises(P.PlanError):
        submit(ready, res=0.0)
    assert submit(ready, x0="0.0")["status"] == 1  # float() of a string, as ever


def test_changed_parameters_are_seen(ready):
    w = ready[0]
    cost = dict(w.cost)
    a = submit(ready, cost=cost)
    cost["w_g"] = cost["w_g"] * 3
    b = submit(ready, cost=cost)
    assert a["best_cost"] != b["best_cost"]
