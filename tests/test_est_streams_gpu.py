"""Launches that share their steps between the waves use one hand-off per context:
those on different streams, also on streams destroyed with their launch pending
(whose handles may come back), follow one another and each returns its own
results."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import plan as P  # noqa: E402
from tests.test_est_ahead_gpu import many, narrow  # noqa: E402

pytestmark = pytest.mark.gpu


def problem(n):
    """A context, n different sets of controls, their outputs, and the results
    of unshared launches."""
    pl, st, u, K, simds = many(3, 121, 8, 6)
    us = [u * (1.0 - 0.1 * i) for i in range(n)]
    want = [narrow(pl, st, v, simds) for v in us]
    outs = [(torch.full((K,), -7.0, device="cuda"), torch.full((7, K), -7.0, device="cuda"))
            for _ in us]
    torch.cuda.synchronize()
    return pl, st, us, outs, want


def check(pl, outs, want):
    torch.cuda.synchronize()
    for (J, fs), (Jw, fw) in zip(outs, want):
        assert torch.equal(J, Jw) and torch.equal(fs, fw)
    pl.close()


def test_streams_in_turn_without_waits():
    pl, st, us, outs, want = problem(9)
    streams = [torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.default_stream()]
    for i, (u, out) in enumerate(zip(us, outs)):
        P.plan_set_stream(pl.ctx, streams[i % 3])
        pl.rollout_est(st, u, *out)
    check(pl, outs, want)


def test_streams_destroyed_with_their_launch_pending():
    pl, st, us, outs, want = problem(9)
    with open("/proc/self/maps") as f:  # the HIP runtime that is loaded already
        hip = ctypes.CDLL(next(ln.split()[-1] for ln in f if "libamdhip64" in ln))
    for u, out in zip(us, outs):
        s = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(s)) == 0
        P.plan_set_stream(pl.ctx, s.value)
        pl.rollout_est(st, u, *out)
        P.plan_set_stream(pl.ctx, 0)
        assert hip.hipStreamDestroy(s) == 0
    check(pl, outs, want)


def test_shared_beside_a_replayed_graph():
    """A captured launch keeps no shared state, so a replay beside a shared
    launch changes neither."""
    pl, st, us, outs, want = problem(2)
    side = torch.cuda.Stream()
    P.plan_set_stream(pl.ctx, side)
    pl.rollout_est(st, us[0], *outs[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        pl.rollout_est(st, us[1], *outs[1])
    P.plan_set_stream(pl.ctx, 0)
    for _ in range(3):
        for J, fs in outs:
            J.fill_(-7.0)
            fs.fill_(-7.0)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay()
        pl.rollout_est(st, us[0], *outs[0])
        torch.cuda.synchronize()
        for (J, fs), (Jw, fw) in zip(outs, want):
            assert torch.equal(J, Jw) and torch.equal(fs, fw)
    pl.close()
