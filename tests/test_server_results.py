"""Server.result from several host threads at once, as a program may read
finished requests: each call returns its own request's record. The library call
is replaced by one that lets another thread run before it returns, as the real
one does (the interpreter's lock is released during it)."""
import ctypes
import threading

from paper_2603_20525_amd import plan as P


def test_results_read_by_several_threads_are_their_own():
    both = threading.Barrier(2, timeout=20)

    def library_result(handle, rid, ref):
        res = ctypes.cast(ref, ctypes.POINTER(P.Result)).contents
        both.wait()
        if rid == 2:
            first.wait(20)
        res.status, res.best_k, res.best_cost = 1, rid, float(rid)
        if rid == 1:
            first.set()
            second.wait(20)  # the other thread's record is written meanwhile
        else:
            second.set()
        return P.PLAN_OK

    first, second = threading.Event(), threading.Event()
    srv = P.Server.__new__(P.Server)
    srv.h, srv._keep = None, {}
    srv._res = P.Result()
    srv._refs = None, None, ctypes.byref(srv._res)
    srv._calls = None, library_result
    got = {}
    threads = [threading.Thread(target=lambda r=r: got.update({r: srv.result(r)})) for r in (1, 2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(30)
    assert {r: got[r]["best_k"] for r in got} == {1: 1, 2: 2}
