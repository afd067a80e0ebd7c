"""The serial backward pass of the adjoint, which launches of more than 24
candidates per compute unit take: its one-, two- and four-lane kernels have the
same bits, as do all checkpoint intervals, and agree with FP64 central finite
differences of the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402
from tests.test_adjoint_gpu import compare_fd, gpu_grad, setup  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P.lib()
    yield
    torch.cuda.synchronize()


def many():
    return 24 * torch.cuda.get_device_properties(0).multi_processor_count + 1


@pytest.mark.parametrize("N,S,C", [(100, 1, 10), (7, 6, 3)])
def test_lanes_change_no_bit_and_gradients_match_differences(N, S, C):
    w = inputs.c2(K=many(), N=N)
    w.integ = dict(w.integ, substeps=S)
    pl, o = setup(w)
    J, g = gpu_grad(pl, w, w.controls, ckpt=C)
    for lanes in (1, 2, 4):
        for block in (64, 256):
            pl.set_launch(lanes, block)
            Jl, gl = gpu_grad(pl, w, w.controls, ckpt=C)
            np.testing.assert_array_equal(Jl, J)
            np.testing.assert_array_equal(gl, g)
    pl.set_launch(0, 0)
    ks = np.argsort(J, kind="stable")[:12]
    worst, used, skipped = compare_fd(o, w, w.controls, g, ks, n_entries=12,
                                      label=f"serial N={N} S={S}")
    print(f"{used} entries, worst {worst:.3g} x tol, {skipped} skipped")
    assert used >= 0.75 * 12 * 12
    pl.close()


@pytest.mark.parametrize("lanes", [1, 2, 4])
def test_checkpoint_interval_changes_no_bit(lanes):
    w = inputs.c2(K=many(), N=40)
    pl, _ = setup(w)
    pl.set_launch(lanes, 64)
    J, g = gpu_grad(pl, w, w.controls, ckpt=10)
    assert np.isfinite(g).all() and g.any()
    for c in (1, 7, 40, 1000):
        Jc, gc = gpu_grad(pl, w, w.controls, ckpt=c)
        np.testing.assert_array_equal(Jc, J)
        np.testing.assert_array_equal(gc, g)
    pl.close()


@pytest.mark.parametrize("K,lanes", [(16384, 4), (16385, 2), (32768, 2), (32769, 2), (65536, 1), (70001, 1)])
def test_automatic_lanes_equal_the_smallest_launch(K, lanes):
    """Candidates of any launch of the serial pass have one gradient."""
    N, Km = 12, many()
    w = inputs.c2(K=8, N=N)
    T = w.terrain
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    pl = P.Planner(w.vehicle, w.cost, w.integ, K, N, T.W, T.H)
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res)
    u = 0.3 * torch.randn(N, 2, K, generator=g, device="cuda")
    weight = torch.rand(K, generator=g, device="cuda")

    def grad(cols):
        part, wt = u[:, :, cols].contiguous(), weight[cols].contiguous()
        J, gr = torch.empty(part.shape[2], device="cuda"), torch.empty_like(part)
        pl.rollout_grad(w.state0, part, J, gr, wt, 5)
        return J, gr

    J, gr = grad(slice(0, K))
    assert pl.get_launch()[0] == lanes
    Jf, gf = grad(slice(0, Km))
    Jb, gb = grad(slice(K - Km, K))
    assert torch.equal(J[:Km], Jf) and torch.equal(gr[:, :, :Km], gf)
    assert torch.equal(J[K - Km:], Jb) and torch.equal(gr[:, :, K - Km:], gb)
    assert gr.any() and torch.isfinite(gr).all()
    pl.close()
