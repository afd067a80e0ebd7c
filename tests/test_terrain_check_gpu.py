"""plan_set_terrain's check of the heights and the costmap: a non-finite node
anywhere is refused, and the next valid terrain is taken again."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2603_20525_amd import inputs  # noqa: E402
from paper_2603_20525_amd import plan as P  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(2, 2), (17, 16), (300, 211)])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_non_finite_nodes_are_refused(W, H, value):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pl = P.Planner(inputs.WORKLOAD_VEHICLE, inputs.BASE_COST, inputs.BASE_INTEG, 8, 8, W, H)
    good = torch.zeros(H, W, device="cuda")
    for at in ((0, 0), (H - 1, W - 1), (H // 2, W // 3)):
        bad = good.clone()
        bad[at] = float(value)
        for h, cm in ((bad, None), (bad, good), (good, bad)):
            with pytest.raises(P.PlanError):
                pl.set_terrain(h, 0.0, 0.0, 0.1, cm)
            pl.set_terrain(good, 0.0, 0.0, 0.1, good)
    pl.close()
