"""fwh_plan_info names the panel ranges that the FP64 gather sums separately: several on
a surface whose observer tiles alone leave the device idle, one where the delay windows are
too wide for the tiled gather; an FP64 plan still takes no choice of them."""
import pytest

from gpu_common import make_plan
from workloads import configs, surfaces

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtau,N,several", [(1 / 16, 200, True), (1 / 2000, 3000, False)])
def test_info_of_an_fp64_plan(dtau, N, several):
    import paper_2312_16263_amd as fwh
    c = configs.Case("splits", surfaces.sphere(1.0, 32, 64), surfaces.observer_circle(8, 10.0, step_deg=45.0), 0.4, 8.0,
                     dtau, N)
    kind, splits = make_plan(c, "f64").info()
    print(f"[fp64 splits] dtau={dtau} N={N}: {splits}", flush=True)
    assert kind == "f64"
    assert 1 < splits <= c.n_panels // 16 if several else splits == 1
    with pytest.raises(fwh.FwhError):
        make_plan(c, "f64", splits=2)
