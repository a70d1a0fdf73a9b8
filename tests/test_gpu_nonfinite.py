"""Values that are not finite, in FP64.  The spline through a record is one linear
system, so a NaN or an infinity in any frame of a panel makes every coefficient of
its series undefined, and with them every sample of every observer (and every
gradient, where dJ/dp' holds one).  The chunked recurrences have to give what the
whole one gives, here the oracle: not the undefined values near the frame alone."""
import numpy as np
import pytest

import oracle
from gpu_common import make_plan, oracle_adjoint, oracle_forward, to_device, valid_mask
from test_gpu_gm import _run_gpu
from workloads import configs, motion, surfaces

pytestmark = pytest.mark.gpu


def _case(N, dtau=1 / 16, P=70, O=3):
    surf = surfaces.sphere(1.0, 16, 32).subset(np.arange(3, 3 + P))
    return configs.Case(f"nonfinite_N{N}", surf, surfaces.observer_circle(O, 10.0, step_deg=120.0), 0.4, 8.0, dtau, N,
                        kind="dipole", omega=2.0)


# the last case's delay windows (one sphere at a high frame rate) are too wide for the tiled gather
@pytest.mark.parametrize("N,dtau,frame,panel", [(300, 1 / 16, 0, 0), (300, 1 / 16, 150, 65), (300, 1 / 16, 299, 69),
                                                (67, 1 / 16, 33, 1), (3000, 1 / 2000, 1500, 12)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_fp64_forward(N, dtau, frame, panel, value):
    import torch
    c = _case(N, dtau)
    rho, u, pp = c.data()
    bad = rho.copy()
    bad[frame, panel] = value
    print(f"[nonfinite] forward N={N} frame={frame} panel={panel} {value}", flush=True)
    ref, _, nt = oracle_forward(c, bad, u, pp)
    plan = make_plan(c, "f64")
    good = plan.forward(*to_device((rho, u, pp))).clone()
    p = plan.forward(*to_device((bad, u, pp))).cpu().numpy()
    valid = valid_mask(nt, p.shape[1]) > 0
    assert not np.isfinite(ref[valid]).any()
    assert not np.isfinite(p[valid]).any()
    assert np.all(p[~valid] == 0.0)
    # and leaves nothing behind for the next call
    assert torch.equal(plan.forward(*to_device((rho, u, pp))), good)


@pytest.mark.parametrize("sample", [0, 100])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_fp64_adjoint(sample, value):
    import torch
    c = _case(300)
    data = c.data()
    plan = make_plan(c, "f64")
    d = to_device(data)
    p = plan.forward(*d)
    good = plan.adjoint(*d, 2 * p)
    gbar = 2 * p
    gbar[1, sample] = value
    print(f"[nonfinite] adjoint sample={sample} {value}", flush=True)
    ref = oracle_adjoint(c, *data, gbar.cpu().numpy())
    for a, b in zip(plan.adjoint(*d, gbar), ref):
        assert not np.isfinite(b).any()
        assert not torch.isfinite(a).any()
    for a, b in zip(plan.adjoint(*d, 2 * p), good):
        assert torch.equal(a, b)


@pytest.mark.parametrize("N,frame,panel", [(131, 0, 0), (131, 70, 14), (131, 130, 3), (34, 20, 7), (700, 400, 9)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_general_motion(N, frame, panel, value):
    body = surfaces.sphere(1.0, 3, 5)
    dtau = max(1 / 64, 2.0 / N)
    ms = motion.moving_surface(body, "orbit", N, dtau, 0.1, spin=0.5)
    rho, u, pp = motion.quiescent_monopole_series(ms, 0.3, 0.01, 6.0, dtau, 0.1, source=(0.05, 0.02, 0.0))
    rho = rho.copy()
    rho[frame, panel] = value
    x = np.array([[9.0, 2.0, 1.0], [-7.0, 5.0, -2.0]])
    print(f"[nonfinite] general motion N={N} frame={frame} panel={panel} {value}", flush=True)
    ref, _, nt = oracle.gm_forward(ms, x, 0.3, dtau, 0.1, rho, u, pp)
    plan, p = _run_gpu(ms, x, 0.3, dtau, 0.1, rho, u, pp)
    valid = valid_mask(nt, p.shape[1]) > 0
    assert valid.any() and not np.isfinite(ref[valid]).any()
    assert not np.isfinite(p[valid]).any()
    assert np.all(p[~valid] == 0.0)
