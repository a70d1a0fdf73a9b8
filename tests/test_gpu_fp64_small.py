"""The FP64 form where it changes its kernels: surfaces small enough for the gather with a thread per output, or just
large enough for the tiled one; records of one chunk of 64 coefficient indices and of one index more, chunks of 128, 256
and 512 frames (large surfaces), with a value that is not finite in one of them.  Against the oracle, tolerance of
the FP64 parity tests; theirs of the signals is for omega = 2, and what dominates it is the rounding of the
mean flow in the frame difference, which does not fall with omega while a compact dipole's far field does, as
omega^2."""
import numpy as np
import pytest

from gpu_common import make_plan, oracle_adjoint, oracle_forward, rel_l2, to_device, valid_mask
from workloads import configs, surfaces

pytestmark = pytest.mark.gpu

TOL = 1e-11
OMEGA = 0.5

def _case(n1, n2, O, N):
    return configs.Case(f"small_O{O}_N{N}", surfaces.sphere(1.0, n1, n2), surfaces.observer_circle(O, 10.0, step_deg=360.0 / max(O, 2)),
                        0.4, 8.0, max(1 / 16, 5.0 / (N - 2)), N, kind="dipole", omega=OMEGA)


@pytest.mark.parametrize("n1,n2,O,N", [(1, 1, 1, 40), (3, 3, 2, 20), (6, 8, 17, 52), (6, 8, 33, 300), (8, 8, 16, 53),
                                       (10, 14, 5, 100), (10, 14, 400, 60), (128, 256, 1, 116), (128, 256, 1, 117),
                                       (128, 256, 1, 300), (128, 256, 2, 515)])
def test_against_the_oracle(n1, n2, O, N):
    c = _case(n1, n2, O, N)
    data = c.data()
    plan = make_plan(c, "f64")
    print(f"[fp64 small] P={c.n_panels} O={O} N={N}: {plan.info()[1]} panel ranges", flush=True)
    d = to_device(data)
    p = plan.forward(*d)
    ref, _, nt = oracle_forward(c, *data)
    assert rel_l2(p.cpu().numpy(), ref, valid_mask(nt, p.shape[1])) <= TOL * (2.0 / OMEGA) ** 2
    for a, b in zip(plan.adjoint(*d, 2 * p), oracle_adjoint(c, *data, 2 * p.cpu().numpy())):
        assert rel_l2(a.cpu().numpy(), b) <= TOL


@pytest.mark.parametrize("frame", [0, 20, 51])
def test_short_record_with_a_value_that_is_not_finite(frame):
    c = _case(6, 8, 3, 52)
    rho, u, pp = c.data()
    rho[frame, 11] = np.nan
    p = make_plan(c, "f64").forward(*to_device((rho, u, pp))).cpu().numpy()
    ref, _, nt = oracle_forward(c, rho, u, pp)
    valid = valid_mask(nt, p.shape[1]) > 0
    assert not np.isfinite(ref[valid]).any() and not np.isfinite(p[valid]).any()
    assert np.all(p[~valid] == 0.0)
