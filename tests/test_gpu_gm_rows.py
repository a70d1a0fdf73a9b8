"""General motion where a block of the spline prefilter takes several rows: surfaces that fill the chip with them, rows that do
not fill the last block, one and several segments per row.  Against the FP64 oracle, tolerance as in the
parity tests of this path."""
import numpy as np
import pytest

import oracle
from test_gpu_gm import TOL, _run_gpu
from workloads import motion, surfaces

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,N", [(11, 23, 30), (11, 23, 100), (8, 16, 35)])
def test_several_rows_per_block(n1, n2, N):
    body = surfaces.sphere(1.0, n1, n2)
    dtau = max(1 / 64, 2.0 / N)
    ms = motion.moving_surface(body, "orbit", N, dtau, 0.1, spin=0.5)
    rho, u, pp = motion.quiescent_monopole_series(ms, 0.3, 0.01, 6.0, dtau, 0.1, source=(0.05, 0.02, 0.0))
    x = np.array([[9.0, 2.0, 1.0], [-7.0, 5.0, -2.0]])
    print(f"[gm rows] N={N} P={ms.n_panels}", flush=True)
    plan, p = _run_gpu(ms, x, 0.3, dtau, 0.1, rho, u, pp)
    ref, _, nt = oracle.gm_forward(ms, x, 0.3, dtau, 0.1, rho, u, pp)
    np.testing.assert_array_equal(plan.window.n_t, nt)
    assert np.abs(p - ref).max() <= TOL * np.abs(ref).max()
