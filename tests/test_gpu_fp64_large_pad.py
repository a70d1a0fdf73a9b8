"""FP64 adjoint of a long record with many observers: the zero-padded copy of dJ/dp' has more
than 2^32 elements, which is more than one launch holds threads.  Only the last observer's
row, past that element, is not zero: the gradients are those of a plan of that observer."""
import numpy as np
import pytest

import paper_2312_16263_amd as fwh
from workloads import surfaces

pytestmark = pytest.mark.gpu

O, N, MACH = 32768, 65535, 0.01
DTAU = 2 * MACH / 64000  # the sphere's delay spread takes most of the record: short windows


def test_padded_gradient_beyond_one_launch():
    import torch
    if torch.cuda.mem_get_info()[0] < 200e9:
        pytest.skip("takes 180 GB of device memory")
    s = surfaces.sphere(1.0, 86, 96)
    x = surfaces.observer_circle(O, 10.0, step_deg=360.0 / O)

    def plan(x_obs):
        return fwh.Plan(s.y, s.normal, s.dS, x_obs, MACH, 0.0, DTAU, 0.0, N, mode="f64")

    gen = torch.Generator(device="cuda").manual_seed(1)
    rho, p = (0.01 * torch.randn(N, s.n_panels, device="cuda", generator=gen) for _ in range(2))
    u = 0.01 * torch.randn(3, N, s.n_panels, device="cuda", generator=gen)
    rho += 1
    u[0] += 1
    one = plan(x[-1:])
    row = torch.randn(1, one.window.n_t_max, device="cuda", generator=gen, dtype=torch.float64)
    ref = one.adjoint(rho, u, p, row)
    del one
    many = plan(x)
    print(f"[large pad] P={s.n_panels} N={N} O={O}: workspace {many.workspace_bytes / 1e9:.0f} GB", flush=True)
    grad = torch.zeros(O, many.window.n_t_max, device="cuda", dtype=torch.float64)
    grad[-1, :row.shape[1]] = row[0]
    for a, b in zip(many.adjoint(rho, u, p, grad), ref):
        assert float(b.abs().max()) > 0.0
        assert torch.equal(a, b)  # the other observers add exact zeros
    del many, grad
    torch.cuda.empty_cache()
