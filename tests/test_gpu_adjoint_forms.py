"""The two forms of the transposed gather, at the sizes where their index blocks, observer groups and tiles
end, against the FP64 oracle:

* records of at most 320 coefficient indices and small surfaces: blocks of 64 indices, four observers
  at a time (groups past the last observer, tiles of 16, records of 1 to 5 blocks and of a second wave);
* the others: blocks of 252 indices, one observer at a time;
* a batch that holds both, against the single plans bit for bit.

Tolerance: that of the FP32 gradient tests."""
import numpy as np
import pytest

from gpu_common import make_plan, oracle_adjoint, rel_l2, to_device
from workloads import configs, surfaces

pytestmark = pytest.mark.gpu

TOL = 1e-5


def _case(O, N, surf):
    # the delays' spread takes about a quarter of the record
    return configs.Case(f"adj_O{O}_N{N}", surf, surfaces.observer_circle(O, 10.0, step_deg=360.0 / max(O, 2)), 0.4, 8.0,
                        5.0 / (N - 2), N, kind="dipole", omega=2.0, data_dtype=np.float32)


def _check(c):
    import torch
    plan = make_plan(c, "f32")
    d = to_device(c.data())
    gbar = torch.randn(c.n_obs, plan.window.n_t_max, generator=torch.Generator().manual_seed(5))
    g = plan.adjoint(*d, gbar.cuda())
    ref = oracle_adjoint(c, *c.data(), gbar.double().numpy())
    for a, b in zip(g, ref):
        assert rel_l2(a.cpu().numpy(), b) <= TOL


@pytest.mark.parametrize("O,N", [(1, 20), (2, 52), (3, 53), (12, 116), (13, 117), (16, 180), (17, 181), (24, 244), (35, 245),
                                 (32, 308), (33, 309), (12, 628), (18, 629), (50, 1000)])
def test_blocks_of_64(O, N):
    print(f"[adjoint forms] 64 O={O} N={N}", flush=True)
    _check(_case(O, N, surfaces.sphere(1.0, 16, 32).subset(np.arange(3, 100))))


@pytest.mark.parametrize("O,N", [(5, 100), (17, 309), (16, 502), (33, 503), (21, 754), (12, 1007)])
def test_blocks_of_252(O, N):
    print(f"[adjoint forms] 252 O={O} N={N}", flush=True)
    _check(_case(O, N, surfaces.sphere(1.0, 40, 65)))


def test_batch_with_both():
    import torch
    import paper_2312_16263_amd as fwh
    surf = surfaces.sphere(1.0, 40, 65)
    cases = [_case(33, 503, surf), _case(20, 60, surf), _case(6, 700, surf.subset(np.arange(77))), _case(40, 200, surf)]
    plans = [make_plan(c, "f32") for c in cases]
    inputs = [tuple(to_device(c.data(), torch.float32)) for c in cases]
    batch = fwh.Batch(plans, inputs)
    batch.forward()
    for p, g in zip(batch.p_out, batch.grad_p):
        torch.mul(p, 2.0, out=g)
    batch.adjoint()
    torch.cuda.synchronize()
    for plan, d, gbar, g in zip(plans, inputs, batch.grad_p, batch.grads):
        for a, b in zip(g, plan.adjoint(*d, gbar)):
            assert torch.equal(a, b)
