"""Every compiled form of the matrix-core forward gather against the LDS-staged one, and the
few-observer gather against the streaming one, over the launch shapes that choose between the forms:

* single plans: blocks of 4, 2 and 1 rows of 61 samples with operands four panels ahead (launches that leave
  room on the device) and of 4 rows with one panel ahead (launches that fill it), record lengths that leave 1
  to 4 rows in the last block, full and partly filled tiles of observers, more than 256 panels per
  split (partial sums of a chunk are added to the output);
* batches: 2, 3 and 4 rows per block, against the LDS-staged batch with the same panel ranges;
* few observers: several splits, more than 256 panels per split, a split without panels.

FP32 storage: the same products summed in the same order, bit for bit.  BF16 storage: the matrix cores
add the 16 exact products of an index (8 channels, high and low part of the weight) in another order,
at most 16 roundings of 2^-24 each, 1e-6 of a term; 2e-6 of the signal allows for terms that cancel.
A weight without its low part would be 2^-9 off."""
import numpy as np
import pytest

from gpu_common import make_plan, rel_l2, to_device
from workloads import configs, surfaces

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-6


def _case(surf, O, N, dtau=1 / 16):
    return configs.Case(f"equal_O{O}_N{N}", surf, surfaces.observer_circle(O, 10.0, step_deg=360.0 / max(O, 2)), 0.4,
                        8.0, dtau, N, kind="dipole", omega=2.0, data_dtype=np.float32)


def _equal(p, ref, mode):
    import torch
    if mode == "f32":
        assert torch.equal(p, ref), float((p - ref).abs().max())
    else:
        err = rel_l2(p.double().cpu().numpy(), ref.double().cpu().numpy())
        print(f"    rel L2 {err:.2e}", flush=True)
        assert err <= BF16_TOL


@pytest.mark.parametrize("mode", ["f32", "bf16"])
@pytest.mark.parametrize("O,N,splits", [(100, 1400, 20), (100, 1461, 20), (100, 1522, 20), (100, 1583, 20),  # 4 rows, full
                                        (400, 1500, 8),                              # the same, 325 panels per split
                                        (100, 1500, 12),                             # 4 rows, few blocks
                                        (100, 1500, 8), (33, 1500, 2), (17, 600, 1)])  # 2 rows; 1 row
def test_matrix_core_forms(O, N, splits, mode):
    import torch
    c = _case(surfaces.sphere(1.0, 40, 65), O, N)
    d = to_device(c.data(), torch.float32)
    print(f"[gather equality] {mode} O={O} N={N} splits={splits}", flush=True)
    ref = make_plan(c, mode, gather="lds", splits=splits).forward(*d)
    plan = make_plan(c, mode, gather="mfma", splits=splits)
    assert plan.info() == ("mfma", splits)
    _equal(plan.forward(*d), ref, mode)


@pytest.mark.parametrize("mode", ["f32", "bf16"])
@pytest.mark.parametrize("rows", [2, 3, 4])
def test_batched_matrix_core_forms(rows, mode):
    import torch
    import paper_2312_16263_amd as fwh
    surf = surfaces.sphere(1.0, 16, 32)
    cases = [_case(surf.subset(np.arange(P)), O, N) for O, N, P in ((16, 306, 300), (17, 500, 512), (35, 430, 257),
                                                                    (3, 120, 33))]
    inputs = [tuple(to_device(c.data(), torch.float32)) for c in cases]
    out = {}
    for gather in ("lds", "mfma"):
        plans = [make_plan(c, mode, gather=gather) for c in cases]
        batch = fwh.Batch(plans, inputs, item_units=1e12)  # one panel range per case, whatever the rows
        assert batch.gather == gather
        if gather == "mfma":
            for i in range(len(cases)):
                batch.tune_case(i, None, rows, bind=False)
            batch.bind()
        print(f"[gather equality] batch {gather} {mode} rows={rows}", flush=True)
        out[gather] = [p.clone() for p in batch.forward()]
        torch.cuda.synchronize()
    for p, ref in zip(out["mfma"], out["lds"]):
        _equal(p, ref, mode)
    for c, d, p in zip(cases, inputs, out["mfma"]):  # the single plan's form, one panel range
        _equal(make_plan(c, mode, gather="mfma", splits=1).forward(*d), p, mode)


@pytest.mark.parametrize("mode", ["f32", "bf16"])
@pytest.mark.parametrize("n1,n2,O,N,splits", [(22, 50, 8, 200, 2),      # 550 panels per split: 2 chunks and a rest
                                              (22, 50, 3, 130, 9),      # 123 panels per split
                                              (114, 225, 1, 150, 200)])  # the last split has no panels
def test_few_observers_equal_streaming(n1, n2, O, N, splits, mode):
    import torch
    c = _case(surfaces.sphere(1.0, n1, n2), O, N)
    d = to_device(c.data(), torch.float32)
    print(f"[gather equality] few {mode} P={c.n_panels} O={O} N={N} splits={splits}", flush=True)
    few, stream = (make_plan(c, mode, gather=g, splits=splits) for g in ("auto", "stream"))
    assert few.info() == stream.info() == ("stream", splits)
    assert c.n_panels * O * few.window.n_t_max < 24e6  # the automatic choice is the few-observer kernel
    p, ref = few.forward(*d), stream.forward(*d)
    assert torch.equal(p, ref), float((p - ref).abs().max())
