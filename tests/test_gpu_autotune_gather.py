"""The tuner times every size class on the forward gather that the whole batch runs,
also where the class by itself would run the other one."""
import numpy as np
import pytest

from gpu_common import make_plan, rel_l2, to_device
from workloads import configs, surfaces

pytestmark = pytest.mark.gpu


def _case(O, N, surf):
    return configs.Case(f"tune_O{O}_N{N}", surf, surfaces.observer_circle(O, 10.0, step_deg=360.0 / O), 0.4, 8.0, 1 / 64,
                        N, kind="dipole", omega=2.0, data_dtype=np.float32)


@pytest.mark.parametrize("kind", ["mfma", "lds"])
def test_classes_are_timed_on_the_batch_gather(kind, monkeypatch):
    """mfma: one class is too small for the matrix-core gather by itself; lds: one class alone would take
    it, a plan of the other keeps the batch from it."""
    import torch
    import paper_2312_16263_amd as fwh
    big = _case(360, 1700, surfaces.sphere(1.0, 32, 64))
    small = _case(16, 306, surfaces.sphere(1.0, 16, 32))
    plans = [make_plan(big, "f32"), make_plan(small, "f32", gather="auto" if kind == "mfma" else "lds")]
    batch = fwh.Batch(plans, [tuple(to_device(c.data(), torch.float32)) for c in (big, small)])
    assert batch.gather == kind
    timed = []
    time_forward = fwh._time_forward

    def record(b, reps):
        timed.append((len(b.plans), b.gather))
        return time_forward(b, reps)

    monkeypatch.setattr(fwh, "_time_forward", record)
    batch.forward()
    before = [p.clone() for p in batch.p_out]
    print(f"[autotune] batch of {kind}", flush=True)
    res = fwh.autotune(batch, candidates=[(4, 1e6), (2, 1e7)], bpc_candidates=(2,), reps=1)
    assert set(timed) == {(1, kind), (2, kind)}
    for c in res["classes"].values():  # every shape the batch can use has been timed
        assert sorted(r[0] for r in c["table"]) == ([2, 4] if kind == "mfma" else [4, 4])
    batch.forward()
    for a, b in zip(batch.p_out, before):  # other panel ranges: FP32 rounding of the partial sums
        assert rel_l2(a.double().cpu().numpy(), b.double().cpu().numpy()) <= 1e-6


def test_batch_gather_can_be_named():
    import torch
    import paper_2312_16263_amd as fwh
    c = _case(16, 306, surfaces.sphere(1.0, 16, 32))
    plan, data = make_plan(c, "f32"), tuple(to_device(c.data(), torch.float32))
    out = {}
    for kind in ("lds", "mfma"):
        b = fwh.Batch([plan], [data], gather=kind)
        assert b.gather == kind
        out[kind] = b.forward()[0].clone()
    assert torch.equal(out["lds"], out["mfma"])
    with pytest.raises(KeyError):
        fwh.Batch([plan], [data], gather="stream")
