"""The gather kernels at the sizes where their tiles, chunks and rows end, against
each other where they sum in the same order and against the FP64 oracle elsewhere:

* the matrix-core forward gather (16-observer tiles, 61-sample rows, windows up
  to any spread) equals the LDS-staged one bit for bit in FP32: the same FP32
  products summed in the same order over the same panel ranges;
* BF16 storage with FP64 data takes the LDS-staged gather;
* the few-observer kernel equals the streaming one bit for bit;
* the FP64 form's chunked sweeps, tiled gathers and their fallbacks for wide
  windows (a low frame rate against a large surface is narrow, a high one wide);
* the transposed gather at the ends of its 252-index blocks.

Tolerances: as in the parity tests, FP64 1e-11 at dtau = 1/16 and, since what
dominates there is the rounding of the mean flow in the frame difference over
2 dtau, in proportion to 1/dtau."""
import numpy as np
import pytest

from gpu_common import make_plan, oracle_adjoint, oracle_forward, rel_l2, to_device, valid_mask
from workloads import configs, surfaces

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-3, "f64": 1e-11}
# delay spread over a tile in samples: about 2 M0 / ((1 - M0^2) dtau) of the unit sphere's panels
NARROW, WIDE, WIDER = 1 / 16, 1 / 400, 1 / 2000


def _case(O, N, dtau=NARROW, P=97, dtype=np.float32, radius=10.0):
    surf = surfaces.sphere(1.0, 16, 32).subset(np.arange(3, 3 + P))
    return configs.Case(f"forms_O{O}_N{N}", surf, surfaces.observer_circle(O, radius, step_deg=360.0 / max(O, 2)), 0.4,
                        8.0, dtau, N, kind="dipole", omega=2.0, data_dtype=dtype)


def _run(case, mode, dtype=None, grad=False, **kw):
    import torch
    plan = make_plan(case, mode, **kw)
    d = to_device(case.data(), dtype)
    p = plan.forward(*d)
    g = plan.adjoint(*d, 2 * p) if grad else None
    torch.cuda.synchronize()
    return plan, p, g


@pytest.mark.parametrize("N,dtau", [(90, NARROW), (306, NARROW), (700, NARROW), (1400, WIDE)])
@pytest.mark.parametrize("O", [1, 15, 16, 17, 33])
def test_matrix_core_gather_equals_lds(O, N, dtau):
    import torch
    c = _case(O, N, dtau, P=300)
    print(f"[gather forms] mfma O={O} N={N} dtau={dtau}", flush=True)
    _, p_lds, _ = _run(c, "f32", gather="lds", splits=2)
    try:
        plan, p, _ = _run(c, "f32", gather="mfma", splits=2)
    except Exception as e:  # asked for by name it takes narrow windows only
        assert dtau == WIDE and "matrix-core" in str(e), e
        plan, p, _ = _run(c, "f32", splits=2)
    if plan.info()[0] in ("mfma", "lds"):  # (by itself a plan of few observers takes the streaming one)
        assert torch.equal(p, p_lds), float((p - p_lds).abs().max())
    p_ref, _, nt = oracle_forward(c, *c.data())
    assert rel_l2(p.cpu().numpy(), p_ref, valid_mask(nt, p.shape[1])) <= TOL["f32"]


@pytest.mark.parametrize("O", [9, 33])
def test_bf16_routes(O):
    import torch
    c = _case(O, 700, P=113)
    p_ref, _, nt = oracle_forward(c, *c.data())
    for dtype in (torch.float32, torch.float64):
        _, p, _ = _run(c, "bf16", dtype)
        assert rel_l2(p.cpu().numpy(), p_ref, valid_mask(nt, p.shape[1])) <= TOL["bf16"]
    _, p_lds, _ = _run(c, "bf16", torch.float64, gather="lds")
    assert torch.equal(p, p_lds)


@pytest.mark.parametrize("mode", ["f32", "bf16"])
@pytest.mark.parametrize("O,N", [(1, 70), (3, 306), (8, 500), (8, 1011)])
def test_few_observers_equal_streaming(O, N, mode):
    import torch
    c = _case(O, N)
    _, p, _ = _run(c, mode)
    _, ps, _ = _run(c, mode, gather="stream")
    assert torch.equal(p, ps), float((p - ps).abs().max())


@pytest.mark.parametrize("O,N,dtau,P", [(1, 4, NARROW, 5), (16, 306, NARROW, 97), (17, 211, NARROW, 97),
                                        (33, 700, NARROW, 113), (5, 1400, WIDE, 300), (17, 6000, WIDER, 300)])
def test_fp64_form(O, N, dtau, P):
    c = _case(O, N, dtau, P, np.float64, radius=3.0 if N == 4 else 10.0)
    if N == 4:
        c.dtau = 4.0
    print(f"[gather forms] f64 O={O} N={N} dtau={dtau} P={P}", flush=True)
    tol = TOL["f64"] * max(1.0, NARROW / c.dtau)
    _, p, g = _run(c, "f64", grad=True)
    p = p.cpu().numpy()
    data = c.data()
    p_ref, _, nt = oracle_forward(c, *data)
    assert rel_l2(p, p_ref, valid_mask(nt, p.shape[1])) <= tol
    for a, b in zip(g, oracle_adjoint(c, *data, 2 * p)):
        assert rel_l2(a.cpu().numpy(), b) <= tol


@pytest.mark.parametrize("O,N", [(1, 249), (7, 252), (33, 253), (4, 504), (16, 505), (5, 800)])
def test_transposed_gather_block_ends(O, N):
    c = _case(O, N)
    _, p, g = _run(c, "f32", grad=True)
    gbar = 2 * p.double().cpu().numpy()
    for a, b in zip(g, oracle_adjoint(c, *c.data(), gbar)):
        assert rel_l2(a.cpu().numpy(), b) <= TOL["f32"]


@pytest.mark.parametrize("mode", ["f32", "bf16"])
def test_batched_matrix_core_gather_equals_single(mode):
    import torch
    import paper_2312_16263_amd as fwh
    cases = [_case(O, N, P=P) for O, N, P in ((16, 306, 300), (17, 500, 257), (3, 120, 33))]
    plans = [make_plan(c, mode, gather="mfma", splits=min(2, c.n_panels // 128)) for c in cases]
    inputs = [tuple(to_device(c.data(), torch.float32)) for c in cases]
    batch = fwh.Batch(plans, inputs)
    assert batch.gather == "mfma"
    batch.forward()
    torch.cuda.synchronize()
    for c, plan, d, p in zip(cases, plans, inputs, batch.p_out):
        p_ref, _, nt = oracle_forward(c, *c.data())
        assert rel_l2(p.cpu().numpy(), p_ref, valid_mask(nt, p.shape[1])) <= TOL[mode]


def test_autotune_of_a_batch_with_a_small_class():
    """The batch is large enough for the matrix-core gather, its small class by itself is not."""
    import torch
    import paper_2312_16263_amd as fwh
    surf = surfaces.sphere(1.0, 32, 64)
    big = configs.Case("big", surf, surfaces.observer_circle(360, 10.0, step_deg=1.0), 0.4, 8.0, 1 / 64, 1700,
                       kind="dipole", omega=2.0, data_dtype=np.float32)
    cases = [big, _case(16, 306)]
    plans = [make_plan(c, "f32") for c in cases]
    batch = fwh.Batch(plans, [tuple(to_device(c.data(), torch.float32)) for c in cases])
    assert batch.gather == "mfma"
    batch.forward()
    torch.cuda.synchronize()
    before = [p.clone() for p in batch.p_out]
    res = fwh.autotune(batch, candidates=[(4, 1e6), (3, 1e6), (2, 1e7)], bpc_candidates=(2,), reps=1)
    assert len(res["classes"]) == 2
    batch.forward()
    torch.cuda.synchronize()
    for a, b in zip(batch.p_out, before):  # other panel ranges: FP32 rounding of the partial sums
        assert rel_l2(a.double().cpu().numpy(), b.double().cpu().numpy()) <= 1e-6
