"""GPU parity of the distillation loss where exponentials leave the normal range: logits hundreds apart (terms below
2^-126 count as zero) and teacher logits that overflow to minus infinity (probability zero), with a ragged vocabulary
tile, against the fp64 oracle."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_support import assert_close, dev_bf16, empty_bf16, empty_f32, host_f64_from_bf16, say, sync, workspace

pytestmark = pytest.mark.gpu


def _check(case):
    import paper_2609_33977_amd as gm
    N, d, V = case.N, case.d, case.V
    ws = workspace(gm.gm_distill_workspace_size(N, d, V))
    loss, ce, dH, W = empty_f32(1), empty_f32(N), empty_bf16(N, d), dev_bf16(case.W)
    gm.gm_distill_fwd(dev_bf16(case.Ht), dev_bf16(case.Hs), W, None, loss, ce, ws)
    gm.gm_distill_bwd(W, dH, ws)
    sync()
    Ht, Hs, Wo = (oracle.from_bf16(x) for x in (case.Ht, case.Hs, case.W))
    L_ref, ce_ref, _, _ = oracle.distill_loss(Ht, Hs, Wo)
    # logits of size z carry an absolute error of about 2 d 2^-24 sum|terms|, which enters the loss directly
    zmax = float((np.abs(Hs) @ np.abs(Wo).T).max())
    tol = 1e-5 + 2 * d * 2.0 ** -24 * zmax / max(abs(L_ref), 1.0)
    assert np.isfinite(float(loss.item())) and abs(float(loss.item()) - L_ref) <= tol * max(abs(L_ref), 1.0)
    assert_close("ce", ce.cpu().numpy(), np.asarray(ce_ref), max(tol, 1e-5))
    assert np.all(np.isfinite(host_f64_from_bf16(dH)))


@pytest.mark.parametrize("logit_std", [60.0, 400.0])
def test_distill_far_apart_logits(logit_std):
    say(f"distillation loss, logits of standard deviation {logit_std}")
    _check(workloads.make_distill_case((296, int(logit_std)), 130, 64, 1000, logit_std=logit_std, student_noise=0.05))


def test_distill_teacher_logits_at_minus_infinity():
    case = workloads.make_distill_case((297,), 40, 64, 520)
    say("distillation loss, teacher logits of minus infinity")
    bits = workloads.bf16_bits_from_f32
    case.W[[3, 300, 519], 5] = bits(np.float32([-1e30, -1e30, -1e30]))
    case.Ht[:, 5] = bits(np.full(40, 1e30, np.float32))
    case.Hs[:, 5] = 0
    case.W[np.setdiff1d(np.arange(520), [3, 300, 519]), 5] = 0
    _check(case)
