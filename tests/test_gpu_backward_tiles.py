"""GPU parity of the LM head's backward in each of its tiles against the fp64 oracle, at tile edges."""
import pytest

import oracle
import workloads
from gpu_support import assert_close, dev_bf16, empty_bf16, empty_f32, host_f64_from_bf16, say, sync, workspace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,V", [
    (1, 32, 8),
    (130, 288, 1000),     # 128 x 128 tiles, ragged tokens, columns and vocabulary
    (2050, 4096, 104),    # 256 x 128 tiles
    (4100, 4096, 72),     # 256 x 256 tiles
])
def test_lmhead_backward_tiles(N, d, V):
    import paper_2609_33977_amd as gm
    say(f"LM head backward tiles: N={N} d={d} V={V}")
    case = workloads.make_distill_case((292, N, d, V), N, d, V)
    W = dev_bf16(case.W)
    ws = workspace(gm.gm_distill_workspace_size(N, d, V))
    loss, dH = empty_f32(1), empty_bf16(N, d)
    gm.gm_distill_fwd(dev_bf16(case.Ht), dev_bf16(case.Hs), W, None, loss, None, ws)
    gm.gm_distill_bwd(W, dH, ws)
    sync()
    ref = oracle.distill_loss_bwd(oracle.from_bf16(case.Ht), oracle.from_bf16(case.Hs), oracle.from_bf16(case.W))
    # dz and dH are each rounded to bf16: relative norm error below 2 * 2^-8
    assert_close("dH", host_f64_from_bf16(dH), ref, 2.0 ** -7)
