"""GPU parity of the 2-16 token decode kernel against the fp64 oracle at the edges of its block rule: 16-, 32- and
64-row blocks, with the smaller and the larger staged tables, in place and from the packed export."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_support import (assert_close, dev_bf16, dev_f32, empty_bf16, host_bits, host_f64_from_bf16, ref_fwd, say, sync)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d_in,d_out,g", [
    (2, 1024, 4096, 256),    # 16-row blocks, one per CU
    (16, 1024, 4104, 256),   # 32-row blocks, the last with 8 rows
    (9, 8192, 264, 64),      # 16-row blocks, tables of 2048 selectors
    (8, 8256, 264, 64),      # one group more: the larger tables
    (3, 8192, 4104, 64),     # 32-row blocks, tables of 4096
    (12, 8256, 4104, 64),
    (8, 512, 12296, 256),    # 64-row blocks in place, 32-row packed
    (16, 512, 16392, 256),   # just past one round of 64-row blocks
    (16, 512, 26632, 256),   # a second round
    (14, 5120, 26632, 256),  # ... well filled, of long rows: 64-row blocks in place
])
def test_decode_blocks(T, d_in, d_out, g):
    import torch
    import paper_2609_33977_amd as gm
    say(f"decode blocks: T={T} d_in={d_in} d_out={d_out} g={g}")
    case = workloads.make_linear_case((294, T, d_in, d_out, g), T, d_in, d_out, g, None)
    mask = case.mask.astype(np.float32).copy()
    mask[d_out // 2] = 0.0   # a row that keeps nothing
    mask[-1] = 1.0
    X, W, m = dev_bf16(case.X), dev_bf16(case.W), dev_f32(mask)
    Y, Yp = empty_bf16(T, d_out), empty_bf16(T, d_out)
    gm.gm_masked_linear_fwd(X, W, m, g, Y)
    cap = int(np.count_nonzero(mask))
    Wp, chunk = empty_bf16(cap, g), torch.empty(cap, dtype=torch.int32, device="cuda")
    scale, rowptr = torch.empty(cap, device="cuda"), torch.empty(d_out + 1, dtype=torch.int32, device="cuda")
    gm.gm_pack_rows(W, m, g, cap, Wp, chunk, scale, rowptr)
    gm.gm_packed_linear_fwd(X, Wp, chunk, scale, rowptr, d_out, g, Yp)
    sync()
    ref, b = ref_fwd(oracle.from_bf16(case.X), oracle.from_bf16(case.W), mask, g)
    assert_close("Y", host_f64_from_bf16(Y), ref, bound=b)
    # both layouts sum the same products in the same order, whatever their block height
    assert np.array_equal(host_bits(Y), host_bits(Yp))
