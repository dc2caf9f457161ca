"""GPU parity of the forward's 128 x 128 tiles with K split over blocks and two wave groups against the fp64 oracle,
at tile and share edges (shares with one slice, with none, ragged tokens and rows)."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_support import (assert_close, dev_bf16, dev_f32, empty_bf16, host_bits, host_f64_from_bf16, ref_fwd, say, sync,
                         workspace)

pytestmark = pytest.mark.gpu


# The tile, and the shares that the workspace of the shape holds.
SHAPES = [
    (17, 1024, 1024, 256, 1, "128x128 split", 4),
    (128, 4096, 1032, 512, 1, "128x128 split", 8),   # one unit per share
    (100, 1536, 3080, 64, 1, "128x128 split", 8),
    (300, 2816, 2056, 128, 1, "128x128 split", 5),
    (40, 512, 336, 16, 16, "128x128", 8),   # a workspace, but no split
    (40, 2048, 336, 16, 16, "128x128 split", 8),
    (400, 1024, 1056, 32, 32, "128x128 split", 8),
    (129, 2048, 4096, 64, 64, "128x128 split", 8),
    (150, 2048, 1024, 128, 128, "128x128 split", 8),
]


@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("kept_columns", [None, 1, 3])
@pytest.mark.parametrize("T,d_in,d_out,g,g_out,tile,shares", SHAPES)
def test_split_tiles(T, d_in, d_out, g, g_out, tile, shares, kept_columns, soft):
    import paper_2609_33977_amd as gm
    say(f"split tiles, {tile}: T={T} d_in={d_in} d_out={d_out} g={g} g_out={g_out} kept_columns={kept_columns} soft={soft}")
    case = workloads.make_linear_case((295, T, d_in, d_out, g), T, d_in, d_out, g, None, g_out=g_out)
    mask = case.mask.astype(np.float32).copy()
    if kept_columns is not None:  # fewer kept columns than shares: some shares are empty
        mask[:, :] = 0.0
        mask[::2, -kept_columns:] = 1.0
    if soft:
        mask *= workloads.gen.rng_for(296).uniform(0.1, 1.5, size=mask.shape).astype(np.float32)
    need = gm.gm_workspace_size(gm.GM_OP_FWD, T, d_in, d_out, g, g_out)
    assert need == (shares * T * d_out * 4 + 255) // 256 * 256
    X, W, m, ws = dev_bf16(case.X), dev_bf16(case.W), dev_f32(mask), workspace(need)
    Y, again = empty_bf16(T, d_out), empty_bf16(T, d_out)
    gm.gm_masked_linear_fwd(X, W, m, g, Y, ws, g_out=g_out)
    gm.gm_masked_linear_fwd(X, W, m, g, again, ws, g_out=g_out)
    sync()
    ref, b = ref_fwd(oracle.from_bf16(case.X), oracle.from_bf16(case.W), mask, g, g_out)
    assert_close("Y", host_f64_from_bf16(Y), ref, bound=b)
    assert np.array_equal(host_bits(Y), host_bits(again))
