"""GPU parity of the forward GEMM's tiles (256 x 256, 256 x 128 and 128 x 128 outputs, the latter two with K split
over two wave groups inside the block), in place and from the packed export, against the fp64 oracle (Eq. 1), at the
tile edges and for the pieces the packed tiles take off the matrix path."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_support import (assert_close, bound_fwd, dev_bf16, dev_f32, empty_bf16, host_bits, host_f64_from_bf16, say,
                         sync)

pytestmark = pytest.mark.gpu


def _pack(W, m, g, g_out, kept):
    import torch
    import paper_2609_33977_amd as gm
    cap = max(kept, 1)
    Wp = torch.zeros((cap, g), dtype=torch.bfloat16, device="cuda")
    chunk = torch.zeros(cap, dtype=torch.int32, device="cuda")
    scale = torch.zeros(cap, dtype=torch.float32, device="cuda")
    rowptr = torch.zeros(W.shape[0] + 1, dtype=torch.int32, device="cuda")
    gm.gm_pack_rows(W, m, g, kept, Wp, chunk, scale, rowptr, g_out=g_out)
    return Wp, chunk, scale, rowptr


def _both(case, mask):
    """Y in place (no workspace: one of the three tiles) and from the packed export."""
    import paper_2609_33977_amd as gm
    T, d_out, g, go = case.T, case.d_out, case.g, case.g_out
    X, W, m = dev_bf16(case.X), dev_bf16(case.W), dev_f32(mask)
    Yi, Yp = empty_bf16(T, d_out), empty_bf16(T, d_out)
    gm.gm_masked_linear_fwd(X, W, m, g, Yi, g_out=go)
    packed = _pack(W, m, g, go, int(np.count_nonzero(mask)) * go)
    gm.gm_packed_linear_fwd(X, *packed, d_out, g, Yp)
    sync()
    return Yi, Yp, packed


# The tile that the library chooses for the shape in place and packed (checked on the CPU by test_tile_plan.py).
FWD_TILES = [
    (17, 64, 8, 64, 1, "128x128", "passes16"),           # one unit: the second wave group has a single slice
    (129, 1536, 136, 512, 1, "128x128", "passes16"),     # one row and eight columns past the edge
    (100, 8192, 144, 16, 16, "128x128", "passes16"),     # 512 pieces of 16 weights per row
    (130, 320, 160, 32, 32, "128x128", "passes16"),
    (700, 192, 1032, 64, 1, "128x128", "128x128"),
    (900, 1536, 2056, 512, 1, "128x128", "128x128"),
    (1000, 8192, 1040, 16, 16, "128x128", "128x128"),
    (1000, 320, 2080, 32, 32, "128x128", "128x128"),
    (2040, 512, 4088, 256, 1, "256x128", "256x128"),     # ragged both ways
    (2041, 320, 4096, 32, 32, "256x128", "128x128"),
    (2041, 192, 4096, 64, 64, "256x128", "256x128"),
    (2041, 256, 4096, 128, 128, "256x128", "256x128"),
    (1100, 192, 8192, 64, 64, "256x256", "256x256"),
    (4090, 512, 4088, 128, 1, "256x256", "256x256"),
    (4090, 320, 4096, 16, 16, "256x256", "128x128"),
]


@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("T,d_in,d_out,g,g_out,tile,packed_tile", FWD_TILES)
def test_tiles_in_place_and_packed(T, d_in, d_out, g, g_out, tile, packed_tile, soft):
    say(f"forward tiles {tile}, packed {packed_tile}: T={T} d_in={d_in} d_out={d_out} g={g} g_out={g_out} soft={soft}")
    case = workloads.make_linear_case((280, T, d_in, d_out, g), T, d_in, d_out, g, None, g_out=g_out)
    mask = case.mask.astype(np.float32).copy()
    if soft:
        mask *= workloads.gen.rng_for(284).uniform(0.05, 1.5, size=mask.shape).astype(np.float32)
    mask[-1] = 0.0  # a pruned row of groups
    Yi, Yp, _ = _both(case, mask)
    Xo, Wo = oracle.from_bf16(case.X), oracle.from_bf16(case.W)
    ref = oracle.linear_fwd(Xo, Wo, mask, g, g_out)
    b = bound_fwd(Xo, Wo, mask, g, g_out, ref)
    assert_close("Y in place", host_f64_from_bf16(Yi), ref, bound=b)
    assert_close("Y packed", host_f64_from_bf16(Yp), ref, bound=b)


def test_packed_tiles_with_nothing_kept():
    T, d_in, d_out, g = 40, 512, 256, 256
    case = workloads.make_linear_case((281,), T, d_in, d_out, g, None)
    _, Yp, _ = _both(case, np.zeros_like(case.mask))
    assert not np.any(host_bits(Yp) & 0x7FFF)


@pytest.mark.parametrize("T,d_in,d_out,g", [(150, 1024, 264, 128), (2040, 512, 4088, 256)])
def test_packed_tiles_with_fractional_selectors_and_shuffled_pieces(T, d_in, d_out, g):
    # a few fractional selectors: their tiles keep selectors and products in
    # fp32 (the bound of binary selectors holds), the other tiles stay on the
    # matrix path; the pieces of a row in any order give the same rows
    import torch
    import paper_2609_33977_amd as gm
    say(f"packed tiles, fractional selectors: T={T} d_in={d_in} d_out={d_out} g={g}")
    case = workloads.make_linear_case((282, T), T, d_in, d_out, g, None)
    mask = case.mask.astype(np.float32).copy()
    mask[3, 1], mask[d_out - 1, 0] = 0.37, 1.21
    _, Yp, (Wp, chunk, scale, rowptr) = _both(case, mask)
    Xo, Wo = oracle.from_bf16(case.X), oracle.from_bf16(case.W)
    ref = oracle.linear_fwd(Xo, Wo, mask, g)
    S = oracle.linear_fwd(np.abs(Xo), np.abs(Wo), mask, g)
    acc = 2.0 * (d_in + 2) * 2.0 ** -24 * S  # fp32 sums and the fp32 product with the selector
    assert_close("Y packed", host_f64_from_bf16(Yp), ref, bound=2.0 ** -8 * (np.abs(ref) + acc) + acc)
    rp = rowptr.cpu().numpy()
    perm = np.arange(chunk.numel())
    a, b = rp[5], rp[6]
    perm[a:b] = perm[a:b][::-1]
    p = torch.from_numpy(perm).cuda()
    Ys = empty_bf16(T, d_out)
    gm.gm_packed_linear_fwd(dev_bf16(case.X), Wp[p].contiguous(), chunk[p].contiguous(), scale[p].contiguous(), rowptr,
                            d_out, g, Ys)
    sync()
    assert_close("Y of shuffled pieces", host_f64_from_bf16(Ys), ref, bound=2.0 ** -8 * (np.abs(ref) + acc) + acc)
