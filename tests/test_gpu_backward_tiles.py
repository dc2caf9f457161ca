"""GPU parity of the backward GEMMs' tiles against the fp64 oracle, at tile edges: dX over column lists in its
64- to 256-column tiles with and without two K groups, dX of 16 x 16 and 32 x 32 groups over every row, dgate in its
256-, 128- and 64-column tiles, and the LM head's backward in each of its tiles."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_support import (assert_close, dev_bf16, dev_f32, empty_bf16, empty_f32, host_bits, host_f64_from_bf16, ref_dgate, ref_dx,
                         say, sync, workspace)

pytestmark = pytest.mark.gpu


def _dx(case, mask, with_dgate):
    import paper_2609_33977_amd as gm
    T, d_in, d_out, g, go = case.T, case.d_in, case.d_out, case.g, case.g_out
    dX = empty_bf16(T, d_in)
    dgate = empty_f32(*mask.shape) if with_dgate else None
    ws = workspace(gm.gm_workspace_size(gm.GM_OP_BWD, T, d_in, d_out, g, go))
    gm.gm_masked_linear_bwd(dev_bf16(case.dY), dev_bf16(case.X), dev_bf16(case.W), dev_f32(mask), g, dX, dgate, ws,
                            g_out=go)
    sync()
    return dX


def _soften(mask, key):
    r = workloads.gen.rng_for(key)
    soft = np.where(mask != 0, r.uniform(0.05, 1.5, size=mask.shape), 0.0).astype(np.float32)
    soft[mask.shape[0] // 2:, 0] = 1.0
    return soft


# Each list gives the tile that the library chooses for the shape (checked on the CPU by test_tile_plan.py).
DX_TILES = [
    (17, 64, 8, 64, 1, "64x256"),
    (40, 1024, 2056, 512, 1, "64x128"),     # ragged tokens and rows
    (128, 4096, 1056, 256, 1, "128x128"),
    (128, 4096, 4104, 256, 1, "64x128"),
    (130, 1024, 1032, 256, 1, "128x128"),
    (260, 512, 512, 512, 1, "128x128"),
    (1030, 2816, 520, 128, 1, "128x128"),
    (2041, 4096, 264, 256, 1, "256x128"),
    (4090, 4096, 264, 512, 1, "256x256"),
    (2050, 4096, 264, 128, 1, "128x256"),
    (300, 384, 384, 128, 128, "128x128"),
    (1000, 16384, 128, 64, 64, "64x256"),   # two blocks per CU
    (33, 64, 32, 16, 16, "dense 128x128"),  # every row: one slice, a single mask-row pair
    (140, 320, 336, 16, 16, "dense 128x128"),  # K not a multiple of 32, columns past the last tile
    (257, 576, 96, 32, 32, "dense 128x128"),
    (1100, 4096, 160, 32, 32, "dense 128x128"),
    (17, 4096, 2048, 32, 32, "dense 128x128"),  # dX before dgate in their common launch
    (2041, 4096, 160, 32, 32, "dense 256x128"),
    (2041, 4096, 144, 16, 16, "dense 256x128"),
    (4090, 4096, 96, 32, 32, "dense 256x256"),
    (4000, 4096, 64, 16, 16, "dense 256x256"),
    (17, 64, 32784, 16, 16, "64x256"),      # more mask rows than a tile holds: lists of four groups a column
    (17, 64, 65568, 32, 32, "64x256"),      # ... and of two
    (300, 128, 65568, 32, 32, "64x256"),
]


@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("T,d_in,d_out,g,g_out,tile", DX_TILES)
def test_dx_tiles(T, d_in, d_out, g, g_out, tile, soft):
    say(f"dX tiles {tile}: T={T} d_in={d_in} d_out={d_out} g={g} g_out={g_out} soft={soft}")
    case = workloads.make_linear_case((290, T, d_in, d_out, g), T, d_in, d_out, g, None, g_out=g_out)
    mask = case.mask.astype(np.float32).copy()
    mask[:, -1] = 0.0  # a pruned column
    if soft:
        mask = _soften(mask, 291)
    ref, b = ref_dx(oracle.from_bf16(case.dY), oracle.from_bf16(case.W), mask, g, g_out)
    dX = _dx(case, mask, True)
    assert_close("dX", host_f64_from_bf16(dX), ref, bound=b)
    assert np.array_equal(host_bits(dX), host_bits(_dx(case, mask, False))), "dX differs without dgate beside it"


@pytest.mark.parametrize("fill", [0xFF, 0x7F])
@pytest.mark.parametrize("T,d_in,d_out,g,g_out", [
    (17, 64, 40, 64, 1),     # offsets of the unwritten entry -1 end just below 2^32
    (96, 128, 104, 64, 1),
    (1000, 192, 72, 64, 1),
    (1000, 16384, 128, 64, 64),
    (2050, 4096, 264, 128, 1),
    (4090, 4096, 520, 256, 1),
])
def test_dx_does_not_read_unwritten_list_entries(T, d_in, d_out, g, g_out, fill):
    """A column's list ends after its kept rows; the entries up to the end of the last 32-row slice hold whatever
    the workspace held, here 0xFF bytes (row -1, selector NaN), and must not choose an address."""
    import paper_2609_33977_amd as gm
    say(f"dX, workspace of {fill:#x} bytes: T={T} d_in={d_in} d_out={d_out} g={g} g_out={g_out}")
    case = workloads.make_linear_case((297, T, d_in, d_out, g), T, d_in, d_out, g, None, g_out=g_out)
    dY, W, m = dev_bf16(case.dY), dev_bf16(case.W), dev_f32(case.mask)
    ws = workspace(gm.gm_workspace_size(gm.GM_OP_BWD, T, d_in, d_out, g, g_out))
    ws.fill_(fill)
    dX = empty_bf16(T, d_in)
    gm.gm_masked_linear_bwd(dY, dev_bf16(case.X), W, m, g, dX, None, ws, g_out=g_out)
    sync()
    ref, b = ref_dx(oracle.from_bf16(case.dY), oracle.from_bf16(case.W), case.mask, g, g_out)
    assert_close("dX", host_f64_from_bf16(dX), ref, bound=b)


DGATE_TILES = [
    (1, 64, 8, 64, 1, "256x64"),           # one slice: the second K group has none
    (33, 192, 72, 64, 1, "256x64"),        # a row past the first tile, columns past 128
    (100, 1024, 1000, 512, 1, "256x64"),   # two tiles add to a group
    (70, 640, 264, 128, 1, "256x64"),
    (1000, 2816, 2056, 128, 1, "256x128"),
    (900, 4096, 1032, 256, 1, "256x128"),
    (650, 4096, 1000, 64, 1, "256x64"),
    (700, 4096, 2000, 512, 1, "256x128"),
    (650, 4096, 2000, 64, 1, "256x128"),
    (40, 320, 336, 16, 16, "256x128"),
    (33, 320, 160, 32, 32, "256x128"),
    (200, 832, 448, 64, 64, "256x128"),
    (65, 384, 384, 128, 128, "256x128"),
    (300, 4096, 4096, 128, 128, "256x256"),
    (130, 4096, 3848, 64, 1, "256x256"),
]


@pytest.mark.parametrize("T,d_in,d_out,g,g_out,tile", DGATE_TILES)
def test_dgate_tiles(T, d_in, d_out, g, g_out, tile):
    say(f"dgate tiles {tile}: T={T} d_in={d_in} d_out={d_out} g={g} g_out={g_out}")
    import paper_2609_33977_amd as gm
    case = workloads.make_linear_case((293, T, d_in, d_out, g), T, d_in, d_out, g, None, g_out=g_out)
    dgate, dX = empty_f32(*case.mask.shape), empty_bf16(T, d_in)
    ws = workspace(gm.gm_workspace_size(gm.GM_OP_BWD, T, d_in, d_out, g, g_out))
    dY, X, W = dev_bf16(case.dY), dev_bf16(case.X), dev_bf16(case.W)
    gm.gm_masked_linear_bwd(dY, X, W, dev_f32(case.mask), g, dX, dgate, ws, g_out=g_out)
    sync()
    ref, b = ref_dgate(oracle.from_bf16(case.dY), oracle.from_bf16(case.X), oracle.from_bf16(case.W), g, g_out)
    assert_close("dgate", dgate.cpu().numpy(), ref, bound=b)
    alone = empty_f32(*case.mask.shape)
    gm.gm_masked_linear_bwd(dY, X, W, None, g, None, alone, None, g_out=g_out)
    sync()
    assert np.array_equal(alone.cpu().numpy(), dgate.cpu().numpy()), "dgate differs without dX beside it"


LM_TILES = [
    (1, 32, 8, "128x128"),
    (130, 288, 1000, "128x128"),  # ragged tokens, columns and vocabulary
    (2041, 4096, 104, "256x128"),
    (2050, 4096, 104, "256x256"),
    (4100, 4096, 72, "256x256"),
]


@pytest.mark.parametrize("N,d,V,tile", LM_TILES)
def test_lmhead_backward_tiles(N, d, V, tile):
    import paper_2609_33977_amd as gm
    say(f"LM head backward tiles {tile}: N={N} d={d} V={V}")
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
