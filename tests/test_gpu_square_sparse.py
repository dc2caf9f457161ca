"""dX of 16 x 16 and 32 x 32 groups under sparse masks, where the tiles walk the mask rows that keep something in their
columns: parity against the fp64 oracle in each tile, and a time that falls with the density."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_support import assert_close, dev_bf16, dev_f32, empty_bf16, host_f64_from_bf16, ref_dx, say, sync, workspace

pytestmark = pytest.mark.gpu


def _sparse(case, kind, r):
    rows, cols = case.mask.shape
    m = (r.uniform(size=(rows, cols)) < (0.02 if kind == "2 %" else 0.1)).astype(np.float32)
    if kind == "one row":  # one entry: the second half of its slice, and the second K group, have none
        m[:] = 0.0
        m[rows // 2, 1::3] = 1.0
    elif kind == "rows pruned":
        m = (r.uniform(size=(rows, cols)) < 0.5).astype(np.float32)
        m[r.uniform(size=rows) < 0.6] = 0.0
    elif kind == "columns pruned":  # tiles with nothing to do beside full ones
        m[:, cols // 2:] = 0.0
        m[:, :cols // 4] = 1.0
    return m


SHAPES = [
    (140, 320, 336, 16, "dense 128x128"),
    (257, 576, 1056, 32, "dense 128x128"),
    (2041, 4096, 336, 16, "dense 256x128"),
    (2041, 4096, 800, 32, "dense 256x128"),
    (4090, 4096, 272, 16, "dense 256x256"),
    (4090, 4096, 288, 32, "dense 256x256"),
]


@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("kind", ["2 %", "10 %", "one row", "rows pruned", "columns pruned"])
@pytest.mark.parametrize("T,d_in,d_out,g,tile", SHAPES)
def test_dx_of_sparse_masks(T, d_in, d_out, g, tile, kind, soft):
    import paper_2609_33977_amd as gm
    say(f"sparse dX, {tile}: T={T} d_in={d_in} d_out={d_out} g={g} {kind} soft={soft}")
    case = workloads.make_linear_case((300, T, d_in, d_out, g), T, d_in, d_out, g, None, g_out=g)
    r = workloads.gen.rng_for(301, T, g)
    m = _sparse(case, kind, r)
    if soft:
        m *= r.uniform(0.05, 1.5, size=m.shape).astype(np.float32)
    dX = empty_bf16(T, d_in)
    ws = workspace(gm.gm_workspace_size(gm.GM_OP_BWD, T, d_in, d_out, g, g))
    gm.gm_masked_linear_bwd(dev_bf16(case.dY), dev_bf16(case.X), dev_bf16(case.W), dev_f32(m), g, dX, None, ws, g_out=g)
    sync()
    ref, b = ref_dx(oracle.from_bf16(case.dY), oracle.from_bf16(case.W), m, g, g)
    assert_close("dX", host_f64_from_bf16(dX), ref, bound=b)


@pytest.mark.parametrize("g", [16, 32])
def test_dx_time_falls_with_the_density(g):
    # 3 % kept: 0.57 (16 x 16) and 0.40 (32 x 32) of the time of half kept; 1.0 if every row were visited
    import torch
    import paper_2609_33977_amd as gm
    T, d = 2048, 4096
    say(f"sparse dX time: g={g}")
    gen = torch.Generator(device="cuda").manual_seed(7)
    W = torch.randn(d, d, generator=gen, device="cuda").mul_(0.02).bfloat16()
    dY = torch.randn(T, d, generator=gen, device="cuda").bfloat16()
    u = torch.rand(d // g, d // g, generator=gen, device="cuda")
    ws = workspace(gm.gm_workspace_size(gm.GM_OP_BWD, T, d, d, g, g))
    dX = empty_bf16(T, d)

    def best(mask):
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                gm.gm_masked_linear_bwd(dY, dY, W, mask, g, dX, None, ws, g_out=g)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    sparse, half = best((u < 0.03).float()), best((u < 0.5).float())
    say(f"  3 % kept {100 * sparse:.1f} us, half kept {100 * half:.1f} us")
    assert sparse < 0.8 * half


@pytest.mark.parametrize("kept", [0.08, 0.6])
@pytest.mark.parametrize("T,d_in,d_out,g", [(140, 320, 336, 16), (257, 576, 1056, 32), (2041, 4096, 800, 32),
                                            (4090, 4096, 272, 16)])
def test_dx_of_pruned_groups_ignores_non_finite_dy(T, d_in, d_out, g, kept):
    # an infinite or NaN dY[t, o] reaches dX[t, i] only through a kept group of (o, i)
    import paper_2609_33977_amd as gm
    say(f"sparse dX, non-finite dY: T={T} d_in={d_in} d_out={d_out} g={g} kept={kept}")
    case = workloads.make_linear_case((302, T, d_in, d_out, g), T, d_in, d_out, g, None, g_out=g)
    r = workloads.gen.rng_for(303, T, g)
    m = (r.uniform(size=case.mask.shape) < kept).astype(np.float32)
    m[m.shape[0] // 2] = 0.0  # a mask row that keeps nothing
    m[1, 0] = 0.75
    bad = {(3, d_out // 2): 0x7F80, (T - 1, 5): 0xFF80, (T // 2, d_out - 1): 0x7FC0}
    dY, hit = case.dY.copy(), np.zeros((T, d_in), dtype=bool)
    clean = case.dY.copy()
    for (t, o), bits in bad.items():
        dY[t, o], clean[t, o] = bits, 0
        hit[t] |= np.repeat(m[o // g] != 0, g)
    dX = empty_bf16(T, d_in)
    ws = workspace(gm.gm_workspace_size(gm.GM_OP_BWD, T, d_in, d_out, g, g))
    gm.gm_masked_linear_bwd(dev_bf16(dY), dev_bf16(case.X), dev_bf16(case.W), dev_f32(m), g, dX, None, ws, g_out=g)
    sync()
    got = host_f64_from_bf16(dX)
    assert not np.any(np.isfinite(got[hit])), "a kept group's infinity or NaN is lost"
    ref, b = ref_dx(oracle.from_bf16(clean), oracle.from_bf16(case.W), m, g, g)
    got[hit], ref[hit] = 0.0, 0.0
    assert_close("dX", got, ref, bound=b)
