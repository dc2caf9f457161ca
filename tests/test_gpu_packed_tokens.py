"""GPU parity of the packed forward beyond 16 tokens against the fp64 oracle: fractional selectors, which keep their 32
bits on every path, pieces out of column order, ragged rows and tokens, and what a fractional selector costs."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_support import assert_close, dev_bf16, dev_f32, empty_bf16, host_bits, host_f64_from_bf16, say, sync

pytestmark = pytest.mark.gpu


def _pack(W, m, g, g_out=1):
    import torch
    import paper_2609_33977_amd as gm
    cap = max(int((m != 0).sum().item()) * g_out, 1)
    Wp = torch.zeros((cap, g), dtype=torch.bfloat16, device="cuda")
    chunk = torch.zeros(cap, dtype=torch.int32, device="cuda")
    scale = torch.zeros(cap, dtype=torch.float32, device="cuda")
    rowptr = torch.zeros(W.shape[0] + 1, dtype=torch.int32, device="cuda")
    gm.gm_pack_rows(W, m, g, cap, Wp, chunk, scale, rowptr, g_out=g_out)
    return Wp, chunk, scale, rowptr


def _bound(X, W, mask, g, g_out, ref):
    # fp32 products with the selectors and fp32 sums (twice the worst case), then one rounding to bf16: no rounded weights
    S = oracle.linear_fwd(np.abs(X), np.abs(W), mask, g, g_out)
    acc = 2.0 * (X.shape[1] + 2) * 2.0 ** -24 * S
    return 2.0 ** -8 * (np.abs(ref) + acc) + acc


def _shuffled(packed, rows):
    import torch
    Wp, chunk, scale, rowptr = packed
    rp = rowptr.cpu().numpy()
    perm = np.arange(chunk.numel())
    for o in rows:
        perm[rp[o]:rp[o + 1]] = perm[rp[o]:rp[o + 1]][::-1]
    p = torch.from_numpy(perm).cuda()
    return Wp[p].contiguous(), chunk[p].contiguous(), scale[p].contiguous(), rowptr


@pytest.mark.parametrize("kind", ["every", "one", "shuffled"])
@pytest.mark.parametrize("T,d_in,d_out,g", [
    (17, 64, 8, 64),          # one group; the second pass has one token
    (31, 1536, 520, 512),
    (33, 320, 160, 32),       # rows of 16 past the last full block of 32
    (40, 512, 336, 16),       # two groups in a slice
    (48, 4096, 1000, 64),
    (20, 12288, 48, 16),      # more groups in a row than the tables hold
    (300, 2048, 264, 128),    # 128 x 128 tiles
    (300, 1024, 272, 16),
    (1000, 320, 288, 32),
    (129, 13824, 136, 256),
    (2040, 512, 4088, 256),   # 256 x 128 tiles
    (4090, 512, 4088, 128),   # 256 x 256 tiles
])
def test_packed_fractional_selectors(T, d_in, d_out, g, kind):
    import paper_2609_33977_amd as gm
    say(f"packed, fractional selectors ({kind}): T={T} d_in={d_in} d_out={d_out} g={g}")
    g_out = g if g < 64 else 1
    case = workloads.make_linear_case((310, T, d_in, d_out, g), T, d_in, d_out, g, None, g_out=g_out)
    r = workloads.gen.rng_for(311, T, g)
    mask = case.mask.astype(np.float32).copy()
    if kind == "every":
        mask *= r.uniform(0.05, 1.5, size=mask.shape).astype(np.float32)
    else:
        mask[-1, 0] = 0.37
    X, W, m = dev_bf16(case.X), dev_bf16(case.W), dev_f32(mask)
    packed = _pack(W, m, g, g_out)
    if kind == "shuffled":
        packed = _shuffled(packed, [0, d_out // 2])
    Y, again = empty_bf16(T, d_out), empty_bf16(T, d_out)
    gm.gm_packed_linear_fwd(X, *packed, d_out, g, Y)
    gm.gm_packed_linear_fwd(X, *packed, d_out, g, again)
    sync()
    Xo, Wo = oracle.from_bf16(case.X), oracle.from_bf16(case.W)
    ref = oracle.linear_fwd(Xo, Wo, mask, g, g_out)
    assert_close("Y", host_f64_from_bf16(Y), ref, bound=_bound(Xo, Wo, mask, g, g_out, ref))
    assert np.array_equal(host_bits(Y), host_bits(again))


def _best(fn):
    import torch
    times = []
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            fn()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


def _layer(T, d_out, d_in, g, soft):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(11)
    X = torch.randn(T, d_in, generator=gen, device="cuda").bfloat16()
    W = torch.randn(d_out, d_in, generator=gen, device="cuda").mul_(0.02).bfloat16()
    u = torch.rand(d_out, d_in // g, generator=gen, device="cuda")
    return X, _pack(W, (u < 0.5).float() * ((0.5 + u) if soft else 1.0), g), empty_bf16(T, d_out)


@pytest.mark.parametrize("T", [128, 512])
def test_a_fractional_export_costs_little_more_than_a_binary_one(T):
    # 2.0 times the binary export; one wave per row inside the tile took 40 times it
    import paper_2609_33977_amd as gm
    d, g = 4096, 128
    (X, hard, Y), (_, soft, _) = _layer(T, d, d, g, False), _layer(T, d, d, g, True)
    h = _best(lambda: gm.gm_packed_linear_fwd(X, *hard, d, g, Y))
    s = _best(lambda: gm.gm_packed_linear_fwd(X, *soft, d, g, Y))
    say(f"packed, T={T}: binary {100 * h:.1f} us, fractional {100 * s:.1f} us")
    assert s < 4.0 * h


PASSES = [
    (17, 512, 8, 512),
    (32, 8256, 5120, 64),     # 129 groups per row: 16-row blocks
    (47, 4096, 5128, 128),    # 32-row blocks, 8 rows past the last
    (64, 1024, 1056, 32),
    (33, 16384, 64, 32),      # 512 groups per row
    (18, 5120, 4112, 16),     # 320 groups per row
]


@pytest.mark.parametrize("T,d_in,d_out,g", PASSES)
def test_packed_passes_of_16_tokens(T, d_in, d_out, g):
    import paper_2609_33977_amd as gm
    say(f"packed passes: T={T} d_in={d_in} d_out={d_out} g={g}")
    g_out = g if g < 64 else 1
    case = workloads.make_linear_case((312, T, d_in, d_out, g), T, d_in, d_out, g, None, g_out=g_out)
    mask = case.mask.astype(np.float32).copy()
    mask[0], mask[-1, 1:] = 0.0, 0.0
    X, m = dev_bf16(case.X), dev_f32(mask)
    packed = _pack(dev_bf16(case.W), m, g, g_out)
    Y = empty_bf16(T, d_out)
    gm.gm_packed_linear_fwd(X, *packed, d_out, g, Y)
    sync()
    Xo, Wo = oracle.from_bf16(case.X), oracle.from_bf16(case.W)
    ref = oracle.linear_fwd(Xo, Wo, mask, g, g_out)
    assert_close("Y", host_f64_from_bf16(Y), ref, bound=_bound(Xo, Wo, mask, g, g_out, ref))


def test_one_token_more_than_16_costs_little():
    # 10 us both, with the calls' own time (12 and 14 us for the kernels); 44 us in the GEMM's eight 128 x 128 tiles
    import paper_2609_33977_amd as gm
    d_out, d_in, g = 1024, 4096, 64
    X, packed, Y = _layer(17, d_out, d_in, g, False)
    a = _best(lambda: gm.gm_packed_linear_fwd(X[:16], *packed, d_out, g, Y[:16]))
    b = _best(lambda: gm.gm_packed_linear_fwd(X, *packed, d_out, g, Y))
    say(f"packed {d_out} x {d_in}: 16 tokens {100 * a:.1f} us, 17 tokens {100 * b:.1f} us")
    assert b < 3.0 * a


@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("T,d_in,d_out,g", [
    (17, 1024, 264, 128),     # passes
    (300, 1024, 272, 16),     # 128 x 128 tiles
    (300, 2048, 520, 256),
    (2040, 512, 4088, 256),   # 256 x 128 tiles
    (4090, 512, 4088, 128),   # 256 x 256 tiles
])
def test_packed_pruned_groups_ignore_non_finite_x(T, d_in, d_out, g, soft):
    # an infinite or NaN X[t, i] reaches Y[t, o] only through a kept group of (o, i)
    import paper_2609_33977_amd as gm
    say(f"packed, non-finite X: T={T} d_in={d_in} d_out={d_out} g={g} soft={soft}")
    g_out = g if g < 64 else 1
    case = workloads.make_linear_case((313, T, d_in, d_out, g), T, d_in, d_out, g, None, g_out=g_out)
    r = workloads.gen.rng_for(314, T, g)
    mask = (r.uniform(size=case.mask.shape) < 0.4).astype(np.float32)
    if soft:
        mask *= r.uniform(0.05, 1.5, size=mask.shape).astype(np.float32)
    bad = {(0, 3): 0x7F80, (T - 1, d_in - 1): 0xFF80, (T // 2, d_in // 2): 0x7FC0}
    X, clean, hit = case.X.copy(), case.X.copy(), np.zeros((T, d_out), dtype=bool)
    for (t, i), bits in bad.items():
        X[t, i], clean[t, i] = bits, 0
        hit[t] |= np.repeat(mask[:, i // g] != 0, g_out)
    packed = _pack(dev_bf16(case.W), dev_f32(mask), g, g_out)
    Y = empty_bf16(T, d_out)
    gm.gm_packed_linear_fwd(dev_bf16(X), *packed, d_out, g, Y)
    sync()
    got = host_f64_from_bf16(Y)
    assert not np.any(np.isfinite(got[hit])), "a kept group's infinity or NaN is lost"
    Xo, Wo = oracle.from_bf16(clean), oracle.from_bf16(case.W)
    ref = oracle.linear_fwd(Xo, Wo, mask, g, g_out)
    b = _bound(Xo, Wo, mask, g, g_out, ref)
    got[hit], ref[hit] = 0.0, 0.0
    assert_close("Y", got, ref, bound=b)
