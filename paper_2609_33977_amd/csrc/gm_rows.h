// One output row of the packed export on one wave: dot products straight from
// the pieces, shared by the row-per-wave decode kernel and by the tiles of the
// packed GEMM that hold pieces it has no matrix form for.
#pragma once

#include "gm_device.h"

namespace gm {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Dot product of two vectors of 8 bf16 with fp32 accumulation (v_dot2_f32_bf16).
// The bf16 pairs are moved out of the 32-bit lanes with memcpy: a bit_cast of
// a subscripted vector element inside this unrolled loop was folded to element
// 0 by the compiler (every step used the first pair).
__device__ __forceinline__ float dot8_bf16(u32x4 w, u32x4 x) {
  const uint32_t wa[4] = {w.x, w.y, w.z, w.w};
  const uint32_t xa[4] = {x.x, x.y, x.z, x.w};
  float acc = 0.0f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    bf16x2 a, b;
    __builtin_memcpy(&a, &wa[q], sizeof(a));
    __builtin_memcpy(&b, &xa[q], sizeof(b));
    acc = __builtin_amdgcn_fdot2_f32_bf16(a, b, acc, false);
  }
  return acc;
}

// Sums over the wave of TB per-lane values, left in every lane.
template <int TB>
__device__ __forceinline__ void wave_sums(float (&acc)[TB]) {
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    float s = acc[t];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
    acc[t] = s;
  }
}

// acc[t] = sum over pieces p0 .. p0 + nk - 1 of scale * (piece . X[t0 + t, its columns]), t < ntok <= TB, in fp32
// (pieces in any order; those with a column past d_in add nothing).
template <int TB>
__device__ __forceinline__ void packed_row(const uint16_t* __restrict__ X, const uint16_t* __restrict__ Wp,
                                           const int* __restrict__ chunk, const float* __restrict__ scale, int64_t p0,
                                           int nk, int t0, int ntok, int d_in, int g, int lane, float (&acc)[TB]) {
  const int lanes_per_group = g >> 3;
  const int gps = 64 / lanes_per_group;  // pieces per wave step (>= 1 for g <= 512)
  const int slot = lane / lanes_per_group;
  const int e = (lane % lanes_per_group) * 8;
  const int G_in = d_in / g;
#pragma unroll
  for (int t = 0; t < TB; ++t) acc[t] = 0.0f;
  for (int k0 = 0; k0 < nk; k0 += 2 * gps) {
    const int ka = k0 + slot, kb = k0 + gps + slot;
    int va = 0, vb = 0;
    float ma = 0.0f, mb = 0.0f;
    u32x4 wa = zero16(), wb = zero16();
    if (ka < nk) {  // the weights do not wait for the column
      va = chunk[p0 + ka];
      ma = scale[p0 + ka];
      wa = ld16(Wp + (p0 + ka) * g + e);
    }
    if (kb < nk) {
      vb = chunk[p0 + kb];
      mb = scale[p0 + kb];
      wb = ld16(Wp + (p0 + kb) * g + e);
    }
    if (uint32_t(va) >= uint32_t(G_in)) va = 0, ma = 0.0f;
    if (uint32_t(vb) >= uint32_t(G_in)) vb = 0, mb = 0.0f;
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      if (t < ntok) {
        const uint16_t* xr = X + int64_t(t0 + t) * d_in + e;
        float p = 0.0f;
        if (ka < nk) p += ma * dot8_bf16(wa, ld16(xr + int64_t(va) * g));
        if (kb < nk) p += mb * dot8_bf16(wb, ld16(xr + int64_t(vb) * g));
        acc[t] += p;
      }
    }
  }
  wave_sums(acc);
}

// Tokens [t0, t1) of rows o, o + step, ... below o1 of Y on one wave.
__device__ __forceinline__ void packed_rows(const uint16_t* __restrict__ X, const uint16_t* __restrict__ Wp,
                                            const int* __restrict__ chunk, const float* __restrict__ scale,
                                            const int* __restrict__ rowptr, int o, int o1, int step, int t0, int t1,
                                            int d_in, int d_out, int g, int lane, uint16_t* __restrict__ Y) {
  for (; o < o1; o += step) {
    const int p = rowptr[o], nk = rowptr[o + 1] - p;
    for (int t = t0; t < t1; t += 16) {
      const int ntok = min(16, t1 - t);
      float sum[16];
      packed_row<16>(X, Wp, chunk, scale, p, nk, t, ntok, d_in, g, lane, sum);
#pragma unroll
      for (int q = 0; q < 16; ++q)
        if (lane == 0 && q < ntok) Y[int64_t(t + q) * d_out + o] = uint16_t(f32_to_bf16_bits(sum[q]));
    }
  }
}

}  // namespace gm
