// One dgate tile (gemm.hip, square.hip).
#pragma once

#include "gm_gemm.h"
#include "gm_lists.h"

namespace gm {

constexpr int kDgateWaves = 8;

// C[i, o] = sum_t X[t, i] dY[t, o], tile 256 (i) x BN (o); waves 2 (i) x WN (o).
// The epilogue forms dgate[o, v] = sum_{i in v} W[o, i] C[i, o].  For g = 512 a
// group spans two tiles, each adding its half onto a zeroed dgate (two
// addends onto zero: the same sum whichever lands first).
//
// KS = 2: two wave groups split the tokens' slices (contiguous shares, the
// last padded with zero slices) over their own rings, for launches with too
// few 256 x 256 tiles to fill the chip.  The group sums are linear in C, so
// each wave group weights and sums its own part of C, and only the group sums
// are added, in LDS: no accumulators are exchanged (dgate of a 1024 x 1024
// linear at T = 2048: 49 us in 16 256 x 256 tiles, 26 us in 64 256 x 64 tiles).
//
// Blocks past the tiles (when the dX GEMM follows) build the mask's column
// lists, one col_lists_unit each: they start as the first tiles finish, on
// CUs that would otherwise idle through the last tiles' tail (or a partial
// last round of tiles), instead of in a launch of their own before dgate.
struct ListArgs {
  const float* mask;
  int nunits, nchunks, nsub;
  int *colcount, *colsoft, *rows, *subbits;
  float* scales;
};

// u32x4 of LDS: the X rings, then the dY rings; afterwards the group sums.
constexpr int dgate_smem(int BN, int KS) { return KS * (KS * (256 + BN) > 512 ? 3 : 4) * (256 + BN) * 4; }

// bid: this block's number among the launch's dgate blocks (tiles, then list units).
template <int G, int GO, int BN, int KS, bool LISTS>
__device__ __forceinline__ void dgate_tile(const uint16_t* __restrict__ dY, const uint16_t* __restrict__ X,
                                           const uint16_t* __restrict__ W, int T, int d_in, int d_out,
                                           float* __restrict__ dgate, uint16_t* __restrict__ dYt, int ldt,
                                           const ListArgs& la, int bid, u32x4* smem) {
  constexpr int NW = kDgateWaves, NG = NW / KS, WN = NG / 2;  // waves per block, per K group; wave grid 2 (i) x WN (o)
  constexpr int BM = 256, MB = 8, NB = BN / WN / 16;
  constexpr int CA = BM / 16 / NG, CB = BN / 16 / NG;  // copies of the X tile, of the dY tile per wave per slice
  constexpr int PER_STAGE = CA + CB;
  constexpr int STAGES = KS * (BM + BN) > 512 ? 3 : 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NG, wg = wave % NG;  // K group, wave within it
  const int wm = wg / WN, wn = wg % WN;
  const int G_in = d_in / G;
  const int tiles_m = (d_in + BM - 1) / BM, tiles_n = (d_out + BN - 1) / BN, tiles = tiles_m * tiles_n;
  if constexpr (LISTS)
    if (bid >= tiles) {
      col_lists_unit<64 * NW>(bid - tiles, la.nchunks, la.mask, d_out, G_in, GO, la.nsub, la.colcount, la.colsoft, la.rows,
                              la.scales, la.subbits);
      return;
    }
  u32x4(*As)[kBK * BM / 8] = reinterpret_cast<u32x4(*)[kBK * BM / 8]>(smem) + kg * STAGES;
  u32x4(*Bs)[kBK * BN / 8] = reinterpret_cast<u32x4(*)[kBK * BN / 8]>(smem + KS * STAGES * BM * 4) + kg * STAGES;
  int tm, tn;
  tile_coords(bid, tiles, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int all = (T + kBK - 1) / kBK, nst = (all + KS - 1) / KS;
  const int s0 = kg * nst;  // this group's slices: [s0, s0 + nst), those from `all` on zeros

  // Byte offsets of this lane's DMA chunks within a K slice (columns past the
  // matrix read zeros; rows past T fall outside the slice's range).
  uint32_t offA[CA], offB[CB];
#pragma unroll
  for (int j = 0; j < CA; ++j) {
    int row, c;
    mn_dma_target<BM>((wg * CA + j) * 64 + lane, row, c);
    offA[j] = group_voffset(m0 + 8 * c < d_in ? uint32_t(row * d_in + m0 + 8 * c) * 2u : kOOB, j);
  }
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    int row, c;
    mn_dma_target<BN>((wg * CB + j) * 64 + lane, row, c);
    offB[j] = group_voffset(n0 + 8 * c < d_out ? uint32_t(row * d_out + n0 + 8 * c) * 2u : kOOB, j);
  }
  const uint32_t bytesX = uint32_t(T) * uint32_t(d_in) * 2u;
  const uint32_t bytesY = uint32_t(T) * uint32_t(d_out) * 2u;
  i32x4_t rA, rB;  // buffer resources of the slice being copied (zero length past the end)
  auto prepare = [&](int st) {
    const bool live = st < nst && s0 + st < all;
    const int k0 = live ? (s0 + st) * kBK : 0;
    rA = make_rsrc_grouped(X + int64_t(k0) * d_in, live ? bytesX - uint32_t(k0) * uint32_t(d_in) * 2u : 0u);
    rB = make_rsrc_grouped(dY + int64_t(k0) * d_out, live ? bytesY - uint32_t(k0) * uint32_t(d_out) * 2u : 0u);
  };
  const uint32_t ldsA = lds_addr(smem) + uint32_t(kg) * (STAGES * BM * 64);
  const uint32_t ldsB = lds_addr(smem) + uint32_t(KS * STAGES * BM * 64) + uint32_t(kg) * (STAGES * BN * 64);
  auto issue = [&](int st, int p) {  // copies 0 .. CA-1: X tile, CA .. CA+CB-1: dY tile
    if (p < CA)
      dma16_group(p, rA, offA[p], ldsA + (st % STAGES) * (kBK * BM * 2) + wg * CA * 1024);
    else
      dma16_group(p - CA, rB, offB[p - CA], ldsB + (st % STAGES) * (kBK * BN * 2) + wg * CB * 1024);
  };

  // dY^T side output (for the dX GEMM): lane (G, i) of a B fragment holds
  // dY[k0 + 8 G .. k0 + 8 G + 7, o] for o = n0 + wn*NB*16 + nb*16 + i, which is a
  // 16-byte chunk of row o of dY^T.  The tiles sharing this dY panel split
  // the slices between them (slice kt goes to tile row kt * tiles_m / all), and
  // within a tile the two wave rows, which hold the same B fragments, alternate.
  // Buffer stores: one 32-bit offset per lane (out of range for rows past d_out).
  const __amdgpu_buffer_rsrc_t rT =
      __builtin_amdgcn_make_buffer_rsrc(dYt, short(0), int(uint32_t(d_out) * uint32_t(ldt) * 2u), 0x00020000);
  const uint32_t offT = (uint32_t(n0 + wn * NB * 16 + (lane & 15)) * uint32_t(ldt) + 8u * uint32_t(lane >> 4)) * 2u;
  auto bhook = [&](int st, const u32x4(&bf)[NB]) {
    const int kt = s0 + st;
    if (!LISTS || dYt == nullptr || (kt * tiles_m) / all != tm || (kt & 1) != wm) return;
    if (kt * kBK + 8 * (lane >> 4) >= ldt) return;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      __builtin_amdgcn_raw_buffer_store_b128(
          bf[nb], rT,
          n0 + wn * NB * 16 + nb * 16 + (lane & 15) < d_out ? offT + uint32_t(nb * 16 * ldt + kt * kBK) * 2u : kOOB, 0, 0);
  };

  f32x4 acc[MB][NB];
  constexpr int kRowsAfter = 4;  // MFMA rows after the slice's barrier: 2.5-5 % faster than one
  constexpr int RA = CA > 2 ? kRowsAfter - 1 : kRowsAfter;  // four copies' offsets take a row's registers
  gemm_mainloop<MB, NB, false, false, BM, BN, PER_STAGE, STAGES, RA>(
      As, Bs, nst, wm * 128, wn * NB * 16, lane, acc, prepare, issue, [](int) {}, bhook);

  // Epilogue.  Lane (l >> 4, l & 15) holds, for every (mb, nb), rows
  // i = i0 .. i0 + 3 of column o: W[o, i0 .. i0 + 3] is one 8-byte load.  The
  // waves' sums meet in LDS once every wave has left its K-loop (its copies
  // have drained), and are added in a fixed order.
  int el = lane;  // opaque: the epilogue's addresses are not computed (and kept in registers) before the K-loop
  asm volatile("" : "+v"(el));
  const int ibase = m0 + wm * 128 + 4 * (el >> 4);
  float* s_sum = reinterpret_cast<float*>(smem);
  if constexpr (GO > 1) {
    // Square groups (GO = G = 16 .. 128): a 16 x 16 fragment lies inside one
    // group, so each lane sums its products per group of the wave's 128 (i) x
    // 64 (o) sub-tile, and one reduction over the 64 lanes finishes the wave's
    // share of each group.  Groups of 128 rows span two waves (wn pairs).
    static_assert(NB == 4, "64 columns per wave");
    constexpr int IB = 128 / G;                  // groups along i in a wave
    constexpr int OS = GO < 64 ? 64 / GO : 1;    // groups (or group halves) along o in a wave
    float part[IB][OS];
#pragma unroll
    for (int a = 0; a < IB; ++a)
#pragma unroll
      for (int b = 0; b < OS; ++b) part[a][b] = 0.0f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int o = n0 + wn * NB * 16 + nb * 16 + (el & 15);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int i0 = ibase + mb * 16;
        if (o < d_out && i0 < d_in) {
          const uint2 w = *reinterpret_cast<const uint2*>(W + int64_t(o) * d_in + i0);
          part[mb * 16 / G][nb * 16 / (GO < 64 ? GO : 64)] +=
              acc[mb][nb][0] * bf16_lo(w.x) + acc[mb][nb][1] * bf16_hi(w.x) + acc[mb][nb][2] * bf16_lo(w.y) +
              acc[mb][nb][3] * bf16_hi(w.y);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < IB; ++a)
#pragma unroll
      for (int b = 0; b < OS; ++b) {
        float x = part[a][b];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d);
        if (lane == 0) s_sum[(wave * IB + a) * OS + b] = x;
      }
    __syncthreads();
    constexpr int NV = 256 / G, NU = BN / GO;  // groups of the tile along i, along o
    const int b = tid % NU, a = tid / NU;      // at most 256 groups (16 x 16)
    const int u = n0 / GO + b, v = m0 / G + a;
    if (a < NV && u < d_out / GO && v < G_in) {
      auto sum_of = [&](int k, int n) {  // the share of K group k's wave column n
        return s_sum[(((k * 2 + a / IB) * WN + n) * IB + a % IB) * OS + (GO < 64 ? b % OS : 0)];
      };
      float x = 0.0f;
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const float p = GO < 128 ? sum_of(k, b / OS) : sum_of(k, 2 * b) + sum_of(k, 2 * b + 1);
        x = k == 0 ? p : x + p;
      }
      dgate[int64_t(u) * G_in + v] = x;
    }
  } else {
    float part[NB][2];  // per o column: group sums over this wave's first / second 64 rows of i
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int o = n0 + wn * NB * 16 + nb * 16 + (el & 15);
      float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int i0 = ibase + mb * 16;
        if (o < d_out && i0 < d_in) {
          const uint2 w = *reinterpret_cast<const uint2*>(W + int64_t(o) * d_in + i0);
          const float s = acc[mb][nb][0] * bf16_lo(w.x) + acc[mb][nb][1] * bf16_hi(w.x) +
                          acc[mb][nb][2] * bf16_lo(w.y) + acc[mb][nb][3] * bf16_hi(w.y);
          if (mb < MB / 2) s0 += s; else s1 += s;
        }
      }
      // sum over the four lane groups (they hold the other i of the same o)
      s0 += __shfl_xor(s0, 16);
      s0 += __shfl_xor(s0, 32);
      s1 += __shfl_xor(s1, 16);
      s1 += __shfl_xor(s1, 32);
      part[nb][0] = s0;
      part[nb][1] = s1;
    }
    __syncthreads();
    if (lane < 16) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int h = 0; h < 2; ++h) s_sum[((kg * 2 + wm) * 2 + h) * BN + wn * NB * 16 + nb * 16 + lane] = part[nb][h];
    }
    __syncthreads();
    const int o = n0 + tid;
    if (tid < BN && o < d_out) {
      float q[4];  // column o's sums over each 64 rows of i
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        q[h] = s_sum[h * BN + tid];
        if constexpr (KS == 2) q[h] += s_sum[(4 + h) * BN + tid];
      }
      if constexpr (G <= 128) {
        const int v = m0 / G;
#pragma unroll
        for (int a = 0; a < 256 / G; ++a)
          if (v + a < G_in) dgate[int64_t(o) * G_in + v + a] = G == 64 ? q[a] : q[(2 * a) & 3] + q[(2 * a + 1) & 3];
      } else if constexpr (G == 256) {
        dgate[int64_t(o) * G_in + m0 / 256] = (q[0] + q[1]) + (q[2] + q[3]);
      } else {
        atomicAdd(dgate + int64_t(o) * G_in + m0 / 512, (q[0] + q[1]) + (q[2] + q[3]));
      }
    }
  }
}

}  // namespace gm
