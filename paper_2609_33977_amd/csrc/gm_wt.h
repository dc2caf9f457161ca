// out[t, j] = sum_k B[t, k] W'[k, j] with K-contiguous rows of B and W' row-major with K as its row index: the LM
// head's backward (W' the head) and the dX of small square groups (W' the weight with its pruned groups zero).
#pragma once

#include "gm_gemm.h"

namespace gm {

// Tile BM (j) x BN (t) on eight waves: KS wave groups of 2 (j) x NW/KS/2 (t)
// waves split the K slices (contiguous shares, the last padded with zero
// slices).  W' tiles are MN-major (transposing reads), B tiles K-major.
//
// G > 0: W' = W (.) expand(mask) with square G x G groups (G = 16 or 32): the
// 16-byte chunks of a pruned group are zero-filled instead of read, soft
// selectors scale the landed chunks.  The tile's kept bits, one 16-bit word
// of 256 / G groups per mask row, are read once into LDS (at most
// kWtMaskRows mask rows).
constexpr int kWtMaskRows = 2048;

template <int G, int BM, int BN, int KS>
__device__ __forceinline__ void wt_gemm(const uint16_t* __restrict__ B, int ldb, const uint16_t* __restrict__ W, int K,
                                        int d, int N, const float* __restrict__ mask, uint16_t* __restrict__ out) {
  constexpr int NW = 8, NG = NW / KS, WN = NG / 2;
  constexpr int MB = BM / 32, NB = BN / WN / 16;
  constexpr int CA = BM / 16 / NG, CB = BN / 16 / NG, PER_STAGE = CA + CB;
  constexpr int STAGES = KS * (BM + BN) > 512 ? 3 : 4;
  constexpr int HC = BM == 256 ? MB / 4 : MB / 2;
  static_assert(KS == 1 || KS * STAGES * (BM + BN) * 64 >= NW * HC * NB * 1024 + 2 * BM * BN, "LDS");
  __shared__ u32x4 smem[KS * STAGES * (BM + BN) * 4];  // the W rings, then the B rings; afterwards the output tile
  __shared__ uint16_t s_bits[G ? kWtMaskRows : 1];
  __shared__ float s_msoft[G ? STAGES : 1][G ? 64 * NW : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NG, wg = wave % NG, wm = wg / WN, wn = wg % WN;
  u32x4(*As)[kBK * BM / 8] = reinterpret_cast<u32x4(*)[kBK * BM / 8]>(smem) + kg * STAGES;
  u32x4(*Bs)[BN * 4] = reinterpret_cast<u32x4(*)[BN * 4]>(smem + KS * STAGES * BM * 4) + kg * STAGES;
  const int tiles_m = (d + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  int tm, tn;
  tile_coords(gridDim.x, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int all = (K + kBK - 1) / kBK, nst = (all + KS - 1) / KS;
  const int s0 = kg * nst, ng = KS == 1 ? nst : min(nst, all - s0);  // this group's slices [s0, s0 + ng)

  bool soft = false;
  if constexpr (G > 0) {
    // One thread per (mask row, group): the kept bits of a row are one ballot segment.
    constexpr int GT = BM / G, RPW = 64 / GT;  // groups of the tile per mask row, mask rows per wave pass
    const int G_in = d / G, G_out = K / G;
    int any = 0;
    for (int u0 = wave * RPW; u0 < G_out; u0 += NW * RPW * 4) {
      float m[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int u = u0 + i * NW * RPW + lane / GT, v = m0 / G + lane % GT;
        m[i] = u < G_out && v < G_in ? mask[int64_t(u) * G_in + v] : 0.0f;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int u = u0 + i * NW * RPW + lane / GT;
        const uint64_t bal = __ballot(m[i] != 0.0f);
        if (lane % GT == 0 && u < G_out) s_bits[u] = uint16_t((bal >> lane) & ((1ull << GT) - 1));
        any |= m[i] != 0.0f && m[i] != 1.0f;
      }
    }
    soft = __syncthreads_or(any);
  }

  // Byte offsets of this lane's copies within a K slice (columns past the matrix read zeros).
  uint32_t offA[CA], offB[CB];
  int vA[G ? CA : 1];  // group of this lane's W chunk j, from the tile's first
  int cB = 0;          // this lane's chunk of a B row (the same in every copy: its rows are 16 apart)
#pragma unroll
  for (int j = 0; j < CA; ++j) {
    int row, c;
    mn_dma_target<BM>((wg * CA + j) * 64 + lane, row, c);
    offA[j] = group_voffset(m0 + 8 * c < d ? uint32_t(row * d + m0 + 8 * c) * 2u : kOOB, j);
    if constexpr (G > 0) vA[j] = 8 * c / G;
  }
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    int row;
    km_dma_target((wg * CB + j) * 64 + lane, row, cB);
    offB[j] = group_voffset(uint32_t((n0 + row) * ldb + 8 * cB) * 2u, j);
  }
  const uint32_t bytesW = uint32_t(K) * uint32_t(d) * 2u;
  const uint32_t bytesB = uint32_t(N) * uint32_t(ldb) * 2u;
  i32x4_t rA, rB;
  uint32_t dead = 0;  // bit 31: the B chunk starts past K (the last slice's columns there are the next row's)
  // A wave's rows of a slice lie in one mask row (8 or fewer rows, aligned): its kept bits, read one slice ahead.
  constexpr int GG = G ? G : 16;
  constexpr int WR = kBK / NG;  // rows of a slice copied by one wave
  static_assert(GG % WR == 0, "one mask row per wave and slice");
  uint32_t bits = 0, bits_cur = 0;
  auto read_bits = [&](int st) {
    if constexpr (G > 0)
      bits = s_bits[min(((st + s0) * kBK + wg * WR) / G, K / G - 1)];
  };
  read_bits(0);
  auto prepare = [&](int st) {
    const bool live = st < ng;
    const int k0 = live ? (st + s0) * kBK : 0;
    const uint32_t wskip = uint32_t(k0) * uint32_t(d) * 2u;
    rA = make_rsrc_grouped(W + int64_t(k0) * d, live && wskip < bytesW ? bytesW - wskip : 0u);
    rB = make_rsrc_grouped(B + k0, live ? bytesB - 2u * uint32_t(k0) : 0u);
    dead = uint32_t(k0 + 8 * cB >= K) << 31;
    if constexpr (G > 0) bits_cur = ~uint32_t(__builtin_amdgcn_readfirstlane(bits));
    read_bits(st + 1);
  };
  const uint32_t ldsA = lds_addr(smem) + uint32_t(kg) * (STAGES * BM * 64);
  const uint32_t ldsB = lds_addr(smem) + uint32_t(KS * STAGES * BM * 64) + uint32_t(kg) * (STAGES * BN * 64);
  auto issue = [&](int st, int p) {
    if (p < CA)
      dma16_group(p, rA, G ? offA[p] | ((bits_cur >> vA[G ? p : 0]) << 31) : offA[p], ldsA + (st % STAGES) * (BM * 64) + wg * CA * 1024);
    else
      dma16_group(p - CA, rB, offB[p - CA] | dead, ldsB + (st % STAGES) * (BN * 64) + wg * CB * 1024);
  };
  f32x4 acc[MB][NB];
  constexpr int RA = MB > 4 ? 4 : MB / 2;
  auto hook = [](int, const u32x4(&)[NB]) {};
  if (G > 0 && soft) {
    // Each wave also copies the slice's selectors (BM / G groups of the 32 / G
    // mask rows its 32 rows lie in) and scales its own chunks once both landed.
    constexpr int HS = CA > 2 ? 1 : 2;  // chunks scaled at once: the larger tile has fewer registers to spare
    constexpr int gg = G ? G : 16, GT = BM / gg, MR = kBK / gg;
    static_assert(GT * MR <= 64, "one lane per selector");
    const int G_in = d / gg, G_out = K / gg;
    const i32x4_t rM = make_rsrc(mask, uint32_t(G_out) * uint32_t(G_in) * 4u);
    const uint32_t ldsM = lds_addr(s_msoft) + uint32_t(wave) * 256u;
    auto prepare_soft = [&](int st) {
      const int u = (st + s0) * MR + lane / GT, v = m0 / gg + lane % GT;
      const bool ok = st < ng && lane < GT * MR && u < G_out && v < G_in;
      dma4_buf(rM, ok ? (uint32_t(u) * uint32_t(G_in) + uint32_t(v)) * 4u : kOOB,
               ldsM + uint32_t(st % STAGES) * uint32_t(64 * NW * 4));
      prepare(st);
    };
    auto rescale = [&](int st) {
      const float* ms = s_msoft[G ? st % STAGES : 0] + (G ? 64 * wave : 0);
      u32x4* p = As[st % STAGES] + wg * CA * 64 + lane;
#pragma unroll
      for (int h = 0; h < CA; h += HS) {
        float m[HS];
        u32x4 w[HS];
#pragma unroll
        for (int j = 0; j < HS; ++j) {
          m[j] = ms[wg * WR / gg * GT + vA[G ? h + j : 0]];
          w[j] = p[(h + j) * 64];
        }
#pragma unroll
        for (int j = 0; j < HS; ++j)
          if (m[j] != 0.0f && m[j] != 1.0f) p[(h + j) * 64] = scale_bf16x8(w[j], m[j]);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    gemm_mainloop<MB, NB, false, true, BM, 0, PER_STAGE, STAGES, RA, 1>(As, Bs, nst, wm * MB * 16, wn * NB * 16, lane,
                                                                        acc, prepare_soft, issue, rescale, hook);
  } else {
    gemm_mainloop<MB, NB, false, true, BM, 0, PER_STAGE, STAGES, RA>(As, Bs, nst, wm * MB * 16, wn * NB * 16, lane, acc,
                                                                     prepare, issue, [](int) {}, hook);
  }
  if constexpr (KS == 1)
    store_tile_rows<BM, MB, NB, NW>(acc, reinterpret_cast<char*>(smem), reinterpret_cast<char*>(smem + STAGES * BM * 4),
                                    wm, wn, tid, lane, out, d, n0, N, m0, d);
  else
    store_tile_ksum2<BM, BN, MB, NB, NW, HC>(acc, reinterpret_cast<f32x4*>(smem),
                                             reinterpret_cast<char*>(smem) + NW * HC * NB * 1024, kg, wg, wm, wn, tid,
                                             lane, out, d, n0, N, m0, d);
}

}  // namespace gm
