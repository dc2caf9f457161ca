// out[t, j] = sum_k B[t, k] W'[k, j] with K-contiguous rows of B and W' row-major with K as its row index: the LM
// head's backward (W' the head) and the dX of small square groups (W' the weight with its pruned groups zero).
#pragma once

#include "gm_gemm.h"
#include "gm_plan.h"

namespace gm {

// Selectors of a tile's columns (small square groups): per mask row the kept
// bits of the tile's 16-column fragments, and the rows that keep any.
struct WtMask {
  uint16_t bits[kWtMaskRows];
  uint16_t list[kWtMaskRows];
  int nlist, nan;
};

constexpr int wt_stages(int BM, int BN, int KS) { return KS * (BM + BN) > 512 ? 3 : 4; }
constexpr int wt_smem(int BM, int BN, int KS) { return KS * wt_stages(BM, BN, KS) * (BM + BN) * 4; }  // u32x4

// Kept bits of the columns [m0, m0 + BM); returns whether a selector is fractional (uniform).  Ends with a barrier.
template <int G, int BM>
__device__ __forceinline__ bool wt_mask(const float* __restrict__ mask, int G_out, int G_in, int m0, WtMask& sm) {
  constexpr int NW = 8, GT = BM / G, RPW = 64 / GT;  // groups of the tile per mask row, mask rows per wave pass
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  // One thread per (mask row, group): the kept bits of a row are one ballot
  // segment.  Wave 0 then lists the rows that keep any.
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
      uint32_t f = uint32_t(bal >> lane) & ((1u << GT) - 1);
      if constexpr (G == 32) {  // a group is two fragments
        f = (f | f << 4) & 0x0f0fu;
        f = (f | f << 2) & 0x3333u;
        f = (f | f << 1) & 0x5555u;
        f |= f << 1;
      }
      if (lane % GT == 0 && u < G_out) sm.bits[u] = uint16_t(f);
      any |= m[i] != 0.0f && m[i] != 1.0f;
    }
  }
  const bool soft = __syncthreads_or(any);
  if (wave == 0) {
    int cnt = 0;
    for (int ub = 0; ub < G_out; ub += 64) {
      const int u = ub + lane;
      const bool f = u < G_out && sm.bits[u] != 0;
      const uint64_t bal = __ballot(f);
      if (f) sm.list[cnt + __popcll(bal & ((uint64_t(1) << lane) - 1))] = uint16_t(u);
      cnt += __popcll(bal);
    }
    if (lane == 0) sm.nlist = cnt, sm.nan = 0;
  }
  __syncthreads();
  return soft;
}

// The outputs of a tile that came out NaN, from the kept groups alone: a
// pruned group's zeros times a non-finite B would make every output that
// shares its K slices NaN.
template <int G, int BM, int BN>
__device__ __forceinline__ void wt_kept_only(const uint16_t* __restrict__ B, int ldb, const uint16_t* __restrict__ W, int K,
                                          int d, int N, const float* __restrict__ mask, uint16_t* out,
                                          const uint16_t* bits, int m0, int n0) {
  __threadfence();  // the tile's stores
  __syncthreads();
  int e0 = threadIdx.x;  // opaque: nothing here is computed (and kept in registers) before the K-loop
  asm volatile("" : "+v"(e0));
  for (int e = e0; e < BM * BN; e += 512) {
    const int j = m0 + e % BM, t = n0 + e / BM;
    if (j >= d || t >= N) continue;
    uint16_t* o = out + int64_t(t) * d + j;
    if ((*reinterpret_cast<volatile uint16_t*>(o) & 0x7fffu) <= 0x7f80u) continue;
    float a = 0.0f;
    for (int u = 0; u < K / G; ++u) {
      if (!(bits[u] >> (e % BM / 16) & 1)) continue;
      const float m = mask[int64_t(u) * (d / G) + j / G];
#pragma unroll
      for (int q = 0; q < G; ++q) {
        const int k = u * G + q;
        float w = bf16_to_f32(W[int64_t(k) * d + j]);
        if (m != 1.0f) w = bf16_to_f32(uint16_t(f32_to_bf16_bits(m * w)));
        a += bf16_to_f32(B[int64_t(t) * ldb + k]) * w;
      }
    }
    *o = uint16_t(f32_to_bf16_bits(a));
  }
}

// Tile BM (j) x BN (t) on eight waves: KS wave groups of 2 (j) x NW/KS/2 (t)
// waves split the K slices (contiguous shares, the last padded with zero
// slices).  W' tiles are MN-major (transposing reads), B tiles K-major.
//
// G > 0: W' = W (.) expand(mask) with square G x G groups (G = 16 or 32): the
// 16-byte chunks of a pruned group are zero-filled instead of read, soft
// selectors scale the landed chunks.  WALK: K runs over the listed mask rows
// only, one to a K slice, or two of 16.
template <int G, int BM, int BN, int KS, bool WALK>
__device__ __forceinline__ void wt_tile(const uint16_t* __restrict__ B, int ldb, const uint16_t* __restrict__ W, int K,
                                        int d, int N, const float* __restrict__ mask, uint16_t* __restrict__ out,
                                        u32x4* smem, WtMask* sm, float* s_msoft, int m0, int n0, bool soft) {
  constexpr int NW = 8, NG = NW / KS, WN = NG / 2;
  constexpr int MB = BM / 32, NB = BN / WN / 16;
  constexpr int CA = BM / 16 / NG, CB = BN / 16 / NG, PER_STAGE = CA + CB;
  constexpr int STAGES = wt_stages(BM, BN, KS);
  constexpr int HC = BM == 256 ? MB / 4 : MB / 2;
  constexpr int GG = G ? G : 16, GT = BM / GG;  // groups of the tile per mask row
  constexpr bool PAIR = WALK && G == 16;        // a slice is two mask rows, anywhere
  static_assert(KS == 1 || wt_smem(BM, BN, KS) * 16 >= NW * HC * NB * 1024 + 2 * BM * BN, "LDS");
  static_assert(G == 0 || BM / 16 <= 16, "fragment bits");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NG, wg = wave % NG, wm = wg / WN, wn = wg % WN;
  // smem: the W rings, then the B rings; afterwards the output tile
  u32x4(*As)[kBK * BM / 8] = reinterpret_cast<u32x4(*)[kBK * BM / 8]>(smem) + kg * STAGES;
  u32x4(*Bs)[BN * 4] = reinterpret_cast<u32x4(*)[BN * 4]>(smem + KS * STAGES * BM * 4) + kg * STAGES;
  const int nlist = WALK ? __builtin_amdgcn_readfirstlane(sm->nlist) : 0;
  const int all = ((WALK ? nlist * GG : K) + kBK - 1) / kBK, nst = (all + KS - 1) / KS;
  const int s0 = kg * nst, ng = KS == 1 ? nst : min(nst, all - s0);  // this group's slices [s0, s0 + ng)

  // Byte offsets of this lane's copies within a K slice (columns past the matrix read zeros).  A wave's W rows lie in
  // one mask row; in a slice of a pair, they lie in its half `half` and this lane's chunk of a B row in half cB / 2.
  constexpr int WR = kBK / NG;  // rows of a slice copied by one wave
  static_assert(GG % WR == 0, "one mask row per wave and slice");
  const int half = PAIR ? wg * WR / 16 : 0;
  uint32_t offA[CA], offB[CB];
  uint32_t vA = 0;  // bits 5 j .. 5 j + 4: fragment of this lane's W chunk j
  int cB = 0;       // this lane's chunk of a B row (the same in every copy: its rows are 16 apart)
#pragma unroll
  for (int j = 0; j < CA; ++j) {
    int row, c;
    mn_dma_target<BM>((wg * CA + j) * 64 + lane, row, c);
    offA[j] = group_voffset(m0 + 8 * c < d ? uint32_t((row - 16 * half) * d + m0 + 8 * c) * 2u : kOOB, j);
    vA |= uint32_t(c / 2) << (5 * j);
  }
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    int row;
    km_dma_target((wg * CB + j) * 64 + lane, row, cB);
    offB[j] = group_voffset(uint32_t((n0 + row) * ldb + 8 * (PAIR ? cB & 1 : cB)) * 2u, j);
  }
  const uint32_t bytesW = uint32_t(K) * uint32_t(d) * 2u;
  const uint32_t bytesB = uint32_t(N) * uint32_t(ldb) * 2u;
  i32x4_t rA, rB;
  uint32_t pastB = 0;              // bit 31: the B chunk starts past K (the last slice's columns there are the next row's)
  uint32_t col0 = 0, col1 = 0;     // a pair's columns of B (byte offsets)
  // Kept bits of this wave's W rows, read one slice ahead; WALK: and the mask
  // rows of a slice, read two ahead (u: of the next slice, v: of the one after).
  uint32_t bits = 0, dead = 0;  // dead: bit f: fragment f is pruned in this slice's rows
  int u0 = 0, u1 = 0, v0 = 0, v1 = 0;
  auto read_rows = [&](int st) {
    if constexpr (PAIR) {
      v0 = sm->list[max(min(2 * (st + s0), nlist - 1), 0)];
      v1 = 2 * (st + s0) + 1 < nlist ? sm->list[2 * (st + s0) + 1] : -1;  // an empty half
    } else if constexpr (WALK) {
      v0 = sm->list[max(min(st + s0, nlist - 1), 0)];
    }
  };
  auto advance = [&](int st) {  // to slice st
    if constexpr (WALK) {
      u0 = __builtin_amdgcn_readfirstlane(v0);
      if constexpr (PAIR) u1 = __builtin_amdgcn_readfirstlane(v1);
      bits = sm->bits[half ? max(u1, 0) : u0];
      read_rows(st + 1);
    } else if constexpr (G > 0) {
      bits = sm->bits[min(((st + s0) * kBK + wg * WR) / G, K / G - 1)];
    }
  };
  read_rows(0);
  advance(0);
  auto prepare = [&](int st) {
    const bool live = st < ng;
    if constexpr (G > 0) dead = ~uint32_t(__builtin_amdgcn_readfirstlane(bits));
    if constexpr (WALK) {
      const int k0 = (half && u1 >= 0 ? u1 : u0) * G;
      if (half && u1 < 0) dead = ~0u;
      rA = make_rsrc_grouped(W + int64_t(k0) * d, live ? bytesW - uint32_t(k0) * uint32_t(d) * 2u : 0u);
      if constexpr (PAIR) {  // (an empty half repeats the other's columns of B)
        rB = make_rsrc_grouped(B, live ? bytesB : 0u);
        col0 = uint32_t(u0) * 32u;
        col1 = uint32_t(u1 < 0 ? u0 : u1) * 32u;
      } else {
        rB = make_rsrc_grouped(B + k0, live ? bytesB - 2u * uint32_t(k0) : 0u);
      }
    } else {
      const int k0 = live ? (st + s0) * kBK : 0;
      const uint32_t wskip = uint32_t(k0) * uint32_t(d) * 2u;
      rA = make_rsrc_grouped(W + int64_t(k0) * d, live && wskip < bytesW ? bytesW - wskip : 0u);
      rB = make_rsrc_grouped(B + k0, live ? bytesB - 2u * uint32_t(k0) : 0u);
      pastB = uint32_t(k0 + 8 * cB >= K) << 31;
    }
    advance(st + 1);
  };
  const uint32_t ldsA = lds_addr(smem) + uint32_t(kg) * (STAGES * BM * 64);
  const uint32_t ldsB = lds_addr(smem) + uint32_t(KS * STAGES * BM * 64) + uint32_t(kg) * (STAGES * BN * 64);
  auto issue = [&](int st, int p) {
    if (p < CA)
      dma16_group(p, rA, G ? offA[p] | ((dead >> ((vA >> (5 * p)) & 31)) << 31) : offA[p], ldsA + (st % STAGES) * (BM * 64) + wg * CA * 1024);
    else
      dma16_group(p - CA, rB, PAIR ? offB[p - CA] + (cB < 2 ? col0 : col1) : offB[p - CA] | pastB, ldsB + (st % STAGES) * (BN * 64) + wg * CB * 1024);
  };
  f32x4 acc[MB][NB];
  constexpr int RA = WALK && CA > 2 ? 3 : MB > 4 ? 4 : MB / 2;  // (four copies and the lists take a row's registers)
  auto hook = [](int, const u32x4(&)[NB]) {};
  if (G > 0 && soft) {
    // Each wave also copies the slice's selectors (BM / G groups of its one or
    // two mask rows) and scales its own chunks once both landed.
    constexpr int HS = CA > 2 ? 1 : 2;  // chunks scaled at once: the larger tile has fewer registers to spare
    constexpr int MR = kBK / GG;
    static_assert(GT * MR <= 64, "one lane per selector");
    const int G_in = d / GG, G_out = K / GG;
    const i32x4_t rM = make_rsrc(mask, uint32_t(G_out) * uint32_t(G_in) * 4u);
    const uint32_t ldsM = lds_addr(s_msoft) + uint32_t(wave) * 256u;
    auto prepare_soft = [&](int st) {
      int el = lane;  // opaque in the largest tile: nothing is computed from it (and kept in registers) before the K-loop
      if constexpr (CA > 2) asm volatile("" : "+v"(el));
      const int u = WALK ? (el < GT ? u0 : u1) : (st + s0) * MR + el / GT, v = m0 / GG + el % GT;
      const bool ok = st < ng && el < GT * MR && u >= 0 && u < G_out && v < G_in;
      dma4_buf(rM, ok ? (uint32_t(u) * uint32_t(G_in) + uint32_t(v)) * 4u : kOOB,
               ldsM + uint32_t(st % STAGES) * uint32_t(64 * NW * 4));
      prepare(st);
    };
    auto rescale = [&](int st) {
      const float* ms = s_msoft + (st % STAGES) * 64 * NW + 64 * wave;
      uint32_t va = vA;  // opaque, as above
      if constexpr (CA > 2) asm volatile("" : "+v"(va));
      u32x4* p = As[st % STAGES] + wg * CA * 64 + lane;
#pragma unroll
      for (int h = 0; h < CA; h += HS) {
        float m[HS];
        u32x4 w[HS];
#pragma unroll
        for (int j = 0; j < HS; ++j) {
          m[j] = ms[wg * WR / GG * GT + ((va >> (5 * (h + j))) & 31) * 16 / GG];
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
  int et = tid, el = lane;  // opaque: the epilogue's addresses are not computed (and kept in registers) before the K-loop
  asm volatile("" : "+v"(et), "+v"(el));
  if constexpr (G > 0)
    if (any_nan(acc)) sm->nan = 1;
  if constexpr (KS == 1)
    store_tile_rows<BM, MB, NB, NW>(acc, reinterpret_cast<char*>(smem), reinterpret_cast<char*>(smem + STAGES * BM * 4),
                                    wm, wn, et, el, out, d, n0, N, m0, d);
  else
    store_tile_ksum2<BM, BN, MB, NB, NW, HC>(acc, reinterpret_cast<f32x4*>(smem),
                                             reinterpret_cast<char*>(smem) + NW * HC * NB * 1024, kg, wg, wm, wn, et,
                                             el, out, d, n0, N, m0, d);
  if constexpr (G > 0)
    if (sm->nan)  // (visible: the stores above have barriers)
      wt_kept_only<G, BM, BN>(B, ldb, W, K, d, N, mask, out, sm->bits, m0, n0);
}

// Every row of W'.
template <int BM, int BN, int KS>
__device__ __forceinline__ void wt_gemm(const uint16_t* __restrict__ B, int ldb, const uint16_t* __restrict__ W, int K,
                                        int d, int N, uint16_t* __restrict__ out) {
  __shared__ u32x4 smem[wt_smem(BM, BN, KS)];
  int tm, tn;
  tile_coords(gridDim.x, (d + BM - 1) / BM, (N + BN - 1) / BN, tm, tn);
  wt_tile<0, BM, BN, KS, false>(B, ldb, W, K, d, N, nullptr, out, smem, nullptr, nullptr, tm * BM, tn * BN, false);
}

// Small square groups.  The walk over the listed rows costs 3-10 % per slice
// (pairs of 16-row entries most), so it is taken where it drops at least one
// mask row in 16.  4096 x 4096, T = 2048, 32 x 32 groups, us with the walk / with
// every slice: 3 % kept 26 / 65, 10 % 47 / 65, 20 % 59 / 65, half kept 66 (no
// walk); 16 x 16: 38 / 66, 61 / 66, 20 % 66 (no walk).  Skipping the MFMAs of a pruned
// fragment as well was 5-20 % slower from 30 % kept on and level below; narrower
// tiles of the same block (half the columns each, over their own rows) gained
// 4-15 % below 20 % kept in the 256 x 128 tile and lost in the others.
template <int G, int BM, int BN, int KS>
__device__ __forceinline__ void wt_gemm_masked(const uint16_t* __restrict__ B, int ldb, const uint16_t* __restrict__ W,
                                               int K, int d, int N, const float* __restrict__ mask,
                                               uint16_t* __restrict__ out, int bid, int blocks, u32x4* smem, WtMask& sm,
                                               float* s_msoft) {
  int tm, tn;
  tile_coords(bid, blocks, (d + BM - 1) / BM, (N + BN - 1) / BN, tm, tn);
  const bool soft = wt_mask<G, BM>(mask, K / G, d / G, tm * BM, sm);
  if (sm.nlist * 16 < K / G * 15)
    wt_tile<G, BM, BN, KS, true>(B, ldb, W, K, d, N, mask, out, smem, &sm, s_msoft, tm * BM, tn * BN, soft);
  else
    wt_tile<G, BM, BN, KS, false>(B, ldb, W, K, d, N, mask, out, smem, &sm, s_msoft, tm * BM, tn * BN, soft);
}

}  // namespace gm
