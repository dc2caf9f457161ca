// bf16 MFMA GEMMs of the group-masked linear layer on gfx950.
//
//   fwd   Y[t, o]     = sum_v mask[u(o), v] sum_{i in v} X[t, i] W[o, i]        (Eq. 1)
//   dX    dX[t, i]    = sum_{o kept in column v(i)} mask[u(o), v] dY[t, o] W[o, i]
//   dgate dgate[u, v] = sum_{o in u, i in v} W[o, i] sum_t dY[t, o] X[t, i]
//
// Groups are g_out x g blocks (Sec. 2.1): u(o) = o / g_out is the mask row of
// output row o, v(i) = i / g its mask column; 1 x g groups have g_out = 1.
//
// Shared machinery (gm_gemm.h, gm_pipe.h): 256 x 256 output tiles (smaller ones,
// most with K over two wave groups, for launches that would leave the chip part
// empty; dX: at most max(g, 64) rows), eight waves of 128 x 64 (dX tiles of 64 rows:
// four waves of 32 x 128) accumulated in AGPRs and VGPRs with
// v_mfma_f32_16x16x32_bf16, and a four-stage pipeline of 32-deep K slices
// copied global -> LDS by buffer loads with the lds modifier (no registers in
// flight), with one block barrier per slice.  Each lane keeps a fixed 32-bit
// byte offset per copy; the K advance lives in the scalar buffer resource,
// and out-of-range offsets read zeros (padding, ragged tails, pruned groups).
// M is always the dimension that is contiguous in the output, so every lane
// stores 4 adjacent bf16 (8 bytes).
//
// Operand tiles:
//   fwd   W rows and X rows are K-contiguous: K-major tiles, ds_read_b128.
//         A pruned group is never read: its copy lanes get an out-of-range offset.
//         The K-loop visits only group columns that some row of the tile keeps.
//   dgate X and dY are stored [T, .]: K (= tokens) is the row index, so the
//         tiles are MN-major and fragments come from ds_read_b64_tr_b16.
//         Epilogue: the fp32 tile of X^T dY is multiplied by W and summed over
//         each group in registers and across lanes; dY^T X never reaches HBM.
//         The transposing reads of dY are 16-byte chunks of dY^T, which the
//         first row of tiles stores for the dX GEMM.
//   dX    K = the kept rows of one group column (its column list): whole rows
//         of W and of dY^T are gathered, MN-major tiles, transposing reads.
#include "gm_dgate.h"
#include "gm_gemm.h"
#include "gm_launch.h"
#include "gm_lists.h"
#include "gm_rows.h"

namespace gm {

// Waves per block of the GEMMs: eight waves of 128 x 64 per 256 x 256 tile,
// two per SIMD, so one wave's copy issue and barrier wait hide behind the
// other's MFMAs.
constexpr int kFwdWaves = 8;
constexpr int kDxWaves = 8;
// dX: 8 waves for tiles of 128 and 256 rows; the 64-row tile keeps 4 (its W
// slice is four copies, one per wave).
constexpr int dx_waves(int bm, int ks) { return bm >= 128 || ks > 1 ? kDxWaves : 4; }

// MFMA rows of a wave tile issued after each slice's barrier (the K-loop's RA):
// four for the forward (2.5-5 % faster than one), one for dX (level).
constexpr int kFwdRowsAfter = 4, kDxRowsAfter = 1;

// ============================================================================ fwd

// C[o, t] over K = d_in, tile BM (o) x BM (t).
//
// The K-loop walks column units of U = max(g, 32) input columns (a 16-wide
// group shares its 32-deep slice with its neighbour) and visits only the
// units that some row of the tile keeps; inside a visited unit each 16-byte
// chunk of W whose group is pruned for its row is zero-filled instead of read.
//
// Split K (ksplit > 1, 256 x 256 and 128 x 128 tiles, for launches with fewer tiles than half the CUs):
// block b works on tile b / ksplit and takes share b % ksplit of the tile's
// list of visited units (contiguous, in order), and stores its fp32 partial
// tile into part[share][t][o]; fwd_reduce_kernel then adds the shares in
// order and rounds once.
//
// KS wave groups per block split the block's slices (contiguous shares, the
// last one padded with zero slices so that every wave meets every barrier)
// over their own LDS rings and add their tiles in LDS: a 128 x 128 tile with
// KS = 2 keeps eight waves of 64 x 64 busy, where a launch has too few 256 x
// 256 tiles to fill the chip.
//
// PACKED: W is the row-packed export (Appendix F): pieces of g weights, the
// row's kept groups in column order from rowptr[o]; scale holds their
// selectors.  The piece of (row, group) is the row's first piece plus the
// number of kept groups before it, from the tile's kept bits (built in the
// prologue from chunk[]) and a running count per 32-bit word.  A tile with a
// fractional selector (which this K-loop would round into bf16 weights) multiplies
// each slice's products by it in fp32 instead; a tile with pieces out of column
// order computes its rows piece by piece (packed_row).
struct PackedArgs {
  const int *chunk, *rowptr;
  const float* scale;
};

template <int G, int GO, int BM, int BN, int KS, bool PACKED>
__global__ __launch_bounds__(64 * kFwdWaves) void fwd_kernel(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
                                                  const float* __restrict__ mask, int T, int d_in, int d_out,
                                                  uint16_t* __restrict__ Y, int ksplit, float* __restrict__ part,
                                                  PackedArgs pk) {
  constexpr int NW = kFwdWaves, NG = NW / KS;  // waves per block, per K group
  constexpr int WN = NG / 2;                   // wave grid of a K group: 2 (M) x WN (N)
  constexpr int MB = BM / 32, NB = BN / WN / 16;
  constexpr int U = G < kBK ? kBK : G;        // input columns of one unit
  constexpr int UG = U / G;                   // groups per unit (2 for g = 16)
  constexpr int SUB = U / kBK;                // K slices per unit
  constexpr int RB = BM / GO;                 // mask rows met by one tile
  // selectors and units per mask row (fwd_tile_fits): the tiles with less LDS to spare hold shorter rows
  constexpr int MAXG = GO == 1 && BM == 256 && (PACKED || KS > 1) ? fwd_max_groups(G, PACKED, KS > 1)
                       : GO == 1 && G > 16                        ? 512
                                                                  : 1024;
  constexpr int MAXU = MAXG / UG < 512 ? MAXG / UG : 512;
  constexpr int CA = BM / 16 / NG, CB = BN / 16 / NG;  // copies of the W tile, of the X tile per wave per slice
  constexpr int PER_STAGE = CA + CB;          // DMA instructions per wave per slice
  constexpr int STAGES = (PACKED && G == 16) || BM * KS > 256 ? 3 : 4;
  constexpr int HC = BM == 256 ? MB / 4 : MB / 2;  // fragment rows exchanged at once between two K groups
  static_assert(GO == 1 || GO == G, "groups are 1 x g or square");
  static_assert(KS == 1 || (KS == 2 && KS * STAGES * (BM + BN) * 64 >= NW * HC * NB * 1024 + 2 * BM * BN), "LDS");
  static_assert(!PACKED || GO == 1, "the export holds row pieces");
  __shared__ u32x4 smem[KS * STAGES * (BM + BN) * 4];  // the A rings, then the B rings; afterwards the output tile
  u32x4(*As)[BM * 4] = reinterpret_cast<u32x4(*)[BM * 4]>(smem);
  u32x4(*Bs)[BN * 4] = reinterpret_cast<u32x4(*)[BN * 4]>(smem + KS * STAGES * BM * 4);
  __shared__ uint32_t s_bits[RB][MAXG / 32];  // kept bits of the tile's mask rows
  __shared__ int s_base[PACKED ? RB : 1][MAXG / 32];  // packed: piece (from the tile's first) of the word's first kept group
  __shared__ uint32_t s_any[MAXU / 32];       // unit kept by some row of the tile
  __shared__ int s_cols[MAXU];
  __shared__ uint32_t s_live[GO >= 32 ? MAXU : 1];  // per listed unit: bit f = 16-row fragment f of the tile keeps it
  __shared__ int s_ncols, s_soft, s_nan;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NG, wg = wave % NG;  // K group, wave within it
  const int wm = wg / WN, wn = wg % WN;
  const int G_in = d_in / G, NU = d_in / U;
  const int tiles_m = (d_out + BM - 1) / BM, tiles_n = (T + BN - 1) / BN;
  const int share = int(blockIdx.x) % ksplit;
  int tm, tn;
  tile_coords(int(blockIdx.x) / ksplit, int(gridDim.x) / ksplit, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;

  // Prologue: kept bits of every mask row of the tile, the units some row keeps, soft values.
  if (tid < MAXU / 32) s_any[tid] = 0;
  if (tid == 0) {
    s_soft = 0;
    if constexpr (PACKED) s_nan = 0;
    s_cols[0] = 0;  // read (unused) by the zero-fill copies when no unit is kept
  }
  const int words = (G_in + 31) / 32;
  // units of the 32 groups of word w with kept bits b
  auto mark_units = [&](int w, uint32_t b) {
    if constexpr (UG == 1) {
      if (b) atomicOr(&s_any[w], b);
    } else {
      // 16-wide groups: unit u holds groups 2u and 2u + 1; pack the pairs' ORs
      uint32_t u = (b | (b >> 1)) & 0x55555555u;
      u = (u | (u >> 1)) & 0x33333333u;
      u = (u | (u >> 2)) & 0x0f0f0f0fu;
      u = (u | (u >> 4)) & 0x00ff00ffu;
      u = (u | (u >> 8)) & 0x0000ffffu;
      if (u) atomicOr(&s_any[w >> 1], u << (16 * (w & 1)));
    }
  };
  int p0 = 0, np = 0;  // packed: the tile's first piece and number of pieces
  if constexpr (PACKED) {
    // TPR threads per row walk its pieces, eight loads at a time.
    constexpr int TPR = 64 * NW / RB, LP = 8;
    const int rows = min(RB, d_out - m0);
    const int r = tid / TPR;
    p0 = pk.rowptr[m0];
    np = pk.rowptr[m0 + rows] - p0;
    const int rp0 = r < rows ? pk.rowptr[m0 + r] : 0, rp1 = r < rows ? pk.rowptr[m0 + r + 1] : 0;
    for (int e = tid; e < RB * words; e += 64 * NW) s_bits[e % RB][e / RB] = 0;
    __syncthreads();
    bool odd = false, soft = false;
    for (int e = rp0 + tid % TPR; e < rp1; e += TPR * LP) {
      int v[LP], before[LP];
      float m[LP];
#pragma unroll
      for (int i = 0; i < LP; ++i) {
        const int p = e + i * TPR;
        v[i] = p < rp1 ? pk.chunk[p] : -1;
        before[i] = p < rp1 && p > rp0 ? pk.chunk[p - 1] : -1;
        m[i] = p < rp1 ? pk.scale[p] : 1.0f;
      }
#pragma unroll
      for (int i = 0; i < LP; ++i) {
        const bool in = e + i * TPR < rp1, ok = v[i] > before[i] && v[i] < G_in;
        if (in && ok) atomicOr(&s_bits[r][v[i] >> 5], 1u << (v[i] & 31));
        odd |= in && !ok;
        soft |= m[i] != 1.0f;
      }
    }
    if (soft) s_soft = 1;
    if (__syncthreads_or(odd)) {
      packed_rows(X, W, pk.chunk, pk.scale, pk.rowptr, m0 + wave, m0 + rows, NW, n0, min(n0 + BN, T), d_in, d_out, G, lane, Y);
      return;
    }
    if (tid % TPR == 0) {
      // (rows past d_out: base 0, so that the offsets of their pruned chunks stay far from 2^32, where the copy's
      // instruction offset could wrap them into range)
      int at = r < rows ? rp0 - p0 : 0;
      for (int w = 0; w < words; ++w) {
        const uint32_t b = s_bits[r][w];
        s_base[r][w] = at;
        at += __popc(b);
        mark_units(w, b);
      }
    }
  } else {
    // The tile's RB mask rows are one contiguous run of RB * G_in selectors.
    // Pass 1 reads it coalesced, eight independent loads per thread at a time
    // (past the run or the layer's last mask row they read zeros), and stores
    // the kept flags as a flat bitmap, one ballot per 64 selectors, into the
    // first stages of the A tile, which the K-loop has not started to fill.
    uint32_t* flat = reinterpret_cast<uint32_t*>(&As[0][0]);
    {
      const int u0 = m0 / GO, rows = min(RB, d_out / GO - u0), n = RB * G_in;
      const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(mask + int64_t(u0) * G_in), short(0), rows * G_in * 4, 0x00020000);
      bool soft = false;
      for (int e0 = wave * 64; e0 < n; e0 += 8 * 64 * NW) {
        float m[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int e = e0 + i * 64 * NW + lane;
          m[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rm, e < n ? uint32_t(e) * 4u : kOOB, 0, 0));
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint64_t bal = __ballot(m[i] != 0.0f);
          soft |= m[i] != 0.0f && m[i] != 1.0f;
          const int e = e0 + i * 64 * NW;
          if (lane < 2 && e < n) flat[e / 32 + lane] = uint32_t(bal >> (32 * lane));
        }
      }
      __syncthreads();
      if (soft) s_soft = 1;
    }
    // Pass 2: word w of mask row r holds bits 32w .. 32w+31 of the row's G_in
    // (bits past the run are never extracted: a word stops at its row's end).
    for (int e = tid; e < RB * words; e += 64 * NW) {
      const int r = e % RB, w = e / RB;
      const int p = r * G_in + 32 * w, nb = min(32, G_in - 32 * w);
      const uint64_t two = (uint64_t(flat[p / 32 + 1]) << 32) | flat[p / 32];
      const uint32_t b = uint32_t(two >> (p & 31)) & (nb == 32 ? ~0u : (1u << nb) - 1u);
      s_bits[r][w] = b;
      mark_units(w, b);
    }
  }
  __syncthreads();
  if (wave == 0) {
    int cnt = 0;
    for (int ub = 0; ub < NU; ub += 64) {
      const int un = ub + lane;
      const bool f = un < NU && ((s_any[un >> 5] >> (un & 31)) & 1);
      const uint64_t bal = __ballot(f);
      if (f) {
        const int pos = cnt + __popcll(bal & ((uint64_t(1) << lane) - 1));
        s_cols[pos] = un;
        if constexpr (GO >= 32) {
          // square groups: all rows of a mask row share the unit's kept bits
          uint32_t live = 0;
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            uint32_t k = 0;
#pragma unroll
            for (int q = 0; q < UG; ++q) k |= s_bits[rb][(un * UG + q) >> 5] >> ((un * UG + q) & 31);
            if (k & 1u) live |= ((1u << (GO / 16)) - 1u) << (rb * (GO / 16));
          }
          s_live[pos] = live;
        }
      }
      cnt += __popcll(bal);
    }
    if (lane == 0) s_ncols = cnt;
  }
  __syncthreads();
  // this block's share of the visited units: list entries [c0, c1); of their
  // slices, this K group's: [s0, s0 + ng) (ng <= nst, the number every group runs)
  const int c0 = share * s_ncols / ksplit, c1 = (share + 1) * s_ncols / ksplit;
  const int nst = ((c1 - c0) * SUB + KS - 1) / KS;
  const int s0 = kg * nst, ng = KS == 1 ? nst : min(nst, (c1 - c0) * SUB - s0);
  const int cb = c0 < s_ncols ? c0 : 0;  // an empty share reads (never consumes) entry 0
  const int* cols = s_cols + cb;

  // This lane's DMA rows, 16 (CA wg + j) + lane / 4 of the W tile and
  // 16 (CB wg + j) + lane / 4 of the X tile, their mask rows within the tile,
  // the group of their chunk within a unit, and their byte offsets within a K
  // slice (out-of-range rows read zeros).
  int brow[CA], gsub[CA];
  uint32_t offA[CA], offB[CB];
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    int row, c;
    km_dma_target((wg * CB + j) * 64 + lane, row, c);
    offB[j] = group_voffset(uint32_t((n0 + row) * d_in + 8 * c) * 2u, j);
  }
#pragma unroll
  for (int j = 0; j < CA; ++j) {
    int row, c;
    km_dma_target((wg * CA + j) * 64 + lane, row, c);
    brow[j] = row / GO;
    gsub[j] = UG == 2 ? c >> 1 : 0;
    // packed: the chunk's byte offset within its piece (a unit of 16-wide groups holds two pieces)
    offA[j] = PACKED ? uint32_t(UG == 2 ? 8 * (c & 1) : 8 * c) * 2u
                     : group_voffset(uint32_t((m0 + row) * d_in + 8 * c) * 2u, j);
  }
  const uint32_t bytesW = PACKED ? uint32_t(np) * uint32_t(2 * G) : uint32_t(d_out) * uint32_t(d_in) * 2u;
  const uint32_t bytesX = uint32_t(T) * uint32_t(d_in) * 2u;

  // Per-slice copy state, set by prepare(): the buffer resources of the
  // slice's K range and the W offsets for its unit (chunks of pruned groups
  // get an out-of-range offset).  prepare() has no branches: the unit of the
  // next slice and the kept bits of this lane's chunks for it are read from
  // LDS one slice ahead, so their latency is hidden.
  const uint32_t ldsA = lds_addr(As) + uint32_t(kg) * (STAGES * BM * 64), ldsB = lds_addr(Bs) + uint32_t(kg) * (STAGES * BN * 64);
  auto col_of = [&](int st) { return st < ng ? (st + s0) / SUB : 0; };  // slices past the end reuse unit 0
  auto group_of = [&](int un, int j) { return un * UG + gsub[j]; };
  // packed: piece of group gr in tile row r, from the kept bits b and base of gr's word
  auto piece_of = [](uint32_t b, int base, int gr) { return base + __popc(b & ((1u << (gr & 31)) - 1u)); };
  int v_cur = __builtin_amdgcn_readfirstlane(cols[col_of(0)]);
  int v_nxt = __builtin_amdgcn_readfirstlane(cols[col_of(1)]);
  // Square groups of 32 rows and more: fragment rows of this wave that keep
  // the unit of the slice consumed next (slice st - STAGES + 1 when
  // prepare(st) runs).  With 16 x 16 groups a fragment row skips a 32-deep
  // slice only when both of its groups are pruned, and the branches cost more
  // than the skipped MFMAs save, so every row runs.
  constexpr bool SKIP = GO >= 32;
  uint32_t live_nxt = ~0u;
  uint32_t bits_cur[CA];
  int base_cur[CA];
  auto read_bits = [&](int un) {
#pragma unroll
    for (int j = 0; j < CA; ++j) {
      bits_cur[j] = s_bits[brow[j]][group_of(un, j) >> 5];
      if constexpr (PACKED) base_cur[j] = s_base[brow[j]][group_of(un, j) >> 5];
    }
  };
  read_bits(v_cur);
  uint32_t curA[CA];
  i32x4_t rA, rB;
  if constexpr (PACKED) rA = make_rsrc_grouped(W + int64_t(p0) * G, bytesW);
  auto prepare = [&](int st) {
    const bool live = st < ng;
    const uint32_t past = live ? 0u : kOOB;
    const int sub = (st + s0) % SUB;
#pragma unroll
    for (int j = 0; j < CA; ++j) {
      const int gr = group_of(v_cur, j);
      const uint32_t dead = ((~bits_cur[j] >> (gr & 31)) & 1u) << 31;
      if constexpr (PACKED)
        curA[j] = group_voffset(uint32_t(piece_of(bits_cur[j], base_cur[j], gr)) * uint32_t(2 * G) +
                                    uint32_t(sub * kBK * 2) + offA[j], j) | dead | past;
      else
        curA[j] = offA[j] | dead;
    }
    const int k0 = live ? v_cur * U + sub * kBK : 0;
    if constexpr (!PACKED) rA = make_rsrc_grouped(W + k0, live ? bytesW - 2u * uint32_t(k0) : 0u);
    rB = make_rsrc_grouped(X + k0, live ? bytesX - 2u * uint32_t(k0) : 0u);
    read_bits(v_nxt);
    v_cur = v_nxt;
    v_nxt = __builtin_amdgcn_readfirstlane(cols[col_of(st + 2)]);
    if constexpr (SKIP)
      live_nxt = (__builtin_amdgcn_readfirstlane(s_live[cb + col_of(max(st - STAGES + 1, 0))]) >> (wm * MB)) &
                 ((1u << MB) - 1u);
  };
  auto live = [&](int) { return live_nxt; };
  // copies 0..CA-1 fill this wave's row blocks of the W tile, CA..CA+CB-1 of the X tile
  auto issue = [&](int st, int p) {
    if (p < CA)
      dma16_group(p, rA, curA[p], ldsA + (st % STAGES) * (BM * 64) + wg * CA * 1024);
    else
      dma16_group(p - CA, rB, offB[p - CA], ldsB + (st % STAGES) * (BN * 64) + wg * CB * 1024);
  };
  // Soft selectors.  With every slice's copies, lane l of a wave also copies the
  // mask value of its tile row RW wg + l mod RW (RW = 16 CA rows per wave) for
  // the slice's unit (with 16-wide groups: for the group of the slice's half
  // l >> 5) into LDS; the wave's own rows are exactly those rows, so after its
  // copies land each lane scales its W chunks by values its own wave brought
  // in, with no extra wait.
  constexpr int RW = 16 * CA;
  static_assert(RW == 32 || (RW == 64 && UG == 1), "one lane per (row of the wave, group of the unit)");
  __shared__ float s_msoft[STAGES][64 * NW];
  const i32x4_t rM = make_rsrc(mask, uint32_t(d_out / GO) * uint32_t(G_in) * 4u);
  const uint32_t ldsM = lds_addr(s_msoft) + uint32_t(wave) * 256u;
  auto prepare_soft = [&](int st) {
    const int r = RW * wg + (lane & (RW - 1)), h = lane / RW;
    const bool ok = st < ng && m0 + r < d_out && (UG == 2 || h == 0);
    const int gr = v_cur * UG + (UG == 2 ? h : 0);
    dma4_buf(rM, ok ? (uint32_t((m0 + r) / GO) * uint32_t(G_in) + uint32_t(gr)) * 4u : kOOB, ldsM + uint32_t(st % STAGES) * (64u * NW * 4u));
    prepare(st);
  };
  auto rescale = [&](int st) {
    const float* ms = s_msoft[st % STAGES] + 64 * wave;
    u32x4* A = As[kg * STAGES + st % STAGES];
    float m[CA];
    u32x4 w[CA];  // read beside the selectors: one LDS round trip before the barrier, not two
    u32x4* p = A + wg * CA * 64 + lane;
#pragma unroll
    for (int j = 0; j < CA; ++j) {
      m[j] = ms[16 * j + (lane >> 2) + 32 * gsub[j]];
      w[j] = p[j * 64];
    }
#pragma unroll
    for (int j = 0; j < CA; ++j)
      if (m[j] != 0.0f && m[j] != 1.0f) p[j * 64] = scale_bf16x8(w[j], m[j]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };

  // Hard masks (the common case) run a loop without the rescaling step.
  constexpr int RA = kFwdRowsAfter < MB ? kFwdRowsAfter : MB / 2;
  f32x4 acc[MB][NB];
  u32x4(*Ag)[BM * 4] = As + kg * STAGES;
  u32x4(*Bg)[BN * 4] = Bs + kg * STAGES;
  if (PACKED && s_soft) {
    // Packed, fractional selectors: the K-loop without its interleaving (one
    // barrier per slice); each slice's products start from zero and enter the
    // sums times the rows' selectors, in fp32.  4096 x 4096 half kept, T = 128 /
    // 512: 81 / 82 us, 40 / 43 with binary selectors; computing the tile's rows one
    // wave at a time took 1850 us, one wave per row of the whole matrix 205 / 790.
    if constexpr (PACKED) {
      typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
      const i32x4_t rS = make_rsrc(pk.scale + p0, uint32_t(np) * 4u);
      auto start = [&](int st) {  // the copies of slice st and of its selectors
        const int rr = RW * wg + (lane & (RW - 1)), h = lane / RW, gr = v_cur * UG + (UG == 2 ? h : 0);
        const uint32_t b = s_bits[rr][gr >> 5];
        const bool ok = st < ng && ((b >> (gr & 31)) & 1u) && (UG == 2 || h == 0);
        dma4_buf(rS, ok ? uint32_t(piece_of(b, s_base[rr][gr >> 5], gr)) * 4u : kOOB, ldsM + uint32_t(st % STAGES) * (64u * NW * 4u));
        prepare(st);
#pragma unroll
        for (int p = 0; p < PER_STAGE; ++p) issue(st, p);
      };
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      for (int st = 0; st < (nst ? STAGES - 1 : 0); ++st) start(st);
      for (int kt = 0; kt < nst; ++kt) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this wave's reads of slice kt - 1 are done
        wait_vmcnt<(PER_STAGE + 1) * (STAGES - 2)>();        // ... and its copies of slice kt
        block_sync();
        start(kt + STAGES - 1);  // into the buffer of slice kt - 1
        u32x4 bf[NB];
        load_bfrags<NB, true, 0>(Bg[kt % STAGES], wn * NB * 16, lane, bf);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const u32x4 af = km_frag(Ag[kt % STAGES], (wm * MB + mb) * 16, lane);
          const int row = (wm * MB + mb) * 16 + 4 * (lane >> 4);  // of this lane's four results
#pragma unroll
          for (int h = 0; h < UG; ++h) {
            const f32x4 m = *reinterpret_cast<const f32x4*>(&s_msoft[kt % STAGES][(kg * NG + row / RW) * 64 + row % RW + 32 * h]);
            const u32x4 ah = UG == 1 || lane >> 5 == h ? af : zero16();
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
              acc[mb][nb] += m * __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                     __builtin_bit_cast(bf16x8_t, ah), __builtin_bit_cast(bf16x8_t, bf[nb]),
                                     f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
          }
          if constexpr (MB > 4) __builtin_amdgcn_sched_barrier(0);
        }
      }
      wait_vmcnt<0>();  // zero-fill copies of slices past the end
    }
  } else if (!PACKED && s_soft)
    gemm_mainloop<MB, NB, true, true, 0, 0, PER_STAGE, STAGES, RA, 1>(
        Ag, Bg, nst, wm * MB * 16, wn * NB * 16, lane, acc, prepare_soft, issue, rescale,
        [](int, const u32x4(&)[NB]) {}, live);
  else
    gemm_mainloop<MB, NB, true, true, 0, 0, PER_STAGE, STAGES, RA>(
        Ag, Bg, nst, wm * MB * 16, wn * NB * 16, lane, acc, prepare, issue, [](int) {},
        [](int, const u32x4(&)[NB]) {}, live);

  // Packed: a pruned group's zeros times a non-finite X make its row NaN; such a tile's rows are computed again below.
  if constexpr (PACKED)
    if (any_nan(acc)) s_nan = 1;
  if constexpr (KS == 1) {
    if (part) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const int o = m0 + wm * MB * 16 + mb * 16 + 4 * (lane >> 4);
          const int t = n0 + wn * NB * 16 + nb * 16 + (lane & 15);
          if (t < T && o < d_out) *reinterpret_cast<f32x4*>(part + (int64_t(share) * T + t) * d_out + o) = acc[mb][nb];
        }
      return;
    }
    store_tile_rows<BM, MB, NB, NW>(acc, reinterpret_cast<char*>(&As[0][0]), reinterpret_cast<char*>(&Bs[0][0]), wm,
                                    wn, tid, lane, Y, d_out, n0, T, m0, d_out);
  } else {
    if constexpr (BM == 128 && !PACKED) {
      if (part) {
        ksum2<BM, BN, MB, NB, NW, HC>(acc, reinterpret_cast<f32x4*>(smem), kg, wg, wm, wn, lane,
                                      [&](int m, int n, const f32x4& sum) {
                                        if (n0 + n < T && m0 + m < d_out)
                                          *reinterpret_cast<f32x4*>(part + (int64_t(share) * T + n0 + n) * d_out + m0 + m) = sum;
                                      });
        return;
      }
    }
    store_tile_ksum2<BM, BN, MB, NB, NW, HC>(acc, reinterpret_cast<f32x4*>(smem),
                                             reinterpret_cast<char*>(smem) + NW * HC * NB * 1024, kg, wg, wm, wn, tid,
                                             lane, Y, d_out, n0, T, m0, d_out);
  }
  if constexpr (PACKED)
    if (s_nan) {  // (visible: the stores above have barriers)
      // The arguments are read again: kept through the K-loop they cost the largest tiles registers.
      const auto* args = (const volatile __attribute__((address_space(4))) uint64_t*)(__builtin_amdgcn_kernarg_segment_ptr());
      const uint16_t* Xa = reinterpret_cast<const uint16_t*>(args[0]);
      const uint16_t* Wa = reinterpret_cast<const uint16_t*>(args[1]);
      uint16_t* Ya = reinterpret_cast<uint16_t*>(args[5]);
      const int* ca = reinterpret_cast<const int*>(args[8]);
      const int* ra = reinterpret_cast<const int*>(args[9]);
      const float* sa = reinterpret_cast<const float*>(args[10]);
      __threadfence();  // the tile's stores
      __syncthreads();
      packed_rows(Xa, Wa, ca, sa, ra, m0 + wave, min(m0 + BM, d_out), NW, n0, min(n0 + BN, T), d_in, d_out, G, lane, Ya);
    }
}

// Y = bf16(sum over shares s = 0 .. ksplit-1 of part[s]), eight outputs per thread.
__global__ __launch_bounds__(256) void fwd_reduce_kernel(const float* __restrict__ part, int ksplit, int64_t n,
                                                         uint16_t* __restrict__ Y) {
  const int64_t e = (int64_t(blockIdx.x) * 256 + threadIdx.x) * 8;
  if (e >= n) return;
  f32x4 a = *reinterpret_cast<const f32x4*>(part + e), b = *reinterpret_cast<const f32x4*>(part + e + 4);
  for (int s = 1; s < ksplit; ++s) {
    a += *reinterpret_cast<const f32x4*>(part + int64_t(s) * n + e);
    b += *reinterpret_cast<const f32x4*>(part + int64_t(s) * n + e + 4);
  }
  uint4 w;
  w.x = pack_bf16x2(a[0], a[1]);
  w.y = pack_bf16x2(a[2], a[3]);
  w.z = pack_bf16x2(b[0], b[1]);
  w.w = pack_bf16x2(b[2], b[3]);
  *reinterpret_cast<uint4*>(Y + e) = w;
}

// ============================================================================ dgate

template <int G, int GO>
__global__ __launch_bounds__(64 * kDgateWaves) void dgate_kernel(const uint16_t* __restrict__ dY, const uint16_t* __restrict__ X,
                                                    const uint16_t* __restrict__ W, int T, int d_in, int d_out,
                                                    float* __restrict__ dgate, uint16_t* __restrict__ dYt, int ldt,
                                                    ListArgs la) {
  __shared__ u32x4 smem[dgate_smem(256, 1)];
  dgate_tile<G, GO, 256, 1, true>(dY, X, W, T, d_in, d_out, dgate, dYt, ldt, la, int(blockIdx.x), smem);
}

// 256 x BN tiles, K over two wave groups.
template <int G, int GO, int BN>
__global__ __launch_bounds__(64 * kDgateWaves) void dgate_k2_kernel(const uint16_t* __restrict__ dY, const uint16_t* __restrict__ X,
                                                       const uint16_t* __restrict__ W, int T, int d_in, int d_out,
                                                       float* __restrict__ dgate, uint16_t* __restrict__ dYt, int ldt,
                                                       ListArgs la) {
  __shared__ u32x4 smem[dgate_smem(BN, 2)];
  dgate_tile<G, GO, BN, 2, true>(dY, X, W, T, d_in, d_out, dgate, dYt, ldt, la, int(blockIdx.x), smem);
}

// Fill n floats with zero (before the order-independent two-tile accumulation).
__global__ __launch_bounds__(256) void zero_f32_kernel(float* __restrict__ p, int64_t n) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0.0f;
}

// ============================================================================ dX

// C[i, t] = sum_k W[o_k, i] dYt[o_k, t] over the listed rows o_k of list
// column v (lc = max(g, 64) input columns), tile BM (i, BM = min(lc, 256)) x
// 256 (t); waves 2 (i) x WN (t).  The column list is read with scalar loads
// (KR entries per wave per slice), one slice ahead of its DMA.  With NSUB > 1
// (groups of 16 or 32 columns) a list column holds NSUB groups and lists
// every row that keeps one of them; each entry carries its kept bits, and the
// 16-byte chunks of W in a pruned group are zero-filled instead of read.
//
// KS = 2: two wave groups split the column's slices (contiguous shares, the
// last padded with zero slices) over their own rings and add their tiles in
// LDS, for launches with too few 256 x 256 tiles to fill the chip.
template <int BM, int BN, int KS, int NSUB>
__global__ __launch_bounds__(64 * dx_waves(BM, KS)) void dx_kernel(const uint16_t* __restrict__ dYt, int ldt,
                                                 const uint16_t* __restrict__ W, const int* __restrict__ colcount,
                                                 const int* __restrict__ rows, const float* __restrict__ scales,
                                                 const int* __restrict__ subbits, const int* __restrict__ colsoft,
                                                 int T, int d_in, int d_out, int lc, uint16_t* __restrict__ dX) {
  constexpr int NW = dx_waves(BM, KS), NG = NW / KS, WN = NG / 2;  // waves per block, per K group; wave grid 2 (i) x WN (t)
  constexpr int MB = BM / 32, NB = BN / WN / 16;
  constexpr int KR = kBK / NG;               // k-rows of a slice gathered by one wave
  constexpr int NA = BM / 16 / NG;           // A DMA instructions per wave per slice
  constexpr int NBC = BN / 16 / NG;          // B DMA instructions per wave per slice
  constexpr int PER_STAGE = NA + NBC;
  constexpr int STAGES = KS * (BM + BN) > 512 ? 3 : 4;
  constexpr int HC = BM == 256 ? MB / 4 : MB / 2;
  static_assert(KS == 1 || KS * STAGES * (BM + BN) * 64 >= NW * HC * NB * 1024 + 2 * BM * BN, "LDS");
  static_assert(KR * NSUB <= 64, "one lane per selector of a wave's rows");
  static_assert(KS == 1 || NSUB == 1, "one K group for list columns of several groups");
  __shared__ u32x4 smem[KS * STAGES * (BM + BN) * 4];  // the W rings, then the dY^T rings; afterwards the output tile
  // (the 64 x 256 tile's ring is half a CU's LDS: its soft selectors come from memory)
  constexpr bool MS = BM > 64 || KS > 1;
  __shared__ float s_msoft[MS ? STAGES : 1][MS ? 64 * NW : 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NG, wg = wave % NG;  // K group, wave within it
  const int wm = wg / WN, wn = wg % WN;
  u32x4(*As)[kBK * BM / 8] = reinterpret_cast<u32x4(*)[kBK * BM / 8]>(smem) + kg * STAGES;
  u32x4(*Bs)[kBK * BN / 8] = reinterpret_cast<u32x4(*)[kBK * BN / 8]>(smem + KS * STAGES * BM * 4) + kg * STAGES;
  const int tiles_m = d_in / BM, tiles_n = (T + BN - 1) / BN;
  int tm, tn;
  tile_coords(gridDim.x, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int v = m0 / lc;
  const int kv = colcount[v];
  const bool soft = colsoft[v] != 0;
  const int* __restrict__ rl = rows + int64_t(v) * d_out;
  const int* __restrict__ bl = subbits + int64_t(v) * d_out;
  const float* __restrict__ sl = scales + int64_t(v) * d_out * NSUB;
  const int all = (kv + kBK - 1) / kBK, nst = (all + KS - 1) / KS;
  const int s0 = kg * nst;            // this group's slices: [s0, s0 + nst), those from `all` on zeros
  constexpr int CPS = BM / 8 / NSUB;  // 16-byte chunks per group along i (NSUB > 1)

  // Slice st uses k-rows (s0 + st)*32 + r; this wave gathers rows r = KR wg .. KR wg + KR - 1,
  // whose list entries are read with scalar loads one slice ahead.
  int idx[KR], kbits[NSUB > 1 ? KR : 1];
  auto load_idx = [&](int st) {  // at most 31 + 32 entries past the column's end
    const int base = min(s0 + st, all) * kBK + wg * KR;
#pragma unroll
    for (int q = 0; q < KR; ++q) {
      idx[q] = rl[base + q];  // uniform: scalar loads
      if constexpr (NSUB > 1) kbits[q] = bl[base + q];
    }
  };
  // Copy j of a wave in a tile with C columns (CPR = C / 8 chunks per k-row)
  // covers k-rows KR wave + j * RPI + lane / CPR, RPI = 64 / CPR: the lane's
  // row is one of RPI consecutive list entries of the wave.
  // The entries are wave-uniform.  For chains of more than two, passing them
  // through readfirstlane keeps the compiler from turning the selects into a
  // per-lane indexed load from a stack copy of the array (for two it emits
  // one select, and the extra moves would only cost VALU issue slots).
  auto pick = [&](const auto* a, int j, auto rpi_c, int u) {
    constexpr int rpi = decltype(rpi_c)::value;
    auto entry = [&](int q) { return rpi > 2 ? __builtin_amdgcn_readfirstlane(a[j * rpi + q]) : a[j * rpi + q]; };
    auto o = entry(0);
#pragma unroll
    for (int q = 1; q < rpi; ++q) o = u == q ? entry(q) : o;
    return uint32_t(o);
  };
  constexpr std::integral_constant<int, 512 / BM> RPI_A{};
  constexpr std::integral_constant<int, 512 / BN> RPI_B{};
  const i32x4_t rA = make_rsrc_grouped(W + m0, (uint32_t(d_out) * uint32_t(d_in) - uint32_t(m0)) * 2u);
  const i32x4_t rB = make_rsrc_grouped(dYt + n0, (uint32_t(d_out) * uint32_t(ldt) - uint32_t(n0)) * 2u);
  // Offsets of this lane's chunks within their rows; the row offsets are scalar
  // (bit 31: past the list's end, and dY^T columns past the matrix: zeros).
  uint32_t colA[NA], colB[NBC], pastB[NBC];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    int row, c;
    mn_dma_target<BM>((wg * NA + j) * 64 + lane, row, c);
    colA[j] = group_voffset(uint32_t(16 * c), j);
  }
#pragma unroll
  for (int j = 0; j < NBC; ++j) {
    int row, c;
    mn_dma_target<BN>((wg * NBC + j) * 64 + lane, row, c);
    colB[j] = group_voffset(uint32_t(16 * c), j);
    pastB[j] = uint32_t(n0 + 8 * c >= ldt) << 31;
  }
  // Entries past the column's count were never written: their offsets are
  // replaced, not only flagged (a flagged offset near 2^32 would wrap into
  // range when the copy's bias is added).
  uint32_t offA[NA], offB[NBC];  // this slice's per-lane offsets
  auto prepare = [&](int st) {
    if constexpr (KS == 1) {
      const int k0 = st * kBK;
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        int row, c;
        mn_dma_target<BM>((wg * NA + j) * 64 + lane, row, c);
        bool dead = k0 + row >= kv;
        if constexpr (NSUB > 1) dead |= ((pick(kbits, j, RPI_A, lane / (BM / 8)) >> (c / CPS)) & 1) == 0;
        const uint32_t at = uint32_t(pick(idx, j, RPI_A, lane / (BM / 8)) * d_in + 8 * c) * 2u;
        offA[j] = group_voffset(dead ? kOOB : at, j);
      }
#pragma unroll
      for (int j = 0; j < NBC; ++j) {
        int row, c;
        mn_dma_target<BN>((wg * NBC + j) * 64 + lane, row, c);
        const uint32_t at = uint32_t(pick(idx, j, RPI_B, lane / (BN / 8)) * ldt + 8 * c) * 2u;
        offB[j] = group_voffset(k0 + row >= kv || n0 + 8 * c >= ldt ? kOOB : at, j);
      }
      load_idx(st + 1);
      return;
    }
    const int k0 = (s0 + st) * kBK + wg * KR;
    uint32_t rowA[KR], rowB[KR];
#pragma unroll
    for (int q = 0; q < KR; ++q) {
      rowA[q] = k0 + q < kv ? uint32_t(idx[q]) * uint32_t(d_in) * 2u : kOOB;
      rowB[q] = k0 + q < kv ? uint32_t(idx[q]) * uint32_t(ldt) * 2u : kOOB;
    }
#pragma unroll
    for (int j = 0; j < NA; ++j) offA[j] = pick(rowA, j, RPI_A, lane / (BM / 8)) + colA[j];
#pragma unroll
    for (int j = 0; j < NBC; ++j) offB[j] = (pick(rowB, j, RPI_B, lane / (BN / 8)) + colB[j]) | pastB[j];
    load_idx(st + 1);
  };
  const uint32_t ldsA = lds_addr(smem) + uint32_t(kg) * (STAGES * BM * 64);
  const uint32_t ldsB = lds_addr(smem) + uint32_t(KS * STAGES * BM * 64) + uint32_t(kg) * (STAGES * BN * 64);
  auto issue = [&](int st, int p) {  // copies 0 .. NA-1: W tile, NA .. NA+NBC-1: dY^T tile
    if (p < NA)
      dma16_group(p, rA, offA[p], ldsA + (st % STAGES) * (kBK * BM * 2) + wg * NA * 1024);
    else
      dma16_group(p - NA, rB, offB[p - NA], ldsB + (st % STAGES) * (kBK * BN * 2) + wg * NBC * 1024);
  };
  // Soft selectors: with every slice's copies the wave also copies the
  // selectors of its own KR list entries (a contiguous run of scales), and
  // scales its W chunks once both landed.
  const i32x4_t rM = make_rsrc(sl, uint32_t(kv) * uint32_t(NSUB) * 4u);
  const uint32_t ldsM = lds_addr(s_msoft) + uint32_t(wave) * 256u;
  auto prepare_soft = [&](int st) {
    const uint32_t at = (uint32_t((s0 + st) * kBK + wg * KR) * uint32_t(NSUB) + uint32_t(lane)) * 4u;
    if constexpr (MS) dma4_buf(rM, lane < KR * NSUB ? at : kOOB, ldsM + uint32_t(st % STAGES) * (64u * NW * 4u));
    prepare(st);
  };
  auto rescale = [&](int st) {
    const float* ms = s_msoft[MS ? st % STAGES : 0] + (MS ? 64 * wave : 0);
    u32x4* A = As[st % STAGES];
    constexpr int HS = NA > 2 ? 1 : NA;  // chunks scaled at once (the larger tile has fewer registers to spare)
#pragma unroll
    for (int h = 0; h < NA; h += HS) {
      float m[HS];
      u32x4 w[HS];
#pragma unroll
      for (int j = 0; j < HS; ++j) {
        int row, c;
        mn_dma_target<BM>((wg * NA + h + j) * 64 + lane, row, c);
        const int at = row * NSUB + (NSUB > 1 ? c / CPS : 0);
        m[j] = MS ? ms[at - wg * KR * NSUB] : (s0 + st) * kBK + row < kv ? sl[(s0 + st) * kBK * NSUB + at] : 1.0f;
        w[j] = A[(wg * NA + h + j) * 64 + lane];
      }
#pragma unroll
      for (int j = 0; j < HS; ++j)
        if (m[j] != 1.0f) A[(wg * NA + h + j) * 64 + lane] = scale_bf16x8(w[j], m[j]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };

  // Columns whose kept selectors are all exactly 1 run a loop without the rescaling step.
  f32x4 acc[MB][NB];
  load_idx(0);
  auto hook = [](int, const u32x4(&)[NB]) {};
  if (soft)
    gemm_mainloop<MB, NB, false, false, BM, BN, PER_STAGE, STAGES, kDxRowsAfter, MS>(
        As, Bs, nst, wm * (BM / 2), wn * NB * 16, lane, acc, prepare_soft, issue, rescale, hook);
  else
    gemm_mainloop<MB, NB, false, false, BM, BN, PER_STAGE, STAGES, kDxRowsAfter>(
        As, Bs, nst, wm * (BM / 2), wn * NB * 16, lane, acc, prepare, issue, [](int) {}, hook);

  char* const hi = reinterpret_cast<char*>(smem + STAGES * BM * 4);
  if constexpr (KS == 1)
    store_tile_rows<BM, MB, NB, NW>(acc, BM == 256 ? reinterpret_cast<char*>(smem) : hi, hi, wm, wn, tid, lane, dX,
                                    d_in, n0, T, m0, d_in);
  else
    store_tile_ksum2<BM, BN, MB, NB, NW, HC>(acc, reinterpret_cast<f32x4*>(smem),
                                             reinterpret_cast<char*>(smem) + NW * HC * NB * 1024, kg, wg, wm, wn, tid,
                                             lane, dX, d_in, n0, T, m0, d_in);
}

// ============================================================================ dY^T

// dY [T, d_out] -> dYt [d_out, ldt] (t in [T, ldt) zero).  One 8 x 8 block per thread.
__global__ __launch_bounds__(256) void transpose_kernel(const uint16_t* __restrict__ dY, int T, int d_out,
                                                        uint16_t* __restrict__ dYt, int ldt) {
  const int tchunks = ldt / 8;
  const int64_t blk = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t nblk = int64_t(tchunks) * (d_out / 8);
  if (blk >= nblk) return;
  const int a = int(blk % tchunks);  // token chunk
  const int c = int(blk / tchunks);  // output-row chunk
  u32x4 v[8], tr[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int t = 8 * a + r;
    v[r] = t < T ? ld16(dY + int64_t(t) * d_out + 8 * c) : zero16();
  }
  transpose8x8_b16(v, tr);
#pragma unroll
  for (int cc = 0; cc < 8; ++cc) st16(dYt + int64_t(8 * c + cc) * ldt + 8 * a, tr[cc]);
}

// ============================================================================ launchers

// The group shapes built: 1 x {64, 128, 256, 512} and square {16, 32, 64, 128}.
#define GM_CASE_G(KERNEL, G, GO, GRID, THREADS, ...) \
  case (G << 8) | GO: hipLaunchKernelGGL((KERNEL<G, GO>), dim3(GRID), dim3(THREADS), 0, s, __VA_ARGS__); break;
#define GM_CASE_G1(KERNEL, G, GRID, THREADS, ...) \
  case G: hipLaunchKernelGGL((KERNEL<G, 1>), dim3(GRID), dim3(THREADS), 0, s, __VA_ARGS__); break;
#define GM_CASES_G64(KERNEL, GRID, THREADS, ...)                 \
    GM_CASE_G(KERNEL, 64, 1, GRID, THREADS, __VA_ARGS__)         \
    GM_CASE_G(KERNEL, 128, 1, GRID, THREADS, __VA_ARGS__)        \
    GM_CASE_G(KERNEL, 256, 1, GRID, THREADS, __VA_ARGS__)        \
    GM_CASE_G(KERNEL, 512, 1, GRID, THREADS, __VA_ARGS__)        \
    GM_CASE_G(KERNEL, 64, 64, GRID, THREADS, __VA_ARGS__)        \
    GM_CASE_G(KERNEL, 128, 128, GRID, THREADS, __VA_ARGS__)
#define GM_LAUNCH_G(KERNEL, GRID, THREADS, ...)                  \
  switch ((g << 8) | go) {                                       \
    GM_CASES_G64(KERNEL, GRID, THREADS, __VA_ARGS__)             \
    GM_CASE_G(KERNEL, 16, 16, GRID, THREADS, __VA_ARGS__)        \
    GM_CASE_G(KERNEL, 32, 32, GRID, THREADS, __VA_ARGS__)        \
    default: return hipErrorInvalidValue;                        \
  }

template <int G, int GO>
constexpr auto fwd_big = fwd_kernel<G, GO, 256, 256, 1, false>;
template <int G, int GO>
constexpr auto fwd_half = fwd_kernel<G, GO, 256, 128, 2, false>;
template <int G, int GO>
constexpr auto fwd_mid = fwd_kernel<G, GO, 128, 128, 2, false>;

static int fwd_tiles(FwdTile tile, int T, int d_out) {
  const int bm = tile == FwdTile::k128x128 ? 128 : 256, bn = tile == FwdTile::k256x256 ? 256 : 128;
  return ((T + bn - 1) / bn) * ((d_out + bm - 1) / bm);
}

hipError_t launch_fwd(const uint16_t* X, const uint16_t* W, const float* mask, int T, int d_in, int d_out, int g,
                      int go, uint16_t* Y, FwdTile tile, int ksplit, float* part, hipStream_t s) {
  if (ksplit < 1 || (ksplit > 1 && (part == nullptr || tile == FwdTile::k256x128))) return hipErrorInvalidValue;
  const PackedArgs none{nullptr, nullptr, nullptr};
  float* p = ksplit > 1 ? part : nullptr;
  const int blocks = fwd_tiles(tile, T, d_out) * ksplit;
  if (tile == FwdTile::k128x128) {
    GM_LAUNCH_G(fwd_mid, blocks, 64 * kFwdWaves, X, W, mask, T, d_in, d_out, Y, ksplit, p, none)
  } else if (tile == FwdTile::k256x128) {
    if (g == 16) return hipErrorInvalidValue;
    switch ((g << 8) | go) {
      GM_CASES_G64(fwd_half, blocks, 64 * kFwdWaves, X, W, mask, T, d_in, d_out, Y, 1, p, none)
      GM_CASE_G(fwd_half, 32, 32, blocks, 64 * kFwdWaves, X, W, mask, T, d_in, d_out, Y, 1, p, none)
      default: return hipErrorInvalidValue;
    }
  } else {
    GM_LAUNCH_G(fwd_big, blocks, 64 * kFwdWaves, X, W, mask, T, d_in, d_out, Y, ksplit, p, none)
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || ksplit == 1) return e;
  const int64_t n = int64_t(T) * d_out;  // a multiple of 8 (d_out is)
  hipLaunchKernelGGL(fwd_reduce_kernel, dim3(unsigned((n / 8 + 255) / 256)), dim3(256), 0, s, part, ksplit, n, Y);
  return hipGetLastError();
}

// Forward from the packed export (more than 16 tokens, where packed_passes does
// not send them through the 2-16 token kernel).  The four stacked LLaMA-2-13B
// projections of a layer at T = 512, half the groups kept: 0.41 ms against
// 9.4 ms for one wave per row and 16 tokens.
hipError_t launch_fwd_packed(const uint16_t* X, const uint16_t* Wp, const int* chunk, const float* scale,
                             const int* rowptr, int T, int d_in, int d_out, int g, uint16_t* Y, FwdTile tile,
                             hipStream_t s) {
  const PackedArgs pk{chunk, rowptr, scale};
  const int blocks = fwd_tiles(tile, T, d_out);
#define GM_FWD_PACKED(G, BM, BN, KS)                                                                         \
  hipLaunchKernelGGL((fwd_kernel<G, 1, BM, BN, KS, true>), dim3(blocks), dim3(64 * kFwdWaves), 0, s, X, Wp,  \
                     nullptr, T, d_in, d_out, Y, 1, nullptr, pk)
#define GM_FWD_PACKED_G(G)                                                                                   \
  case G:                                                                                                    \
    if (tile == FwdTile::k256x256) GM_FWD_PACKED(G, 256, 256, 1);                                            \
    else if (tile == FwdTile::k256x128) GM_FWD_PACKED(G, 256, 128, 2);                                       \
    else GM_FWD_PACKED(G, 128, 128, 2);                                                                      \
    break;
  if (g < 64 && tile != FwdTile::k128x128) return hipErrorInvalidValue;
  switch (g) {
    case 16: GM_FWD_PACKED(16, 128, 128, 2); break;
    case 32: GM_FWD_PACKED(32, 128, 128, 2); break;
    GM_FWD_PACKED_G(64)
    GM_FWD_PACKED_G(128)
    GM_FWD_PACKED_G(256)
    GM_FWD_PACKED_G(512)
    default: return hipErrorInvalidValue;
  }
#undef GM_FWD_PACKED_G
#undef GM_FWD_PACKED
  return hipGetLastError();
}

template <int G, int GO>
constexpr auto dgate_half = dgate_k2_kernel<G, GO, 128>;
template <int G, int GO>
constexpr auto dgate_low = dgate_k2_kernel<G, GO, 64>;

hipError_t launch_dgate(const uint16_t* dY, const uint16_t* X, const uint16_t* W, int T, int d_in, int d_out, int g,
                        int go, float* dgate, uint16_t* dYt, int ldt, const float* mask, int nsub, int* colcount,
                        int* colsoft, int* rows, float* scales, int* subbits, hipStream_t s) {
  ListArgs la{mask, 0, (d_out + kListChunk - 1) / kListChunk, nsub, colcount, colsoft, rows, subbits, scales};
  if (colcount) la.nunits = (d_in / g / nsub) * la.nchunks;
  if (g == 512) {
    const int64_t n = int64_t(d_out) * (d_in / g);
    const unsigned blocks = unsigned(n / 256 + 1 < 4096 ? n / 256 + 1 : 4096);
    hipLaunchKernelGGL(zero_f32_kernel, dim3(blocks), dim3(256), 0, s, dgate, n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  auto tiles = [&](int bn) { return ((d_in + 255) / 256) * ((d_out + bn - 1) / bn); };
  const int columns = dgate_columns(T, d_in, d_out, go);
  if (columns == 64) {
    switch (g) {
      GM_CASE_G1(dgate_low, 64, tiles(64) + la.nunits, 64 * kDgateWaves, dY, X, W, T, d_in, d_out, dgate, dYt, ldt, la)
      GM_CASE_G1(dgate_low, 128, tiles(64) + la.nunits, 64 * kDgateWaves, dY, X, W, T, d_in, d_out, dgate, dYt, ldt, la)
      GM_CASE_G1(dgate_low, 256, tiles(64) + la.nunits, 64 * kDgateWaves, dY, X, W, T, d_in, d_out, dgate, dYt, ldt, la)
      GM_CASE_G1(dgate_low, 512, tiles(64) + la.nunits, 64 * kDgateWaves, dY, X, W, T, d_in, d_out, dgate, dYt, ldt, la)
      default: return hipErrorInvalidValue;
    }
  } else if (columns == 128) {
    GM_LAUNCH_G(dgate_half, tiles(128) + la.nunits, 64 * kDgateWaves, dY, X, W, T, d_in, d_out, dgate, dYt, ldt, la)
  } else {
    GM_LAUNCH_G(dgate_kernel, tiles(256) + la.nunits, 64 * kDgateWaves, dY, X, W, T, d_in, d_out, dgate, dYt, ldt, la)
  }
  return hipGetLastError();
}

hipError_t launch_transpose(const uint16_t* dY, int T, int d_out, uint16_t* dYt, int ldt, hipStream_t s) {
  const int64_t nblk = int64_t(ldt / 8) * (d_out / 8);
  hipLaunchKernelGGL(transpose_kernel, dim3(unsigned((nblk + 255) / 256)), dim3(256), 0, s, dY, T, d_out, dYt, ldt);
  return hipGetLastError();
}

hipError_t launch_dx(const uint16_t* dYt, int ldt, const uint16_t* W, const int* colcount, const int* rows,
                     const float* scales, const int* subbits, const int* colsoft, int T, int d_in, int d_out, int g,
                     uint16_t* dX, hipStream_t s) {
  const int lc = g < 64 ? 64 : g;  // list-column width
  auto blocks = [&](int m, int n) { return int64_t(d_in / m) * ((T + n - 1) / n); };
#define GM_DX(BM, BN, KS, NSUB)                                                                                \
  hipLaunchKernelGGL((dx_kernel<BM, BN, KS, NSUB>), dim3(unsigned(blocks(BM, BN))), dim3(64 * dx_waves(BM, KS)), 0, \
                     s, dYt, ldt, W, colcount, rows, scales, subbits, colsoft, T, d_in, d_out, lc, dX)
  if (g == 16) {
    GM_DX(64, 256, 1, 4);
    return hipGetLastError();
  }
  if (g == 32) {
    GM_DX(64, 256, 1, 2);
    return hipGetLastError();
  }
  switch (dx_tile(T, d_in, d_out, g)) {
    case DxTile::kBig: GM_DX(256, 256, 1, 1); break;
    case DxTile::kHalf: GM_DX(256, 128, 2, 1); break;
    case DxTile::kWide: GM_DX(128, 256, 1, 1); break;
    case DxTile::kMid: GM_DX(128, 128, 2, 1); break;
    case DxTile::kLow: GM_DX(64, 128, 2, 1); break;
    case DxTile::kPair: GM_DX(64, 256, 1, 1); break;
  }
#undef GM_DX
  return hipGetLastError();
}

}  // namespace gm
