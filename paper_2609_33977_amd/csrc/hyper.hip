// Hypernetwork of the mask learner (Sec. 2.2, Eq. 3) and its AdamW step (Table 5).
//
//   o_l      = [GRU_fwd(z_1..z_l); GRU_bwd(z_L..z_l)]        (bidirectional GRU, H units per direction)
//   logit[e] = A[e] . o_{l(e)} + c[e]                       (layer-specific affine heads, rows of one
//                                                            [sum G, 2H] matrix in flat selector order)
//
// The GRU is tiny and sequential over the L layers; the heads hold one row of
// 2H weights per selector (25.3 M rows for LLaMA-2-7B) and are the HBM-bound
// part: the forward reads A once, and the backward reads A with its two AdamW
// moments and writes all three back in one pass, which also accumulates
// do_l = A^T dlogit (with the weights before the update) for the GRU backward.
//
// Work split:
//   gru_input_kernel   W_ih z_l + b_ih for every layer and direction (parallel), and the chunk table: every layer's
//                      rows cut into chunks of kHeadRows, so that a head block never straddles two layers
//   gru_fwd_kernel<H>  one block per direction, the recurrence; caches the gates
//   head_fwd_kernel    logits, one wave row group per selector row
//   head_bwd_kernel    AdamW on A and c, chunk partials of do
//   head_do_kernel     do_l = sum of its chunks' partials, in chunk order
//   gru_bwd_kernel<H>  one block per direction, backpropagation through time
//   gru_wgrad_kernel   weight and bias gradients from the per-step gate gradients
//   adamw_kernel       AdamW over a flat parameter vector (the GRU's)
// Every reduction runs in a fixed order, so results are deterministic.
#include "gm_device.h"
#include "gm_launch.h"

#include <math.h>

namespace gm {

constexpr int kHeadRows = 2048;  // selector rows per head block

__device__ __forceinline__ float sigmoidf(float x) { return 1.0f / (1.0f + expf(-x)); }

// ---------------------------------------------------------------- GRU forward

// Chunk c covers rows [start, end) of layer lay; layers are cut at multiples
// of kHeadRows from their first row.  count[0] = number of chunks, first[l] =
// first chunk of layer l (first[L] = count).
__device__ __forceinline__ void chunk_table(const int64_t* __restrict__ offsets, int L, int* __restrict__ lay,
                                            int64_t* __restrict__ start, int64_t* __restrict__ end,
                                            int* __restrict__ first, int* __restrict__ count) {
  __shared__ int s_n[256];
  const int tid = threadIdx.x;
  // per-thread totals over a contiguous run of layers, then a block scan
  const int per = (L + 255) / 256;
  const int l0 = min(tid * per, L), l1 = min(l0 + per, L);
  int n = 0;
  for (int l = l0; l < l1; ++l) n += int((offsets[l + 1] - offsets[l] + kHeadRows - 1) / kHeadRows);
  s_n[tid] = n;
  __syncthreads();
  for (int d = 1; d < 256; d <<= 1) {
    const int add = tid >= d ? s_n[tid - d] : 0;
    __syncthreads();
    s_n[tid] += add;
    __syncthreads();
  }
  int c = s_n[tid] - n;
  for (int l = l0; l < l1; ++l) {
    first[l] = c;
    for (int64_t r = offsets[l]; r < offsets[l + 1]; r += kHeadRows, ++c) {
      lay[c] = l;
      start[c] = r;
      end[c] = min(r + int64_t(kHeadRows), offsets[l + 1]);
    }
  }
  if (tid == 255) {
    first[L] = s_n[255];
    count[0] = s_n[255];
  }
}

// gi[dir][l][i] = b_ih[i] + W_ih[i, :] . z[l]; the last block cuts the heads
// into chunks meanwhile (a launch of its own took 6 us).  Eight columns of the
// dot product are loaded at a time (one at a time: 17 us at L = 224, D = 64).
__global__ __launch_bounds__(256) void gru_input_kernel(const float* __restrict__ z, const float* __restrict__ gru,
                                                       int L, int D, int H, float* __restrict__ gi,
                                                       const int64_t* __restrict__ offsets, int* __restrict__ lay,
                                                       int64_t* __restrict__ start, int64_t* __restrict__ end,
                                                       int* __restrict__ first, int* __restrict__ count) {
  if (blockIdx.x == gridDim.x - 1) {
    chunk_table(offsets, L, lay, start, end, first, count);
    return;
  }
  const int G3 = 3 * H;
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (e >= int64_t(2) * L * G3) return;
  const int i = int(e % G3);
  const int l = int((e / G3) % L);
  const int dir = int(e / (int64_t(L) * G3));
  const float* p = gru + int64_t(dir) * G3 * (D + H + 2);
  const float* w = p + int64_t(i) * D;
  const float* x = z + int64_t(l) * D;
  float a = p[int64_t(G3) * (D + H) + i];
  int j = 0;
  for (; j + 8 <= D; j += 8) {
    float wv[8], xv[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) wv[q] = w[j + q], xv[q] = x[j + q];
#pragma unroll
    for (int q = 0; q < 8; ++q) a += wv[q] * xv[q];
  }
  for (; j < D; ++j) a += w[j] * x[j];
  gi[e] = a;
}

// Sum over the S adjacent lanes of a unit (S = 4 or 8), left in all of them:
// lane exchanges inside the row by DPP (quad permutations, then the mirrored
// half row, whose quad already holds one value), without an LDS round trip.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}

template <int S>
__device__ __forceinline__ float unit_sum(float x) {
  static_assert(S == 4 || S == 8, "lanes per unit");
  x = dpp_add<0xb1>(x);                       // quad_perm [1, 0, 3, 2]
  x = dpp_add<0x4e>(x);                       // quad_perm [2, 3, 0, 1]
  return S == 8 ? dpp_add<0x141>(x) : x;      // row_half_mirror
}

// Barrier for LDS only: the recurrences' global loads (one step ahead) and
// stores stay in flight across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Lanes per hidden unit in the recurrences: with four waves or more, one per SIMD.
template <int H>
constexpr int kUnitLanes = H == 32 ? 8 : 4;

// One block per direction, latency-bound: S lanes per hidden unit hold a
// segment of the unit's three W_hh rows in registers, so that a step is one
// LDS read of the hidden state, 3 H/S multiply-adds, log2(S) lane exchanges,
// the gates (every lane of the unit computes them, no exchange) and one
// barrier: 162 -> 120 us at L = 224, H = 64 against one thread per gate row
// with two barriers per step.  cache[dir][l] = (h_prev, r, u, n, W_hn h_prev +
// b_hn), each H.  The hidden state is double-buffered in LDS.
template <int H>
__global__ __launch_bounds__(kUnitLanes<H>* H) void gru_fwd_kernel(const float* __restrict__ gi,
                                                                   const float* __restrict__ gru, int L, int D,
                                                                   float* __restrict__ o, float* __restrict__ cache) {
  constexpr int G3 = 3 * H, S = kUnitLanes<H>, KS = H / S;
  __shared__ float s_h[2][H];
  const int dir = blockIdx.x, i = threadIdx.x / S, seg = threadIdx.x % S;
  const float* p = gru + int64_t(dir) * G3 * (D + H + 2);
  const float* Whh = p + int64_t(G3) * D;
  float w[3][KS], bh[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    bh[q] = p[int64_t(G3) * (D + H) + G3 + q * H + i];
#pragma unroll
    for (int k = 0; k < KS; ++k) w[q][k] = Whh[(q * H + i) * H + seg * KS + k];
  }
  auto gates_in = [&](int s, float (&x)[3]) {  // input part of step s's gates for unit i
    const int l = dir == 0 ? s : L - 1 - s;
    const float* g = gi + (int64_t(dir) * L + l) * G3;
#pragma unroll
    for (int q = 0; q < 3; ++q) x[q] = g[q * H + i];
  };
  // the gates' input parts of PF steps, loaded PF steps ahead (one step of
  // computing is shorter than a load)
  constexpr int PF = 4;
  float xg[PF][3], xn[PF][3];
  auto load_steps = [&](int s, float (&x)[PF][3]) {
#pragma unroll
    for (int j = 0; j < PF; ++j) gates_in(min(s + j, L - 1), x[j]);
  };
  load_steps(0, xg);
  float h = 0.0f;  // this unit's state
  if (seg == 0) s_h[0][i] = 0.0f;
  __syncthreads();
  auto step = [&](int s, const float (&x)[3]) {
    const int l = dir == 0 ? s : L - 1 - s;
    float hv[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) hv[k] = s_h[s & 1][seg * KS + k];
    float a[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int q = 0; q < 3; ++q) a[q] += w[q][k] * hv[k];
#pragma unroll
    for (int q = 0; q < 3; ++q) a[q] = unit_sum<S>(a[q]) + bh[q];
    const float r = sigmoidf(x[0] + a[0]);
    const float u = sigmoidf(x[1] + a[1]);
    const float n = tanhf(x[2] + r * a[2]);
    const float hn = (1.0f - u) * n + u * h;
    if (seg == 0) s_h[(s + 1) & 1][i] = hn;  // the other buffer: its readers are past the last barrier
    // the five cached values and o, one or two per lane
    float* c = cache + (int64_t(dir) * L + l) * 5 * H + i;
    const float v = seg == 0 ? h : seg == 1 ? r : seg == 2 ? u : n;
    if (seg < 4) c[seg * H] = v;
    if (seg == 0) c[4 * H] = a[2];
    if (seg == 1) o[int64_t(l) * 2 * H + dir * H + i] = hn;
    h = hn;
    lds_barrier();
  };
  for (int s = 0; s < L; s += PF) {
    load_steps(s + PF, xn);
#pragma unroll
    for (int j = 0; j < PF; ++j)
      if (s + j < L) step(s + j, xg[j]);  // uniform
#pragma unroll
    for (int j = 0; j < PF; ++j)
#pragma unroll
      for (int q = 0; q < 3; ++q) xg[j][q] = xn[j][q];
  }
}

// ---------------------------------------------------------------- heads

// LPR = 2H / 4 lanes per row (four weights per lane), RPW = 64 / LPR rows per wave step.
template <int H>
__global__ __launch_bounds__(256) void head_fwd_kernel(const float* __restrict__ A, const float* __restrict__ cb,
                                                       const float* __restrict__ o, const int* __restrict__ lay,
                                                       const int64_t* __restrict__ start,
                                                       const int64_t* __restrict__ end,
                                                       const int* __restrict__ count, float* __restrict__ logits) {
  constexpr int LPR = 2 * H / 4, RPW = 64 / LPR;
  if (int(blockIdx.x) >= count[0]) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l = lay[blockIdx.x];
  const int64_t r0 = start[blockIdx.x], r1 = end[blockIdx.x];
  const int col = (lane % LPR) * 4;
  const f32x4 ov = *reinterpret_cast<const f32x4*>(o + int64_t(l) * 2 * H + col);
  // Eight row steps at a time, so that their loads are in flight together, and
  // nontemporal (the heads stream through once): 824 -> 600 us for the 3.2 GB of
  // 6.3 M rows of 128 weights (5.4 TB/s; four steps 630, cached loads 680).
  constexpr int HU = 8, STEP = 4 * RPW;
  for (int64_t rb = r0 + wave * RPW + lane / LPR; rb - (lane / LPR) < r1; rb += HU * STEP) {
    f32x4 w[HU];
    float a[HU];
#pragma unroll
    for (int q = 0; q < HU; ++q) {
      const int64_t r = rb + q * STEP;
      w[q] = r < r1 ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(A + r * 2 * H + col)) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int q = 0; q < HU; ++q) {
      a[q] = w[q][0] * ov[0] + w[q][1] * ov[1] + w[q][2] * ov[2] + w[q][3] * ov[3];
#pragma unroll
      for (int x = 1; x < LPR; x <<= 1) a[q] += __shfl_xor(a[q], x);
    }
#pragma unroll
    for (int q = 0; q < HU; ++q) {
      const int64_t r = rb + q * STEP;
      if (r < r1 && lane % LPR == 0) logits[r] = a[q] + cb[r];
    }
  }
}

// One AdamW step on a float4 of parameters (decoupled decay, bias-corrected moments).
// The coefficients are formed in fp64 on the host and rounded once (1 - beta
// directly, not from a rounded beta).
struct AdamW {
  float lr, b1, omb1, b2, omb2, eps, decay, bc1, bc2;  // decay = 1 - lr weight_decay; bc = 1 / (1 - beta^t)
  __device__ __forceinline__ float step(float p, float g, float& m, float& v) const {
    m = b1 * m + omb1 * g;
    v = b2 * v + omb2 * g * g;
    return p * decay - lr * (m * bc1) / (sqrtf(v * bc2) + eps);
  }
};

template <int H>
__global__ __launch_bounds__(256) void head_bwd_kernel(const float* __restrict__ dl, float* __restrict__ A,
                                                       float* __restrict__ cb, float* __restrict__ mA,
                                                       float* __restrict__ vA, float* __restrict__ mc,
                                                       float* __restrict__ vc, const float* __restrict__ o,
                                                       const int* __restrict__ lay, const int64_t* __restrict__ start,
                                                       const int64_t* __restrict__ end, const int* __restrict__ count,
                                                       AdamW opt, float* __restrict__ part) {
  constexpr int LPR = 2 * H / 4, RPW = 64 / LPR;
  __shared__ f32x4 s_do[4][64];
  if (int(blockIdx.x) >= count[0]) return;  // uniform across the block
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l = lay[blockIdx.x];
  const int64_t r0 = start[blockIdx.x], r1 = end[blockIdx.x];
  const int col = (lane % LPR) * 4;
  const f32x4 ov = *reinterpret_cast<const f32x4*>(o + int64_t(l) * 2 * H + col);
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  // Weights and moments are read and written once: nontemporal both ways, 4.07
  // -> 3.92 ms for 6.3 M rows of 128 weights (5.0 TB/s, a plain copy's rate;
  // two rows in flight per lane: level).
  for (int64_t r = r0 + wave * RPW + lane / LPR; r < r1; r += 4 * RPW) {
    const float g = dl[r];
    const int64_t at = r * 2 * H + col;
    f32x4 w = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(A + at));
    f32x4 m = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(mA + at));
    f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(vA + at));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      acc[k] += w[k] * g;
      float mk = m[k], vk = v[k];
      w[k] = opt.step(w[k], g * ov[k], mk, vk);
      m[k] = mk;
      v[k] = vk;
    }
    __builtin_nontemporal_store(w, reinterpret_cast<f32x4*>(A + at));
    __builtin_nontemporal_store(m, reinterpret_cast<f32x4*>(mA + at));
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(vA + at));
    if (lane % LPR == 0) {
      float cm = mc[r], cv = vc[r];
      cb[r] = opt.step(cb[r], g, cm, cv);
      mc[r] = cm;
      vc[r] = cv;
    }
  }
  // do partial of this chunk: over the RPW row slots of the wave, then the four waves
#pragma unroll
  for (int x = LPR; x < 64; x <<= 1)
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] += __shfl_xor(acc[k], x);
  s_do[wave][lane] = acc;
  __syncthreads();
  if (threadIdx.x < LPR) {
    const f32x4 s = s_do[0][threadIdx.x] + s_do[1][threadIdx.x] + s_do[2][threadIdx.x] + s_do[3][threadIdx.x];
    *reinterpret_cast<f32x4*>(part + int64_t(blockIdx.x) * 2 * H + threadIdx.x * 4) = s;
  }
}

// do[l][k] = sum over the chunks of layer l, in chunk order.
__global__ __launch_bounds__(256) void head_do_kernel(const float* __restrict__ part, const int* __restrict__ first,
                                                     int L, int H2, float* __restrict__ dout) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= L * H2) return;
  const int l = e / H2, k = e % H2;
  float s = 0.0f;
  const int c1 = first[l + 1];
#pragma unroll 8
  for (int c = first[l]; c < c1; ++c) s += part[int64_t(c) * H2 + k];
  dout[e] = s;
}

// ---------------------------------------------------------------- GRU backward

// One block per direction, latency-bound like the forward: S lanes per hidden
// unit k, each with a segment of column k of W_hh.  Every lane forms the gate
// gradients of its unit from dh = do + carried gradient, the unit's first
// lanes publish them in LDS (double-buffered: one barrier per step), and the
// segments' products with W_hh, summed over the unit's lanes, carry to the
// previous step: 206 -> 97 us at L = 224, H = 64 against two barriers per
// step.  dgi,
// dgh [dir][l][3H] are kept for the weight gradients.
template <int H>
__global__ __launch_bounds__(kUnitLanes<H>* H) void gru_bwd_kernel(const float* __restrict__ dout,
                                                                   const float* __restrict__ gru,
                                                                   const float* __restrict__ cache, int L, int D,
                                                                   float* __restrict__ dgi, float* __restrict__ dgh) {
  constexpr int G3 = 3 * H, S = kUnitLanes<H>, RPT = G3 / S;
  __shared__ float s_g[2][G3];
  const int dir = blockIdx.x, k = threadIdx.x / S, seg = threadIdx.x % S;
  const float* Whh = gru + int64_t(dir) * G3 * (D + H + 2) + int64_t(G3) * D;
  float wc[RPT];  // W_hh[seg * RPT + j, k]
#pragma unroll
  for (int j = 0; j < RPT; ++j) wc[j] = Whh[(seg * RPT + j) * H + k];
  // this unit's cached gates and output gradient of PF steps, loaded PF steps ahead
  constexpr int PF = 4;
  auto fetch = [&](int s, float (&v)[PF][6]) {
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      const int t = max(s - j, 0), l = dir == 0 ? t : L - 1 - t;
      const float* c = cache + (int64_t(dir) * L + l) * 5 * H;
#pragma unroll
      for (int q = 0; q < 5; ++q) v[j][q] = c[q * H + k];
      v[j][5] = dout[int64_t(l) * 2 * H + dir * H + k];
    }
  };
  float cur[PF][6], nxt[PF][6];
  fetch(L - 1, cur);
  float carry = 0.0f;
  auto step = [&](int s, const float (&v)[6]) {
    const int l = dir == 0 ? s : L - 1 - s;
    const float hp = v[0], r = v[1], u = v[2], n = v[3], ghn = v[4];
    const float dh = carry + v[5];
    const float dan = dh * (1.0f - u) * (1.0f - n * n);
    const float dar = dan * ghn * r * (1.0f - r);
    const float dau = dh * (hp - n) * u * (1.0f - u);
    float* g = s_g[s & 1];
    const int64_t at = (int64_t(dir) * L + l) * G3 + k;
    if (seg < 3) {
      const float gh = seg == 0 ? dar : seg == 1 ? dau : dan * r;
      g[seg * H + k] = gh;
      dgh[at + seg * H] = gh;
      dgi[at + seg * H] = seg == 2 ? dan : gh;
    }
    lds_barrier();
    float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
#pragma unroll
    for (int j = 0; j < RPT; j += 4) {
      a0 += wc[j] * g[seg * RPT + j];
      a1 += wc[j + 1] * g[seg * RPT + j + 1];
      a2 += wc[j + 2] * g[seg * RPT + j + 2];
      a3 += wc[j + 3] * g[seg * RPT + j + 3];
    }
    carry = dh * u + unit_sum<S>((a0 + a1) + (a2 + a3));
  };
  for (int s = L - 1; s >= 0; s -= PF) {
    fetch(s - PF, nxt);
#pragma unroll
    for (int j = 0; j < PF; ++j)
      if (s - j >= 0) step(s - j, cur[j]);  // uniform
#pragma unroll
    for (int j = 0; j < PF; ++j)
#pragma unroll
      for (int q = 0; q < 6; ++q) cur[j][q] = nxt[j][q];
  }
}

// Weight and bias gradients of one direction, one thread per parameter, sums over l in order:
//   dW_ih[i, j] = sum_l dgi[l][i] z[l][j],  dW_hh[i, k] = sum_l dgh[l][i] h_prev[l][k],
//   db_ih[i] = sum_l dgi[l][i],             db_hh[i] = sum_l dgh[l][i].
__global__ __launch_bounds__(256) void gru_wgrad_kernel(const float* __restrict__ z, const float* __restrict__ cache,
                                                       const float* __restrict__ dgi, const float* __restrict__ dgh,
                                                       int L, int D, int H, float* __restrict__ dgru) {
  const int G3 = 3 * H;
  const int64_t P = int64_t(G3) * (D + H + 2);
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (e >= 2 * P) return;
  const int dir = int(e / P);
  const int64_t q = e % P;
  const float* gi = dgi + int64_t(dir) * L * G3;
  const float* gh = dgh + int64_t(dir) * L * G3;
  const float* hc = cache + int64_t(dir) * L * 5 * H;  // h_prev is the first of the five
  float s = 0.0f;
  if (q < int64_t(G3) * D) {
    const int i = int(q / D), j = int(q % D);
#pragma unroll 16
    for (int l = 0; l < L; ++l) s += gi[int64_t(l) * G3 + i] * z[int64_t(l) * D + j];
  } else if (q < int64_t(G3) * (D + H)) {
    const int64_t t = q - int64_t(G3) * D;
    const int i = int(t / H), k = int(t % H);
#pragma unroll 16
    for (int l = 0; l < L; ++l) s += gh[int64_t(l) * G3 + i] * hc[int64_t(l) * 5 * H + k];
  } else if (q < int64_t(G3) * (D + H + 1)) {
    const int i = int(q - int64_t(G3) * (D + H));
#pragma unroll 16
    for (int l = 0; l < L; ++l) s += gi[int64_t(l) * G3 + i];
  } else {
    const int i = int(q - int64_t(G3) * (D + H + 1));
#pragma unroll 16
    for (int l = 0; l < L; ++l) s += gh[int64_t(l) * G3 + i];
  }
  dgru[e] = s;
}

__global__ __launch_bounds__(256) void adamw_kernel(float* __restrict__ p, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, int64_t n,
                                                   AdamW opt) {
  const int64_t stride = int64_t(gridDim.x) * 256;
  for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < n; e += stride) {
    float mm = m[e], vv = v[e];
    p[e] = opt.step(p[e], g[e], mm, vv);
    m[e] = mm;
    v[e] = vv;
  }
}

// ---------------------------------------------------------------- launchers

int hyper_max_chunks(int64_t G_total, int L) { return int((G_total + kHeadRows - 1) / kHeadRows) + L; }

static AdamW make_adamw(double lr, double b1, double b2, double eps, double wd, int step) {
  AdamW o;
  o.lr = float(lr);
  o.b1 = float(b1);
  o.omb1 = float(1.0 - b1);
  o.b2 = float(b2);
  o.omb2 = float(1.0 - b2);
  o.eps = float(eps);
  o.decay = float(1.0 - lr * wd);
  o.bc1 = float(1.0 / (1.0 - pow(b1, double(step))));
  o.bc2 = float(1.0 / (1.0 - pow(b2, double(step))));
  return o;
}

// One block per direction, kUnitLanes lanes per hidden unit.
#define GM_HYPER_CASE(KERNEL, HV, ...) \
  case HV: hipLaunchKernelGGL((KERNEL<HV>), dim3(2), dim3(kUnitLanes<HV> * HV), 0, s, __VA_ARGS__); break;
#define GM_HYPER_H(KERNEL, ...)             \
  switch (H) {                              \
    GM_HYPER_CASE(KERNEL, 32, __VA_ARGS__)  \
    GM_HYPER_CASE(KERNEL, 64, __VA_ARGS__)  \
    GM_HYPER_CASE(KERNEL, 128, __VA_ARGS__) \
    default: return hipErrorInvalidValue;   \
  }

hipError_t launch_hyper_fwd(const float* z, const float* gru, const float* A, const float* c, const int64_t* offsets,
                            int L, int D, int H, int64_t G_total, float* logits, const HyperWs& w, hipStream_t s) {
  const int64_t n_in = int64_t(2) * L * 3 * H;
  hipLaunchKernelGGL(gru_input_kernel, dim3(unsigned((n_in + 255) / 256) + 1), dim3(256), 0, s, z, gru, L, D, H, w.gi,
                     offsets, w.lay, w.start, w.end, w.first, w.count);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  GM_HYPER_H(gru_fwd_kernel, w.gi, gru, L, D, w.o, w.cache)
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const unsigned blocks = unsigned(hyper_max_chunks(G_total, L));
  switch (H) {
    case 32: hipLaunchKernelGGL(head_fwd_kernel<32>, dim3(blocks), dim3(256), 0, s, A, c, w.o, w.lay, w.start, w.end, w.count, logits); break;
    case 64: hipLaunchKernelGGL(head_fwd_kernel<64>, dim3(blocks), dim3(256), 0, s, A, c, w.o, w.lay, w.start, w.end, w.count, logits); break;
    case 128: hipLaunchKernelGGL(head_fwd_kernel<128>, dim3(blocks), dim3(256), 0, s, A, c, w.o, w.lay, w.start, w.end, w.count, logits); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_hyper_bwd(const float* dlogits, const float* z, const float* gru, float* A, float* c, float* mA,
                            float* vA, float* mc, float* vc, int L, int D, int H, int64_t G_total, double lr,
                            double beta1, double beta2, double eps, double weight_decay, int step, float* dgru,
                            const HyperWs& w, hipStream_t s) {
  const AdamW opt = make_adamw(lr, beta1, beta2, eps, weight_decay, step);
  const unsigned blocks = unsigned(hyper_max_chunks(G_total, L));
  switch (H) {
    case 32: hipLaunchKernelGGL(head_bwd_kernel<32>, dim3(blocks), dim3(256), 0, s, dlogits, A, c, mA, vA, mc, vc, w.o, w.lay, w.start, w.end, w.count, opt, w.part); break;
    case 64: hipLaunchKernelGGL(head_bwd_kernel<64>, dim3(blocks), dim3(256), 0, s, dlogits, A, c, mA, vA, mc, vc, w.o, w.lay, w.start, w.end, w.count, opt, w.part); break;
    case 128: hipLaunchKernelGGL(head_bwd_kernel<128>, dim3(blocks), dim3(256), 0, s, dlogits, A, c, mA, vA, mc, vc, w.o, w.lay, w.start, w.end, w.count, opt, w.part); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(head_do_kernel, dim3(unsigned((L * 2 * H + 255) / 256)), dim3(256), 0, s, w.part, w.first, L,
                     2 * H, w.dout);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  GM_HYPER_H(gru_bwd_kernel, w.dout, gru, w.cache, L, D, w.dgi, w.dgh)
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int64_t P2 = int64_t(2) * 3 * H * (D + H + 2);
  hipLaunchKernelGGL(gru_wgrad_kernel, dim3(unsigned((P2 + 255) / 256)), dim3(256), 0, s, z, w.cache, w.dgi, w.dgh,
                     L, D, H, dgru);
  return hipGetLastError();
}

hipError_t launch_adamw(float* p, const float* g, float* m, float* v, int64_t n, double lr, double beta1,
                        double beta2, double eps, double weight_decay, int step, hipStream_t s) {
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(adamw_kernel, dim3(unsigned(blocks < 8192 ? blocks : 8192)), dim3(256), 0, s, p, g, m, v, n,
                     make_adamw(lr, beta1, beta2, eps, weight_decay, step));
  return hipGetLastError();
}

}  // namespace gm
