// Host-side launchers of the gfx950 kernels (internal to the library).
// Every launcher enqueues on stream s and returns the launch status; argument
// validation happens in the C-ABI layer before any of these is called.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gm {

hipError_t launch_gate_fwd(const float* logits, const float* noise, int64_t n, float tau, int hard, float* mask,
                           float* soft, hipStream_t s);
hipError_t launch_gate_bwd(const float* dmask, const float* soft, int64_t n, float tau, float* dlogits,
                           hipStream_t s);

hipError_t launch_budget_loss(const float* mask, int64_t n, const int64_t* offsets, const int64_t* params, int L,
                              float s_target, float lambda, int uniform, unsigned long long* kept, double* loss,
                              float* coeff, hipStream_t s);
hipError_t launch_gate_bwd_budget(const float* dgate, const float* soft, int64_t n, float tau,
                                  const int64_t* offsets, int L, const float* coeff, float* dlogits, hipStream_t s);

// Group shapes: g_out x g (go = g_out; 1 for row groups).
hipError_t launch_col_lists(const float* mask, int d_out, int G_in, int go, int nsub, int* colcount, int* colsoft,
                            int* rows, float* scales, int* subbits, hipStream_t s);
hipError_t launch_pack_rows(const uint16_t* W, const float* mask, int d_in, int d_out, int g, int go,
                            int64_t capacity, uint16_t* Wp, int* chunk, float* scale, int* rowptr, hipStream_t s);

hipError_t launch_gemv_inplace(const uint16_t* X, const uint16_t* W, const float* mask, int T, int d_in, int d_out,
                               int g, int go, uint16_t* Y, hipStream_t s);
hipError_t launch_gemv_packed(const uint16_t* X, const uint16_t* Wp, const int* chunk, const float* scale,
                              const int* rowptr, int T, int d_in, int d_out, int g, uint16_t* Y, hipStream_t s);
int gemv_max_groups_per_row();

// Estimated time of a GEMM launch whose blocks (one per CU) take block_ns each:
// whole rounds of 256 blocks, and a last round that is partly empty at half a
// round plus half its fill (its blocks run faster alone); less than one round
// costs a whole one.
inline int64_t rounds_ns(int64_t blocks, int64_t block_ns) {
  const int64_t full = blocks / 256, rest = blocks % 256;
  if (full == 0) return block_ns;
  return full * block_ns + (rest ? block_ns / 2 + block_ns * rest / 512 : 0);
}

// 17 tokens and more of the packed export in passes of 16 through the decode
// kernel: rows per block (0: the block's tables of selectors do not fit).
constexpr int kMmaMaskFloats = 8192;  // staged mask floats per block: mask rows of the block x selectors per row
inline int passes_rows(int64_t T, int64_t d_in, int64_t d_out, int32_t g) {
  const int64_t G_in = d_in / g, passes = (T + 15) / 16;
  if (16 * G_in > kMmaMaskFloats) return 0;
  // 32 rows where they fill the CUs and leave room for a second block on each
  return (32 * G_in <= 4096 || 16 * G_in > 4096) && 32 * G_in <= kMmaMaskFloats && (d_out + 31) / 32 * passes >= 256 ? 32 : 16;
}

// Whether they do, against gemm_ns for the GEMM (half more with 16-wide groups).
// A block takes 7 us, 0.09 us per 32 columns and 0.025 us per group of a row;
// blocks beyond 256 share the CUs (0.042 and 0.016 us per 256 blocks of 32 rows).
// The GEMM is kept unless 15 % slower by this estimate, since its time depends
// less on the density.  5120 x 5120, T = 17 /
// 64 / 128, half the groups kept, us in passes and in the GEMM: 23, 49 / 32, 49
// / 48, 50; 15360 x 5120: 39, 49 / 67, 50 / 117, 55; 1024 x 4096: 14, 44 / 14, 44 /
// 19, 46; 10 % kept, 5120 x 5120: 22, 48 / 31, 49 / 45, 49.  Rows of too many groups
// for the tables (16-wide, above 512) take one wave per row and pass: 2048 x
// 16384, T = 33 / 65 151, 226 / 290, 225.
inline bool packed_passes(int64_t T, int64_t d_in, int64_t d_out, int32_t g, int64_t gemm_ns) {
  const int64_t rows = passes_rows(T, d_in, d_out, g), slices = d_in / 32, G_in = d_in / g;
  if (rows == 0) return T <= 48;
  const int64_t blocks = (d_out + rows - 1) / rows * ((T + 15) / 16);
  const int64_t more = blocks > 256 ? (blocks - 256) * (42 * slices + 16 * G_in) * rows / (32 * 256) : 0;
  return (7000 + 90 * slices + 25 * G_in + more) * 115 < gemm_ns * (g == 16 ? 150 : 100);
}

// Output tiles of the forward GEMM, rows of Y's columns (o) x tokens; the two
// 128-token tiles split K over two wave groups inside the block.
enum class FwdTile { k256x256, k256x128, k128x128 };

// Selectors per row that the 256-row tiles have LDS for beside their rings (1 x g groups; the in-place 256 x 256
// tile and the 128 x 128 tiles hold every row the library accepts).
constexpr int fwd_max_groups(int g, bool packed, bool half) {
  return packed && half && 16384 / g > 128 ? 128 : 16384 / g;
}

// ksplit > 1 (256 x 256 and 128 x 128 tiles) splits each tile's K range over that many blocks, which store fp32
// partial tiles into part [ksplit][T][d_out]; a second kernel adds them in order.
hipError_t launch_fwd(const uint16_t* X, const uint16_t* W, const float* mask, int T, int d_in, int d_out, int g,
                      int go, uint16_t* Y, FwdTile tile, int ksplit, float* part, hipStream_t s);
hipError_t launch_fwd_packed(const uint16_t* X, const uint16_t* Wp, const int* chunk, const float* scale,
                             const int* rowptr, int T, int d_in, int d_out, int g, uint16_t* Y, FwdTile tile,
                             hipStream_t s);
// With colcount set, the launch also builds the column lists (as launch_col_lists).
hipError_t launch_dgate(const uint16_t* dY, const uint16_t* X, const uint16_t* W, int T, int d_in, int d_out, int g,
                        int go, float* dgate, uint16_t* dYt, int ldt, const float* mask, int nsub, int* colcount,
                        int* colsoft, int* rows, float* scales, int* subbits, hipStream_t s);
hipError_t launch_transpose(const uint16_t* dY, int T, int d_out, uint16_t* dYt, int ldt, hipStream_t s);
hipError_t launch_dx(const uint16_t* dYt, int ldt, const uint16_t* W, const int* colcount, const int* rows,
                     const float* scales, const int* subbits, const int* colsoft, int T, int d_in, int d_out, int g,
                     uint16_t* dX, hipStream_t s);

// dX of 16 x 16 and 32 x 32 groups straight from dY and W (no column lists, no dY^T).
bool dx_dense_ok(int d_out, int g);
hipError_t launch_dx_dense(const uint16_t* dY, const uint16_t* W, const float* mask, int T, int d_in, int d_out, int g,
                           uint16_t* dX, hipStream_t s);

// Distillation loss (Sec. 2.4, Eq. 4) through the LM head.
int distill_vocab_tiles(int V);
hipError_t launch_distill_fwd(const uint16_t* Ht, const uint16_t* Hs, const uint16_t* W, const uint8_t* valid, int N,
                              int d, int V, float* zt, float* zs, float* part, float* lse_t, float* lse_s, float* ce,
                              float* wtok, float* loss, float* ce_out, hipStream_t s);
hipError_t launch_distill_bwd(const uint16_t* W, int N, int d, int V, const float* zt, const float* zs,
                              const float* lse_t, const float* lse_s, const float* wtok, uint16_t* dz, int ldv,
                              uint16_t* dH, hipStream_t s);

// Hypernetwork (Sec. 2.2, Eq. 3) and AdamW.
struct HyperWs {
  float* gi;       // [2][L][3H] input part of the gates
  float* cache;    // [2][L][5H] h_prev, r, u, n, W_hn h_prev + b_hn
  float* o;        // [L][2H] GRU outputs
  int* lay;        // [max chunks] layer of each head chunk
  int64_t* start;  // [max chunks] first row
  int64_t* end;    // [max chunks] one past the last row
  int* first;      // [L + 1] first chunk of each layer
  int* count;      // [1] number of chunks
  float* part;     // [max chunks][2H] chunk partials of do
  float* dout;     // [L][2H] gradient of the GRU outputs
  float* dgi;      // [2][L][3H] gate gradients, input side
  float* dgh;      // [2][L][3H] gate gradients, recurrent side
};
int hyper_max_chunks(int64_t G_total, int L);
hipError_t launch_hyper_fwd(const float* z, const float* gru, const float* A, const float* c, const int64_t* offsets,
                            int L, int D, int H, int64_t G_total, float* logits, const HyperWs& w, hipStream_t s);
hipError_t launch_hyper_bwd(const float* dlogits, const float* z, const float* gru, float* A, float* c, float* mA,
                            float* vA, float* mc, float* vc, int L, int D, int H, int64_t G_total, double lr,
                            double beta1, double beta2, double eps, double weight_decay, int step, float* dgru,
                            const HyperWs& w, hipStream_t s);
hipError_t launch_adamw(float* p, const float* g, float* m, float* v, int64_t n, double lr, double beta1,
                        double beta2, double eps, double weight_decay, int step, hipStream_t s);

}  // namespace gm
