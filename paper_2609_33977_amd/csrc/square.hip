// Backward of 16 x 16 and 32 x 32 groups whose dX needs no column lists.
#include "gm_dgate.h"
#include "gm_launch.h"
#include "gm_wt.h"

namespace gm {

// dX over the mask rows that keep something in the tile's columns: a list
// column of 64 input columns (four or two groups) keeps 94 % or 75 % of the rows
// at half the groups kept, so gathering single rows saves little, and its
// 64-column tiles move 1.9 times the operand bytes per MFMA of a 256-column tile.
template <int G, int BM, int BN, int KS>
__global__ __launch_bounds__(512) void dx_dense_kernel(const uint16_t* __restrict__ dY, const uint16_t* __restrict__ W,
                                                       const float* __restrict__ mask, int T, int d_in, int d_out,
                                                       uint16_t* __restrict__ dX) {
  __shared__ u32x4 smem[wt_smem(BM, BN, KS)];
  __shared__ WtMask sm;
  __shared__ float s_msoft[wt_stages(BM, BN, KS) * 512];
  wt_gemm_masked<G, BM, BN, KS>(dY, d_out, W, d_out, d_in, T, mask, dX, int(blockIdx.x), int(gridDim.x), smem, sm, s_msoft);
}

// dX and dgate in one launch (neither needs the other here): its first `first`
// blocks are the dX tiles if dx_first, else the 256 x BND dgate tiles.  32 x 32 groups,
// us in two launches / in one: 4096 x 4096 half kept T = 512 66 / 51, T = 2048 126 /
// 124, 10 % kept 106 / 103; 4096 x 11008 T = 2048 half kept 364 / 327, 10 % 305 /
// 286; 1024 x 1024 T = 1000 44 / 30.
template <int G, int BND, int BM, int BN, int KS>
__global__ __launch_bounds__(512) void square_bwd_kernel(const uint16_t* __restrict__ dY, const uint16_t* __restrict__ X,
                                                         const uint16_t* __restrict__ W, const float* __restrict__ mask,
                                                         int T, int d_in, int d_out, uint16_t* __restrict__ dX,
                                                         float* __restrict__ dgate, int first, bool dx_first) {
  constexpr int KSD = BND == 256 ? 1 : 2, S1 = wt_smem(BM, BN, KS), S2 = dgate_smem(BND, KSD);
  constexpr int SM = wt_stages(BM, BN, KS) * 128;  // of 16 bytes: the dX tiles' selectors, behind their rings
  __shared__ u32x4 smem[S1 + SM > S2 ? S1 + SM : S2];
  __shared__ WtMask sm;
  const bool head = int(blockIdx.x) < first;
  const int bid = head ? int(blockIdx.x) : int(blockIdx.x) - first;
  if (head == dx_first)
    wt_gemm_masked<G, BM, BN, KS>(dY, d_out, W, d_out, d_in, T, mask, dX, bid, dx_first ? first : int(gridDim.x) - first,
                                  smem, sm, reinterpret_cast<float*>(smem + S1));
  else
    dgate_tile<G, G, BND, KSD, false>(dY, X, W, T, d_in, d_out, dgate, nullptr, 0, ListArgs{}, bid, smem);
}

hipError_t launch_square_bwd(const uint16_t* dY, const uint16_t* X, const uint16_t* W, const float* mask, int T, int d_in,
                             int d_out, int g, uint16_t* dX, float* dgate, hipStream_t s) {
  const WtTile tile = dx_dense_tile(T, d_in, d_out);
  const int columns = dgate_columns(T, d_in, d_out, g);  // 128 or 256
  const int dg = dgate ? int(tile_blocks(d_in, d_out, 256, columns)) : 0;
  const bool dx_first = dgate && square_dx_first(T, d_in, d_out, g);
#define GM_SQUARE(G, BM, BN, KS)                                                                                          \
  {                                                                                                                       \
    const int dx = int(tile_blocks(d_in, T, BM, BN)), first = dx_first ? dx : dg;                                         \
    if (!dgate)                                                                                                           \
      hipLaunchKernelGGL((dx_dense_kernel<G, BM, BN, KS>), dim3(dx), dim3(512), 0, s, dY, W, mask, T, d_in, d_out, dX);    \
    else if (columns == 256)                                                                                              \
      hipLaunchKernelGGL((square_bwd_kernel<G, 256, BM, BN, KS>), dim3(dx + dg), dim3(512), 0, s, dY, X, W, mask, T, d_in, \
                         d_out, dX, dgate, first, dx_first);                                                                           \
    else                                                                                                                  \
      hipLaunchKernelGGL((square_bwd_kernel<G, 128, BM, BN, KS>), dim3(dx + dg), dim3(512), 0, s, dY, X, W, mask, T, d_in, \
                         d_out, dX, dgate, first, dx_first);                                                                           \
  }
#define GM_SQUARE_G(G)                                              \
  {                                                                 \
    if (tile == WtTile::k128x128) GM_SQUARE(G, 128, 128, 2)         \
    else if (tile == WtTile::k256x128) GM_SQUARE(G, 256, 128, 2)    \
    else GM_SQUARE(G, 256, 256, 1)                                  \
  }
  if (g == 16)
    GM_SQUARE_G(16)
  else if (g == 32)
    GM_SQUARE_G(32)
  else
    return hipErrorInvalidValue;
#undef GM_SQUARE_G
#undef GM_SQUARE
  return hipGetLastError();
}

}  // namespace gm
