// Which tile a GEMM launch takes: estimated times, on the host, of the tiles
// that fit a shape.  No device code and no HIP headers.
#pragma once

#include <stdint.h>

namespace gm {

// Estimated time of a GEMM launch whose blocks (one per CU) take block_ns each:
// whole rounds of 256 blocks, and a last round that is partly empty at half a
// round plus half its fill (its blocks run faster alone); less than one round
// costs a whole one.
inline int64_t rounds_ns(int64_t blocks, int64_t block_ns) {
  const int64_t full = blocks / 256, rest = blocks % 256;
  if (full == 0) return block_ns;
  return full * block_ns + (rest ? block_ns / 2 + block_ns * rest / 512 : 0);
}

inline int64_t tile_blocks(int64_t m, int64_t n, int64_t bm, int64_t bn) {
  return ((m + bm - 1) / bm) * ((n + bn - 1) / bn);
}

// Output tiles of the forward GEMM, rows of Y's columns (o) x tokens; the two
// 128-token tiles split K over two wave groups inside the block.
enum class FwdTile { k256x256, k256x128, k128x128 };

// Selectors per row that the 256-row tiles have LDS for beside their rings (1 x g groups; the in-place 256 x 256
// tile and the 128 x 128 tiles hold every row the library accepts).
constexpr int fwd_max_groups(int g, bool packed, bool half) {
  return packed && half && 16384 / g > 128 ? 128 : 16384 / g;
}

// Tile of the forward GEMM: the one with the lowest estimated time, rounds of
// blocks (rounds_ns) that take a fixed time (launch, mask bits, pipeline
// fill, epilogue) and a time per 32-deep K slice.  Measured (4096 x 4096, half the groups kept): 256 x 256 tiles 15 us + 0.66
// us per slice; 256 x 128 (K over two wave groups) 14 us + 0.42; 128 x 128
// (same) 9 us + 0.25; a K split over blocks adds a reduction of 4 us and 8
// bytes per output and share (mostly cached: 15 TB/s for the few shares of 256 x
// 256 tiles, 8 TB/s for up to eight of 128 x 128 ones).  Splitting the smaller
// tile: 4096 x 4096, T = 128 22 us (unsplit 38, 256 x 256 split in eight 28), T =
// 512 31 (39, 40); 4096 x 11008 inputs, T = 128 28 (92, 44); 2816 x 2056, T = 300
// 19 (28, 29).  The model picks the
// fastest or within 3 % of it at T = 128 .. 4096 on 1024^2, 2816 x 2056, 4096^2,
// 11008 x 4096 (both ways) and the LLaMA-2-13B shapes: e.g. T = 2048 at 4096^2
// 65 us in 256 x 128 tiles (256 x 256 split in two: 73), T = 1024 41 us in 128 x
// 128 tiles (split in four: 50), T = 4096 98 us in 256 x 256 tiles (125).
struct FwdPlan {
  FwdTile tile;
  int ks;
  int64_t ns;  // estimated time
};

inline bool fwd_tile_fits(FwdTile tile, int64_t d_in, int32_t g, int32_t g_out, bool packed) {
  if (tile == FwdTile::k128x128) return true;
  if (g < 32 || (packed && g < 64)) return tile == FwdTile::k256x256 && !packed;
  if (g_out != 1 || (tile == FwdTile::k256x256 && !packed)) return true;
  return d_in / g <= fwd_max_groups(g, packed, tile == FwdTile::k256x128);
}

// ks: shares of the 256 x 256 tile's K range (1 without a workspace).
inline FwdPlan fwd_plan(int64_t T, int64_t d_in, int64_t d_out, int32_t g, int32_t g_out, bool packed, int ks) {
  const int64_t slices = d_in / 32;
  auto tiles = [&](int64_t bm, int64_t bn) { return ((d_out + bm - 1) / bm) * ((T + bn - 1) / bn); };
  auto reduce_ns = [&](int64_t k, int64_t rate) { return 4000 + k * T * d_out * 8 / rate; };  // rate: bytes per ns
  FwdPlan best{FwdTile::k128x128, 1, rounds_ns(tiles(128, 128), 9000 + 250 * slices)};
  auto consider = [&](FwdTile tile, int k, int64_t ns) {
    if (ns < best.ns) best = {tile, k, ns};
  };
  for (int k = 2; k <= ks; ++k)  // ks: what the workspace holds
    consider(FwdTile::k128x128, k, rounds_ns(tiles(128, 128) * k, 9000 + 250 * slices / k) + reduce_ns(k, 8000));
  if (fwd_tile_fits(FwdTile::k256x128, d_in, g, g_out, packed))
    consider(FwdTile::k256x128, 1, rounds_ns(tiles(256, 128), 14000 + 420 * slices));
  if (fwd_tile_fits(FwdTile::k256x256, d_in, g, g_out, packed))
    consider(FwdTile::k256x256, ks, rounds_ns(tiles(256, 256) * ks, 15000 + 660 * slices / ks) + (ks > 1 ? reduce_ns(ks, 15000) : 0));
  return best;
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
// less on the density.  5120 x 5120, T = 17 / 64 / 128, half the groups kept, us in
// passes and in the GEMM: 23, 49 / 32, 49 / 48, 50; 15360 x 5120: 39, 49 / 67, 50 /
// 117, 55; 1024 x 4096: 14, 44 / 14, 44 / 19, 46; 10 % kept, 5120 x 5120: 22, 48 /
// 31, 49 / 45, 49.  Rows of too many groups for the tables (16-wide, above 512)
// take one wave per row and pass: 2048 x 16384, T = 33 / 65 151, 226 / 290, 225.
inline bool packed_passes(int64_t T, int64_t d_in, int64_t d_out, int32_t g, int64_t gemm_ns) {
  const int64_t rows = passes_rows(T, d_in, d_out, g), slices = d_in / 32, G_in = d_in / g;
  if (rows == 0) return T <= 48;
  if (T > 512) return false;  // not measured beyond
  const int64_t blocks = (d_out + rows - 1) / rows * ((T + 15) / 16);
  const int64_t more = blocks > 256 ? (blocks - 256) * (42 * slices + 16 * G_in) * rows / (32 * 256) : 0;
  return (7000 + 90 * slices + 25 * G_in + more) * 115 < gemm_ns * (g == 16 ? 150 : 100);
}

// Columns (o) of the 256-row (i) tiles of dgate: the tile with the lowest estimated time: rounds of 256 blocks (a partly
// empty last round costs a whole one) of 13 us + 0.62 us per K slice for 256 x
// 256, 13 + 0.415 for 256 x 128, 7 + 0.32 for 256 x 64 (1 x g groups only: its
// waves hold 32 columns).  E.g. 1024 x 1024, T = 2048: 49 us in 256 x 256, 40 in
// 256 x 128, 26 in 256 x 64; 2816 x 2056, T = 1000: 34 / 27 / 33; 4096 x 4096, T
// = 2048: 61 / 80 / 104.
inline int dgate_columns(int64_t T, int64_t d_in, int64_t d_out, int g_out) {
  const int64_t sl = (T + 31) / 32;
  auto est = [&](int64_t bn, int64_t ns) { return (tile_blocks(d_in, d_out, 256, bn) + 255) / 256 * ns; };
  const int64_t big = est(256, 13000 + 620 * sl), half = est(128, 13000 + 415 * sl),
                low = g_out == 1 ? est(64, 7000 + 320 * sl) : INT64_MAX;
  return low < half && low < big ? 64 : half < big ? 128 : 256;
}

// Tiles of dX over column lists: 256 x 256, 256 x 128, 128 x 256, 128 x 128, 64 x
// 128 (the 128-token ones on two K groups), and 64 x 256, two blocks to a CU.
enum class DxTile { kBig, kHalf, kWide, kMid, kLow, kPair };

// The tile with the lowest estimated time among those that divide the list
// column; the slices of a column are taken as half its rows.  Us per block
// and round + us per 32-deep slice, fitted to LLaMA-2-7B shapes at T = 128 ..
// 4096, half the groups kept: 256 x 256 19 + 0.64, 256 x 128 (two K groups)
// 16 + 0.49, 128 x 256 14 + 0.62, 128 x 128 (two) 13 + 0.39, 64 x 128 (two)
// 15 + 0.29; the 64 x 256 tile runs two blocks per CU (13 + 0.78 per round of
// 512, 13 + 0.50 below half of one).  E.g. 4096 x 4096, 1 x 256 groups: T =
// 4096 67 us in 256 x 256 tiles (96 in 256 x 128), T = 2048 51 in 256 x 128 (59),
// T = 1024 38 in 128 x 128 (58), T = 128 32 in 64 x 128 (44 in 64 x 256); 11008
// rows, T = 1024 81 in 128 x 128 (128 in 256 x 256).
inline DxTile dx_tile(int64_t T, int64_t d_in, int64_t d_out, int32_t g) {
  if (g < 64) return DxTile::kPair;  // list columns of several groups
  const int64_t sl = (d_out + 63) / 64;
  auto blocks = [&](int64_t bm, int64_t bn) { return tile_blocks(d_in, T, bm, bn); };
  DxTile tile = DxTile::kLow;
  int64_t best = rounds_ns(blocks(64, 128), 15000 + 290 * sl);
  auto consider = [&](DxTile t, int64_t ns) {
    if (ns < best) tile = t, best = ns;
  };
  if (g >= 128) consider(DxTile::kMid, rounds_ns(blocks(128, 128), 13000 + 390 * sl));
  if (g == 128) consider(DxTile::kWide, rounds_ns(blocks(128, 256), 14000 + 620 * sl));
  if (g >= 256) consider(DxTile::kHalf, rounds_ns(blocks(256, 128), 16000 + 490 * sl));
  if (g >= 256) consider(DxTile::kBig, rounds_ns(blocks(256, 256), 19000 + 640 * sl));
  if (g == 64)
    consider(DxTile::kPair, blocks(64, 256) <= 256 ? 13000 + 500 * sl : rounds_ns(blocks(64, 256) / 2, 13000 + 780 * sl));
  return tile;
}

// dX of 16 x 16 and 32 x 32 groups goes over the mask rows of a tile's columns, straight from dY and W (no column
// lists, no dY^T), where a block has room for their kept bits.
constexpr int kWtMaskRows = 2048;
inline bool dx_dense_ok(int64_t d_out, int32_t g) { return g < 64 && d_out / g <= kWtMaskRows; }

// Tiles of that dX and of the LM head's backward.
enum class WtTile { k256x256, k256x128, k128x128 };
inline WtTile wt_tile_of(int64_t m, int64_t n, int64_t big, int64_t half, int64_t mid) {  // ns per block and round
  big = rounds_ns(tile_blocks(m, n, 256, 256), big);
  half = rounds_ns(tile_blocks(m, n, 256, 128), half);
  mid = rounds_ns(tile_blocks(m, n, 128, 128), mid);
  return mid < half && mid < big ? WtTile::k128x128 : half < big ? WtTile::k256x128 : WtTile::k256x256;
}

// The tile with the lowest estimated time (us per block and round: 10 + 0.70
// per K slice for 256 x 256, 11 + 0.45 for 256 x 128, 7 + 0.24 for 128 x 128;
// 4096 x 4096, 32 x 32 groups: T = 4096 101 / 127 / 150 us, T = 2048 97 / 69 /
// 78, T = 512 88 / 60 / 37).
inline int64_t dx_dense_ns(WtTile tile, int64_t d_out) {  // of one block
  const int64_t slices = (d_out + 31) / 32;
  return tile == WtTile::k256x256 ? 10000 + 700 * slices : tile == WtTile::k256x128 ? 11000 + 450 * slices : 7000 + 240 * slices;
}
inline WtTile dx_dense_tile(int64_t T, int64_t d_in, int64_t d_out) {
  return wt_tile_of(d_in, T, dx_dense_ns(WtTile::k256x256, d_out), dx_dense_ns(WtTile::k256x128, d_out),
                    dx_dense_ns(WtTile::k128x128, d_out));
}

// Time until n1 blocks of t1 ns and then n2 of t2, one per CU and each on the first free CU, have ended: the first
// kind leaves 256 - r CUs free at `free` and r one block later; the end is one of theirs plus whole blocks of t2.
inline int64_t two_kinds_ns(int64_t n1, int64_t t1, int64_t n2, int64_t t2) {
  const int64_t r = n1 % 256, free = n1 / 256 * t1;
  int64_t best = INT64_MAX;
  for (int late = 0; late < 2; ++late) {
    const int64_t from = late ? free + t1 : free;
    auto done = [&](int64_t k) {  // blocks ended by from + k t2
      const int64_t end = from + k * t2;
      return (256 - r) * ((end - free) / t2) + (end > free + t1 ? r * ((end - free - t1) / t2) : 0);
    };
    int64_t lo = 0, hi = n2;  // (n2 on one CU are done by n2 t2)
    while (lo < hi) {
      const int64_t mid = (lo + hi) / 2;
      if (done(mid) >= n2) hi = mid; else lo = mid + 1;
    }
    const int64_t end = from + lo * t2;
    if (end < best) best = end;
  }
  return best > free + (r ? t1 : 0) ? best : free + (r ? t1 : 0);
}

// dX and dgate of those groups share a launch: whether the dX tiles go first.  4096 x 11008, T = 2048, 32 x 32 groups
// half kept: 327 us dX first, 367 dgate first (in two launches 364); 4096 x 4096, T = 512 51, 64 (66); 11008 x 4096, T =
// 1024, equal by this estimate, 220, 203 (204).
inline bool square_dx_first(int64_t T, int64_t d_in, int64_t d_out, int32_t g) {
  const WtTile tile = dx_dense_tile(T, d_in, d_out);
  const int64_t bm = tile == WtTile::k128x128 ? 128 : 256, bn = tile == WtTile::k256x256 ? 256 : 128;
  const int64_t cols = dgate_columns(T, d_in, d_out, g), sl = (T + 31) / 32;
  const int64_t nx = tile_blocks(d_in, T, bm, bn), tx = dx_dense_ns(tile, d_out);
  const int64_t nd = tile_blocks(d_in, d_out, 256, cols), td = 13000 + (cols == 256 ? 620 : 415) * sl;
  return two_kinds_ns(nx, tx, nd, td) < two_kinds_ns(nd, td, nx, tx);
}

// The tile with the fewest estimated rounds of 256 blocks times the time per
// K slice (cold head and dz: 0.72 us for 256 x 256, 0.60 for 256 x 128, 0.37
// for 128 x 128, measured at V = 32000, d = 4096): N = 4096 keeps 256 x 256
// (0.93 ms against 1.18 and 1.56), N = 2048 takes 256 x 128 (0.60 ms against
// 0.72 and 0.73), N <= 1024 128 x 128 (0.37 ms against 0.70 and 0.51).
inline WtTile lm_bwd_tile(int64_t N, int64_t d) { return wt_tile_of(d, N, 720, 600, 370); }

}  // namespace gm
