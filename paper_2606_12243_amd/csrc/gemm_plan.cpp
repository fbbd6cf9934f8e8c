// Kernel choice of the projections (gemm_plan.h).
#include "gemm_plan.h"

#include <algorithm>

namespace via {

namespace {
constexpr int kGroupBlocks = 8;      // 16-column blocks of a kStream work-group at most (one a wave)
constexpr int kHeadTileCols = 256;   // columns of a kHead tile
constexpr int kF32HeadTileCols = 64;  // ... and of an fp32 head tile
int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Time of an fp32 [M, N] partial, written and read back at ~3 TB/s.  Rows count
// in blocks of 32, which every tile height is a multiple of: all row counts of a
// block then get one plan, and a forward's sums do not change their order when
// one row is added inside a block.
double partial_us(int M, int N) { return 8e-6 / 3.0 * (ceil_div(M, 32) * 32) * (double)N; }
}  // namespace

// The tile and split with the smallest estimate: rounds of tiles on 256 compute
// units and every split's partial.  The time of a round per 4096 of K is measured
// on the 8B gate/up projection (48, 96, 128, 160 and 256 rows); QKV, O, down and
// narrower models take it over, it was not measured on each of them.  Up to 4
// splits have at least 8 K steps each, 8 splits 16: the steps of a split run one
// after another, and short K is all latency (a window, at least 16 | 8 steps: width
// 512 33 rows 247 | 222 us, 128 rows 261 | 237; 1B widths, 8 splits of 8 steps, 33
// rows 318 | 310 but 128 rows 374 | 381).  Above
// kFixedOrderRows rows there is one split and one order of summation (that of
// the prefill tiles too), whatever the row count.
RtPlan row_tile_plan(GemmRole role, int M, int N, int K) {
  struct Tile {
    int rows, cols;
    double us;
  };
  static constexpr Tile kTiles[] = {{64, 128, 48.0}, {96, 128, 53.0}, {128, 128, 64.0}, {96, 256, 74.0}, {128, 256, 92.0}};
  const bool split = role != GemmRole::kGateUp && role != GemmRole::kHead && M <= kFixedOrderRows;
  RtPlan best{0, 0, 0, 0.0};
  for (const Tile& tl : kTiles) {
    const int tiles = ceil_div(M, tl.rows) * ceil_div(N, tl.cols);
    for (int ks = 1; ks <= (split ? 8 : 1) && (ks == 1 || K / 32 >= (ks <= 4 ? 8 : 16) * ks); ks *= 2) {
      const double us = 10.0 + tl.us * ceil_div(tiles * ks, 256) * K / (4096.0 * ks) + ks * partial_us(M, N);
      if (!best.ks || us < best.us) best = RtPlan{tl.rows, tl.cols, ks, us};
    }
  }
  return best;
}

GemmPath gemm_path(bool bf16, GemmRole role, int M, int N, int K) {
  if (!bf16) return GemmPath::kF32;
  if (M <= 32) return role == GemmRole::kHead ? GemmPath::kHead : GemmPath::kStream;
  if (M <= 128 || role == GemmRole::kHead) return GemmPath::kRowTile;
  // 256 x 256 tiles take 178 us a round per 4096 of K, less than the two rounds
  // of row tiles they stand for, when there are enough of them
  const int tiles = ceil_div(M, kPfBM) * ceil_div(N, kPfBN);
  const double us = 20.0 + 178.0 * ceil_div(tiles, 256) * K / 4096.0 + partial_us(M, N);
  return us < row_tile_plan(role, M, N, K).us ? GemmPath::kPrefill : GemmPath::kRowTile;
}

void gemm_ki_plan(int N, int K, int* nb, int* ksplit) {
  const int S = K / 32, blocks = N / 16;
  // at least 4 steps per wave in a split; long K (the down projection) in 8
  // splits, which with 8 blocks per work-group halves the activation reads
  // per weight byte and keeps the grid at one round
  const int ks = S >= 256 ? 8 : std::max(1, std::min(4, S / 32));
  *ksplit = ks;
  *nb = std::max(1, std::min(kGroupBlocks, ceil_div(blocks * ks, 256)));
}

int gate_up_blocks_per_group(int F) {
  const int nblocks = F / 8;  // 2 F columns in blocks of 16
  return std::max(1, std::min(kGroupBlocks, ceil_div(nblocks, 256)));
}

int gemm_head_tiles(bool bf16, int M, int N, int K) {
  if (!bf16) return ceil_div(N, kF32HeadTileCols);
  const bool tall = gemm_path(bf16, GemmRole::kHead, M, N, K) == GemmPath::kRowTile;
  return ceil_div(N, tall ? row_tile_plan(GemmRole::kHead, M, N, K).cols : kHeadTileCols);
}

int gemm_padded_rows(int M) {
  const int g = M > 96 ? 128 : M > 64 ? 96 : M > 48 ? 64 : M > 32 ? 48 : M > 16 ? 32 : 16;
  return ceil_div(M, g) * g;
}

GemmShape gemm_shape(GemmRole role, int N, int K) {
  GemmShape g{N, K, role, 1, 1};
  gemm_ki_plan(N, K, &g.nb_ki, &g.ks_ki);
  return g;
}

int GemmShape::splits(bool bf16, int M) const {
  switch (gemm_path(bf16, role, M, N, K)) {
    case GemmPath::kStream: return ks_ki;
    case GemmPath::kRowTile: return row_tile_plan(role, M, N, K).ks;
    default: return 1;
  }
}

// Every row count is looked at, up to where there is one split: the split count
// falls as rows are added, so the peak lies anywhere below max_rows.
size_t gemm_part_floats(bool bf16, const GemmShape* g, int n, int max_rows) {
  size_t most = 0;
  for (int i = 0; i < n; ++i) {
    for (int M = 1; M <= std::min(max_rows, kFixedOrderRows); ++M)
      most = std::max(most, (size_t)g[i].splits(bf16, M) * M * g[i].N);
    if (max_rows > kFixedOrderRows) most = std::max(most, (size_t)max_rows * g[i].N);
  }
  return most;
}

}  // namespace via
