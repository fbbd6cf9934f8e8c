// Which kernel family, tile and K splits a projection runs with.  Plain C++:
// the runtime sizes its workspace from these functions and the GEMM launchers
// follow them, and they build without HIP.
#pragma once
#include <stddef.h>

namespace via {

// Projection a GEMM computes: the head reduces its tiles to row statistics
// instead of writing partials; the gate/up projection runs over all of K and
// applies SwiGLU itself.
enum class GemmRole { kQkv, kO, kGateUp, kDown, kHead };

// Kernel family of an [M, K] x [N, K]^T projection.
//   kStream   bf16, up to 32 rows: weights stream past registers; QKV, O and
//             down in work-groups of 16-column blocks of one K split
//             (gemm_ki_plan), gate/up over all of K
//   kRowTile  bf16, 33 rows and more (the head's only kernel there): LDS-fed
//             tiles of 64 to 128 rows x 128 or 256 columns (row_tile_plan)
//   kPrefill  bf16, enough rows to fill the GPU with 256 x 256 tiles (one partial)
//   kHead     the bf16 head of up to 32 rows
//   kF32      every projection and size of fp32 models (one partial)
enum class GemmPath { kStream, kRowTile, kPrefill, kHead, kF32 };
GemmPath gemm_path(bool bf16, GemmRole role, int M, int N, int K);

// Forwards of more rows than this sum every projection in one order (no K
// splits, K steps one after another), so that a row's result does not depend on
// the rows it is batched with.
constexpr int kFixedOrderRows = 512;
// Tile of the prefill kernel.
constexpr int kPfBM = 256, kPfBN = 256;

// Tile and K splits of one projection on the kRowTile kernel.
struct RtPlan {
  int rows, cols, ks;
  double us;  // estimate
};
RtPlan row_tile_plan(GemmRole role, int M, int N, int K);

// Blocks per work-group and K splits of the kStream kernels for an [N, K]
// weight (about 256 work-groups).
void gemm_ki_plan(int N, int K, int* nb, int* ksplit);
// 16-column blocks per gate/up work-group of the kStream kernel for d_ffn = F
// (1..8, about one work-group per compute unit).
int gate_up_blocks_per_group(int F);
// Column tiles the head of M rows reduces its statistics to.
int gemm_head_tiles(bool bf16, int M, int N, int K);
// Rows of the activation fragments for M rows: M padded to a multiple of 16,
// 32, 48, 64, 96 or 128 (the larger, the more rows); non-decreasing in M.
int gemm_padded_rows(int M);

// A projection that writes partial products, [splits][M][N] fp32.
struct GemmShape {
  int N, K;
  GemmRole role;
  int nb_ki, ks_ki;  // gemm_ki_plan
  // K splits of a forward of M rows: what a launch writes and the workspace
  // is sized by.
  int splits(bool bf16, int M) const;
};
GemmShape gemm_shape(GemmRole role, int N, int K);
// The most partial products (floats) the n projections write in any forward
// of 1 to max_rows rows.
size_t gemm_part_floats(bool bf16, const GemmShape* g, int n, int max_rows);

}  // namespace via
