// Host test of the projections' plans (csrc/gemm_plan.cpp), built with g++ by
// tests/test_gemm_plan.py.
#include "gemm_plan.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>

using namespace via;

#define CHECK(c, ...)                                    \
  do {                                                   \
    if (!(c)) {                                          \
      std::printf("%s:%d: %s: ", __FILE__, __LINE__, #c); \
      std::printf(__VA_ARGS__);                          \
      std::printf("\n");                                 \
      std::exit(1);                                      \
    }                                                    \
  } while (0)

struct Model {
  const char* name;
  int d, H, KVH, hd, F;
  int step;  // of the max_rows looked at
};
constexpr Model kModels[] = {
    {"8b", 4096, 32, 8, 128, 14336, 1},     {"1b", 2048, 16, 4, 128, 5632, 1},  {"small", 512, 8, 2, 128, 1408, 17},
    {"micro", 256, 4, 2, 64, 512, 17},      {"odd", 2112, 16, 4, 128, 4160, 17}, {"wide", 8192, 64, 8, 128, 28672, 17},
    {"narrow", 1024, 16, 16, 64, 8192, 17},
};
constexpr int kRows = 2600;  // past kFixedOrderRows and several of its tile counts

// The workspace of a handle holds the partial products of every forward it
// admits, not only of its largest.
static void partials_fit(const Model& m, bool bf16) {
  const GemmShape g[] = {gemm_shape(GemmRole::kQkv, (m.H + 2 * m.KVH) * m.hd, m.d),
                         gemm_shape(GemmRole::kO, m.d, m.H * m.hd), gemm_shape(GemmRole::kDown, m.d, m.F)};
  size_t need = 0, last = 0;
  for (int R = 1; R <= kRows; ++R) {
    for (const GemmShape& s : g) need = std::max(need, (size_t)s.splits(bf16, R) * R * s.N);  // of any M <= R
    if (R % m.step) continue;
    const size_t have = gemm_part_floats(bf16, g, 3, R);
    CHECK(have >= need, "%s bf16=%d max_rows=%d: %zu floats reserved, %zu written", m.name, bf16, R, have, need);
    CHECK(have >= last, "%s bf16=%d max_rows=%d: shrinks from %zu to %zu", m.name, bf16, R, last, have);
    last = have;
  }
}

// All row counts of a block of 32 get the plan of its last one: a sequence's
// sums keep their order when a row is added inside the block.
static void plans_follow_blocks(const Model& m) {
  const struct {
    GemmRole role;
    int N, K;
  } shapes[] = {{GemmRole::kQkv, (m.H + 2 * m.KVH) * m.hd, m.d}, {GemmRole::kO, m.d, m.H * m.hd},
                {GemmRole::kGateUp, 2 * m.F, m.d},               {GemmRole::kDown, m.d, m.F},
                {GemmRole::kHead, 32000, m.d}};
  for (const auto& s : shapes)
    for (int M = 1; M <= kRows; ++M) {
      const int E = (M + 31) / 32 * 32;
      const GemmPath a = gemm_path(true, s.role, M, s.N, s.K), b = gemm_path(true, s.role, E, s.N, s.K);
      CHECK(a == b, "%s role %d M=%d", m.name, (int)s.role, M);
      if (a != GemmPath::kRowTile) continue;
      const RtPlan p = row_tile_plan(s.role, M, s.N, s.K), q = row_tile_plan(s.role, E, s.N, s.K);
      CHECK(p.rows == q.rows && p.cols == q.cols && p.ks == q.ks, "%s role %d M=%d: %dx%d/%d, M=%d: %dx%d/%d", m.name,
            (int)s.role, M, p.rows, p.cols, p.ks, E, q.rows, q.cols, q.ks);
    }
}

// A short K is split too where its tiles leave the GPU idle (512 columns or
// fewer), into no less than 8 K steps.
static void short_k_is_split() {
  for (int K : {512, 1024, 1408, 2048}) {
    const int ks = row_tile_plan(GemmRole::kO, 33, 512, K).ks;
    CHECK(ks == (K >= 1024 ? 4 : 2), "K=%d: %d splits", K, ks);
  }
}

int main() {
  short_k_is_split();
  for (const Model& m : kModels) plans_follow_blocks(m);
  for (const Model& m : kModels)
    for (bool bf16 : {true, false}) partials_fit(m, bf16);
  std::printf("ALL OK\n");
}
