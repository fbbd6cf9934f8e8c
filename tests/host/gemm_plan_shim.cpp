// C entry points to the projections' plans (csrc/gemm_plan.cpp) for the Python
// tests (tests/gemm_plans.py).
#include "gemm_plan.h"

extern "C" int plan_path(int role, int M, int N, int K) {
  return (int)via::gemm_path(true, (via::GemmRole)role, M, N, K);
}
extern "C" void plan_tile(int role, int M, int N, int K, int* rows, int* cols, int* splits) {
  const via::RtPlan p = via::row_tile_plan((via::GemmRole)role, M, N, K);
  *rows = p.rows;
  *cols = p.cols;
  *splits = p.ks;
}
