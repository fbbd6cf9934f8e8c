// Routing-mask cost of DIMR: the KL-style verification cost R^KL(q || q'_z)
// of Sec. 3 (Eq. 11, ReLU surrogate) for every row of a pair of logit
// matrices, q = the full verifier, p = q'_z the routed slim verifier.  With
// l = log softmax(logits / T):
//   R = sum_v p(v) ReLU(log(1-alpha) + l_p(v) - l_q(v))
//     + sum_v q(v) ReLU(log(beta)    + l_p(v) - l_q(v)).
// One 512-thread work-group per row: a pass for the two log-partition
// functions, then the cost pass.  With few rows the vector ALUs of the compute
// units in use bound it, with many HBM, so:
//  - an exponential is one v_exp_f32, and the running maximum moves once per
//    kIds ids, not per id;
//  - loads run a group of rounds ahead of their use;
//  - between the passes the first KEEP rounds of a row stay in registers and
//    the next LDS in LDS, so the second pass reads neither again.  Up to one
//    row per compute unit a work-group has the whole unit and keeps 57344 ids;
//    with more, two share it and keep 24576 each, one computing while the other
//    loads.
// Partial sums are combined in a fixed order (the cost's in fp64), so the
// result is reproducible.
#include "kernels.h"

namespace via {

namespace {

constexpr int kDimrThreads = 512;
constexpr int kIds = 4;  // consecutive ids of a thread per round
constexpr int kRoundIds = kDimrThreads * kIds;

constexpr float kLog2e = 1.4426950408889634f;
__device__ __forceinline__ float exp_fast(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }

// (maximum, sum of exp(z - maximum)) of some ids' scaled logits
struct Lse {
  float m, s;
};
__device__ __forceinline__ void lse_add(Lse& a, float4 z) {
  const float mx = fmaxf(fmaxf(z.x, z.y), fmaxf(z.z, z.w));
  if (mx > a.m) {
    a.s *= exp_fast(a.m - mx);  // (0 at first)
    a.m = mx;
  }
  const float m = a.m == -INFINITY ? 0.f : a.m;  // only ids past the vocabulary so far: each adds 0
  a.s += (exp_fast(z.x - m) + exp_fast(z.y - m)) + (exp_fast(z.z - m) + exp_fast(z.w - m));
}
__device__ __forceinline__ Lse lse_merge(Lse a, Lse b) {
  if (b.m == -INFINITY) return a;
  if (a.m == -INFINITY) return b;
  const float M = fmaxf(a.m, b.m);
  return Lse{M, a.s * exp_fast(a.m - M) + b.s * exp_fast(b.m - M)};
}

// Logits v .. v + 3 of a row over T (ALIGNED: every row starts on 16 bytes).
template <bool ALIGNED>
__device__ __forceinline__ float4 load_ids(const float* r, float inv_T) {
  float4 z;
  if constexpr (ALIGNED)
    z = *(const float4*)r;
  else
    z = make_float4(r[0], r[1], r[2], r[3]);
  return make_float4(z.x * inv_T, z.y * inv_T, z.z * inv_T, z.w * inv_T);
}
// The same at the end of the vocabulary (n ids left): ids past it read as -inf.
__device__ __forceinline__ float4 load_last(const float* r, int n, float inv_T) {
  return make_float4(n > 0 ? r[0] * inv_T : -INFINITY, n > 1 ? r[1] * inv_T : -INFINITY,
                     n > 2 ? r[2] * inv_T : -INFINITY, n > 3 ? r[3] * inv_T : -INFINITY);
}

template <bool ALIGNED, int KEEP, int LDS, int GROUP, int PER_CU>
__global__ __launch_bounds__(kDimrThreads, 2 * PER_CU) void dimr_cost_kernel(DimrArgs a) {
  static_assert(KEEP % GROUP == 0 && LDS % GROUP == 0, "whole groups are kept");
  constexpr int kGroups = KEEP / GROUP;
  const int row = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const float* q = a.q + (size_t)row * a.ld + t * kIds;
  const float* p = a.p + (size_t)row * a.ld + t * kIds;
  __shared__ __align__(16) float4 kept[LDS][2][kDimrThreads];
  __shared__ Lse part[2][kDimrThreads / 64];
  __shared__ double cost[kDimrThreads / 64][2];
  const int full = a.vocab / kRoundIds;  // rounds without an end, then perhaps one with
  struct Group {
    float4 q[GROUP], p[GROUP];
  };
  auto load = [&](Group& z, int g) {
#pragma unroll
    for (int u = 0; u < GROUP; ++u)
      if (g * GROUP + u < full) {  // uniform
        z.q[u] = load_ids<ALIGNED>(q + (size_t)(g * GROUP + u) * kRoundIds, a.inv_T);
        z.p[u] = load_ids<ALIGNED>(p + (size_t)(g * GROUP + u) * kRoundIds, a.inv_T);
      }
  };

  // first pass: the first kGroups groups into registers, the next LDS rounds into LDS
  Lse lq{-INFINITY, 0.f}, lp{-INFINITY, 0.f};
  auto sum = [&](const Group& z, int g) {
#pragma unroll
    for (int u = 0; u < GROUP; ++u)
      if (g * GROUP + u < full) {
        const int k = g * GROUP + u - KEEP;
        if (k >= 0 && k < LDS) {
          kept[k][0][t] = z.q[u];
          kept[k][1][t] = z.p[u];
        }
        lse_add(lq, z.q[u]);
        lse_add(lp, z.p[u]);
      }
  };
  Group reg[kGroups], s0, s1;
  load(reg[0], 0);
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    load(g + 1 < kGroups ? reg[g + 1] : s0, g + 1);
    sum(reg[g], g);
  }
  for (int g = kGroups; g * GROUP < full; g += 2) {
    load(s1, g + 1);
    sum(s0, g);
    if ((g + 1) * GROUP >= full) break;
    load(s0, g + 2);
    sum(s1, g + 1);
  }
  const int left = a.vocab - full * kRoundIds - t * kIds;  // this thread's ids of the last round
  float4 eq = load_last(q + (size_t)full * kRoundIds, left, a.inv_T);
  float4 ep = load_last(p + (size_t)full * kRoundIds, left, a.inv_T);
  lse_add(lq, eq);
  lse_add(lp, ep);
  // the second pass reads its first group while the sums are merged
  constexpr int kAgain = (KEEP + LDS) / GROUP;
  load(s0, kAgain);
  // log partition functions: lanes in a fixed tree, waves in order
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    lq = lse_merge(lq, Lse{__shfl_xor(lq.m, o, 64), __shfl_xor(lq.s, o, 64)});
    lp = lse_merge(lp, Lse{__shfl_xor(lp.m, o, 64), __shfl_xor(lp.s, o, 64)});
  }
  if (lane == 0) {
    part[0][wave] = lq;
    part[1][wave] = lp;
  }
  __syncthreads();
  lq = part[0][0];
  lp = part[1][0];
  for (int w = 1; w < kDimrThreads / 64; ++w) {
    lq = lse_merge(lq, part[0][w]);
    lp = lse_merge(lp, part[1][w]);
  }
  // an infinite logit makes log Z infinite (above, exp(inf - inf) made the sum a
  // NaN, which the comparisons below would turn into a cost of 0)
  if (lq.m == INFINITY) lq.s = 1.f;
  if (lp.m == INFINITY) lp.s = 1.f;
  const float lzq = lq.m + logf(lq.s), lzp = lp.m + logf(lp.s);

  // second pass
  double c1 = 0.0, c2 = 0.0;
  auto add1 = [&](float zq, float zp) {
    const float vq = zq - lzq, vp = zp - lzp, d = vp - vq;
    const float z1 = a.log_1m_alpha + d, z2 = a.log_beta + d;
    c1 += (double)(z1 > 0.f ? exp_fast(vp) * z1 : 0.f);
    c2 += (double)(z2 > 0.f ? exp_fast(vq) * z2 : 0.f);
  };
  auto add4 = [&](float4 zq, float4 zp) {
    add1(zq.x, zp.x);
    add1(zq.y, zp.y);
    add1(zq.z, zp.z);
    add1(zq.w, zp.w);
  };
  auto add = [&](const Group& z, int g) {
#pragma unroll
    for (int u = 0; u < GROUP; ++u)
      if (g * GROUP + u < full) add4(z.q[u], z.p[u]);
  };
#pragma unroll
  for (int g = 0; g < kGroups; ++g) add(reg[g], g);
  for (int k = 0; k < min(LDS, full - KEEP); ++k) add4(kept[k][0][t], kept[k][1][t]);
  for (int g = kAgain; g * GROUP < full; g += 2) {
    load(s1, g + 1);
    add(s0, g);
    if ((g + 1) * GROUP >= full) break;
    load(s0, g + 2);
    add(s1, g + 1);
  }
  if (left > 0) {
    add1(eq.x, ep.x);
    if (left > 1) add1(eq.y, ep.y);
    if (left > 2) add1(eq.z, ep.z);
    if (left > 3) add1(eq.w, ep.w);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    c1 += __shfl_xor(c1, o, 64);
    c2 += __shfl_xor(c2, o, 64);
  }
  if (lane == 0) {
    cost[wave][0] = c1;
    cost[wave][1] = c2;
  }
  __syncthreads();
  if (t == 0) {
    double r1 = 0.0, r2 = 0.0;
    for (int w = 0; w < kDimrThreads / 64; ++w) {
      r1 += cost[w][0];
      r2 += cost[w][1];
    }
    a.cost[row] = (float)(r1 + r2);
  }
}

}  // namespace

void launch_dimr_cost(const DimrArgs& a, hipStream_t s) {
  if (a.rows <= 0) return;
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(a.rows), dim3(kDimrThreads), 0, s, a); };
  // 16-byte loads where every row of both matrices starts on 16 bytes
  const bool aligned = a.ld % 4 == 0 && ((uintptr_t)a.q | (uintptr_t)a.p) % 16 == 0;
  if (a.rows <= 256)
    aligned ? go(dimr_cost_kernel<true, 20, 8, 4, 1>) : go(dimr_cost_kernel<false, 20, 8, 4, 1>);
  else
    aligned ? go(dimr_cost_kernel<true, 8, 4, 2, 2>) : go(dimr_cost_kernel<false, 8, 4, 2, 2>);
}

}  // namespace via
