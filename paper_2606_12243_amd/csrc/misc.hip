// Small kernels of the verification step: embedding gather, the consumers
// of the split-K GEMM partials (residual + RMSNorm, SwiGLU, QKV RoPE + paged
// K/V write), the tier decision with its gate walk, and tree-path K/V
// compaction.
#include <algorithm>
#include <mutex>
#include <vector>

#include "kernels.h"

namespace via {

namespace {

// Split partials of two float4s (offsets o0 and o1): split_load16 issues
// the loads of splits 0..15 (past the last split it re-reads the last one:
// unconditional loads keep the code branch-free), split_reduce16 sums them
// in split order (the re-reads dropped by a select), and split_sum2 does
// both for splits sp0.. with 16 splits of loads in flight per round.
__device__ __forceinline__ void split_load16(const float* P, size_t stride, int ksplit, int sp0, size_t o0, size_t o1,
                                             float4 (&v0)[16], float4 (&v1)[16]) {
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const size_t base = (size_t)min(sp0 + q, ksplit - 1) * stride;
    v0[q] = *(const float4*)(P + base + o0);
    v1[q] = *(const float4*)(P + base + o1);
  }
}

__device__ __forceinline__ void split_reduce16(int ksplit, int sp0, const float4 (&v0)[16], const float4 (&v1)[16],
                                               float4& s0, float4& s1) {
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const bool ok = sp0 + q < ksplit;
    s0.x += ok ? v0[q].x : 0.f;
    s0.y += ok ? v0[q].y : 0.f;
    s0.z += ok ? v0[q].z : 0.f;
    s0.w += ok ? v0[q].w : 0.f;
    s1.x += ok ? v1[q].x : 0.f;
    s1.y += ok ? v1[q].y : 0.f;
    s1.z += ok ? v1[q].z : 0.f;
    s1.w += ok ? v1[q].w : 0.f;
  }
}

__device__ __forceinline__ void split_sum2(const float* P, size_t stride, int ksplit, int sp0, size_t o0, size_t o1,
                                           float4& s0, float4& s1) {
  for (int sp = sp0; sp < ksplit; sp += 16) {
    float4 v0[16], v1[16];
    split_load16(P, stride, ksplit, sp, o0, o1, v0, v1);
    split_reduce16(ksplit, sp, v0, v1, s0, s1);
  }
}

// Eight consecutive norm gains (the caller's pointer may have any alignment).
__device__ __forceinline__ void load_gain8(const uint16_t* g, float (&v)[8]) {
  if (((uintptr_t)g & 15) == 0) {  // uniform: k0 is a multiple of 8
    const uint4 w = *(const uint4*)g;
    const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[2 * e] = __uint_as_float(u[e] << 16);
      v[2 * e + 1] = __uint_as_float(u[e] & 0xFFFF0000u);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = bf2f(g[e]);
  }
}
__device__ __forceinline__ void load_gain8(const float* g, float (&v)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = g[e];
}

// Residual update and RMSNorm gain, elementwise: x = X[m] + sum_s P[s][m]
// (split order; P may be null), X[m] = x, and x * g is written as
// activation fragments (to fragment row rows[m].lm when `rows` is given;
// rows with lm < 0 only update X).  The RMSNorm scale 1/sqrt(mean(x^2)+eps)
// is a per-row factor that commutes with the next projection, so its
// consumer applies it (row_scale) after the GEMM; here each work-group adds
// the sum of x^2 over its kNormChunk columns to ss[chunk][out].
// Grid (ceil(d / kNormChunk), M), 64 threads of 8 columns each.  The partials,
// the row and the gains are loaded together: one wait for memory, not one each.
template <typename G, bool BF16, int NT, int KS>
__global__ __launch_bounds__(64) void resid_add_kernel(float* X, const float* P, int ksplit, int M, int d,
                                                       const G* g, void* Y, int MBn, const RowInfo* rows,
                                                       float* ss, int ss_stride, float* Xcopy, const G* E,
                                                       const RowInfo* erows) {
  const int m = blockIdx.y, chunk = blockIdx.x;
  const int k0 = chunk * kNormChunk + threadIdx.x * 8;
  const int out = rows ? rows[m].lm : m;
  float* x = X + (size_t)m * d;
  if (Xcopy) {  // uniform per work-group
    const int xr = erows ? erows[m].xs : m;
    Xcopy = xr < 0 ? nullptr : Xcopy + (size_t)xr * d;
  }
  const size_t stride = (size_t)M * d;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float sq = 0.f, gain[8];
  if (k0 < d && E) {
    // embedding rows: X[m] = E[tok]
    load_gain8(g + k0, gain);
    load_gain8(E + (size_t)erows[m].tok * d + k0, v);
    *(float4*)(x + k0) = make_float4(v[0], v[1], v[2], v[3]);
    *(float4*)(x + k0 + 4) = make_float4(v[4], v[5], v[6], v[7]);
    if (Xcopy) {
      *(float4*)(Xcopy + k0) = make_float4(v[0], v[1], v[2], v[3]);
      *(float4*)(Xcopy + k0 + 4) = make_float4(v[4], v[5], v[6], v[7]);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) sq += v[i] * v[i];
  } else if (k0 < d) {
    float4 acc[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)}, u[2];
    if constexpr (KS > 0) {
      // exactly KS splits: all loads in flight, then summed in split order
      float4 v0[KS], v1[KS];
      if (P) {
#pragma unroll
        for (int q = 0; q < KS; ++q) {
          v0[q] = *(const float4*)(P + (size_t)q * stride + (size_t)m * d + k0);
          v1[q] = *(const float4*)(P + (size_t)q * stride + (size_t)m * d + k0 + 4);
        }
      }
      u[0] = *(float4*)(x + k0);
      u[1] = *(float4*)(x + k0 + 4);
      load_gain8(g + k0, gain);
      if (P) {
#pragma unroll
        for (int q = 0; q < KS; ++q) {
          acc[0].x += v0[q].x;
          acc[0].y += v0[q].y;
          acc[0].z += v0[q].z;
          acc[0].w += v0[q].w;
          acc[1].x += v1[q].x;
          acc[1].y += v1[q].y;
          acc[1].z += v1[q].z;
          acc[1].w += v1[q].w;
        }
      }
    } else {
      if (P) split_sum2(P, stride, ksplit, 0, (size_t)m * d + k0, (size_t)m * d + k0 + 4, acc[0], acc[1]);
      u[0] = *(float4*)(x + k0);
      u[1] = *(float4*)(x + k0 + 4);
      load_gain8(g + k0, gain);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (P) {
        u[h].x = u[h].x + acc[h].x;
        u[h].y = u[h].y + acc[h].y;
        u[h].z = u[h].z + acc[h].z;
        u[h].w = u[h].w + acc[h].w;
        *(float4*)(x + k0 + 4 * h) = u[h];
      }
      if (Xcopy) *(float4*)(Xcopy + k0 + 4 * h) = u[h];
      v[4 * h + 0] = u[h].x;
      v[4 * h + 1] = u[h].y;
      v[4 * h + 2] = u[h].z;
      v[4 * h + 3] = u[h].w;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) sq += v[e] * v[e];
  }
  if (out < 0) return;  // uniform per work-group
  sq = wave_sum(sq);
  if (threadIdx.x == 0) ss[(size_t)chunk * ss_stride + out] = sq;
  if (k0 >= d) return;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = v[e] * gain[e];
  put_afrag<BF16, NT>(Y, out, k0, v, d >> 5, MBn);
}

// Many-row form of the residual update (one partial P, no head rows or
// embedding gather): a work-group of four waves owns one 16-row block of the
// fragment layout and one kNormChunk of columns.  Thread t of a wave takes row
// t % 16 and, in each of the wave's K32 steps s = wave + 4 i, the 8-column group
// t / 16, so every fragment store of a wave writes one contiguous 1 KB block
// (the one-row form writes 16 bytes every 256).  The values are those of
// resid_add_kernel: the 8-column group 4 s + t / 16 is that kernel's thread,
// and its partial sums of squares are added in that kernel's wave_sum order
// (two levels within the thread, two across waves, two across lanes).
template <int NT>
__global__ __launch_bounds__(256) void resid_add_rows_kernel(float* X, const float* P, int M, int d, const uint16_t* g,
                                                             void* Y, int MBn, float* ss, int ss_stride, float* Xcopy,
                                                             const RowInfo* erows) {
  constexpr int kPer = kNormChunk / 32 / 4;  // K32 steps of a wave
  static_assert(kPer == 4, "the sum order below is for 16 steps");
  __shared__ float part[4][64];
  const int chunk = blockIdx.x, w = threadIdx.x >> 6, t = threadIdx.x & 63, r = t & 15, j = t >> 4;
  const int m = blockIdx.y * 16 + r;
  const bool live = m < M;
  if (Xcopy && live) {
    const int xr = erows ? erows[m].xs : m;
    Xcopy = xr < 0 ? nullptr : Xcopy + (size_t)xr * d;
  }
  float p[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int k0 = chunk * kNormChunk + (w + 4 * i) * 32 + j * 8;
    p[i] = 0.f;
    if (!live || k0 >= d) continue;
    float* x = X + (size_t)m * d + k0;
    const float* a = P + (size_t)m * d + k0;
    const float4 b[2] = {*(const float4*)a, *(const float4*)(a + 4)};
    float v[8], gain[8];
    float4 xv[2] = {*(float4*)x, *(float4*)(x + 4)};
    load_gain8(g + k0, gain);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float4 u = xv[h];
      u.x = u.x + (0.f + b[h].x);
      u.y = u.y + (0.f + b[h].y);
      u.z = u.z + (0.f + b[h].z);
      u.w = u.w + (0.f + b[h].w);
      *(float4*)(x + 4 * h) = u;
      if (Xcopy) *(float4*)(Xcopy + k0 + 4 * h) = u;
      v[4 * h + 0] = u.x;
      v[4 * h + 1] = u.y;
      v[4 * h + 2] = u.z;
      v[4 * h + 3] = u.w;
    }
    float sq = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) sq += v[e] * v[e];
    p[i] = sq;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] * gain[e];
    put_afrag<true, NT>(Y, m, k0, v, d >> 5, MBn);
  }
  // wave_sum over the one-row form's threads T = 4 s + j: lane xor 32 and 16
  // pair steps s ^ 8 and s ^ 4 (this thread), xor 8 and 4 steps s ^ 2 and s ^ 1
  // (other waves), xor 2 and 1 groups j ^ 2 and j ^ 1 (lanes t ^ 32 and t ^ 16)
  part[w][t] = (p[0] + p[2]) + (p[1] + p[3]);
  __syncthreads();
  if (w != 0) return;
  float sq = (part[0][t] + part[2][t]) + (part[1][t] + part[3][t]);
  sq += __shfl_xor(sq, 32, 64);
  sq += __shfl_xor(sq, 16, 64);
  if (j == 0 && live) ss[(size_t)chunk * ss_stride + m] = sq;
}

// Rotate-half RoPE of the pair (j, j + hd/2) of head hh of row m (Q and K
// heads; V passes through) with the angle's cosine and sine, then the store:
// Q as bf16 hi/lo terms (fp32 models: fp32), K and V into the row's paged
// cache slot in the model dtype.
template <typename T>
__device__ __forceinline__ void qkv_store(const QkvArgs& a, const RowInfo& ri, int m, int hh, int j, float x1,
                                          float x2, double cs, double sn) {
  const int half = a.hd >> 1;
  float y1 = x1, y2 = x2;
  if (hh < a.H + a.KVH) {
    y1 = (float)((double)x1 * cs - (double)x2 * sn);
    y2 = (float)((double)x2 * cs + (double)x1 * sn);
  }
  if (hh < a.H) {
    const size_t o = ((size_t)m * a.H + hh) * a.hd + j;
    if constexpr (sizeof(T) == 2) {
      // Q as bf16 hi (truncated) + lo (rounded) terms for the attention MFMAs
      const uint32_t u1 = __float_as_uint(y1) >> 16, u2 = __float_as_uint(y2) >> 16;
      a.q_hi[o] = (uint16_t)u1;
      a.q_hi[o + half] = (uint16_t)u2;
      a.q_lo[o] = f2bf(y1 - __uint_as_float(u1 << 16));
      a.q_lo[o + half] = f2bf(y2 - __uint_as_float(u2 << 16));
    } else {
      float* q = (float*)a.q_hi;
      q[o] = y1;
      q[o + half] = y2;
    }
    return;
  }
  const int blk = ri.blk, t = ri.slot % kBlock;
  T* pool = (T*)a.pool;
  if (hh < a.H + a.KVH) {
    const int gk = hh - a.H;
    pool[k_off(a.layer_slot, blk, a.pool_blocks, a.KVH, a.hd, gk, t, j)] = from_f<T>(y1);
    pool[k_off(a.layer_slot, blk, a.pool_blocks, a.KVH, a.hd, gk, t, j + half)] = from_f<T>(y2);
  } else {
    const int gv = hh - a.H - a.KVH;
    pool[v_off(a.layer_slot, blk, a.pool_blocks, a.KVH, a.hd, gv, t, j)] = from_f<T>(y1);
    pool[v_off(a.layer_slot, blk, a.pool_blocks, a.KVH, a.hd, gv, t, j + half)] = from_f<T>(y2);
  }
}

// The rotation of pair j at position pos, pos * theta^(-2j/hd), in fp64.
__device__ __forceinline__ void rope_angle(int pos, int j, const QkvArgs& a, double* sn, double* cs) {
  sincos((double)pos * pow((double)a.theta, -2.0 * (double)j / (double)a.hd), sn, cs);
}

// QKV partial sums -> RMSNorm scale of the input row -> rotate-half RoPE at
// the row's position -> Q (bf16 hi/lo terms, or fp32) and paged K/V (model
// dtype).  A work-group of 256 threads takes four (row, head of Q, K or V)
// pairs, 64 threads each; thread j owns the rotation pair (j, j + hd/2), whose
// rotation it computes while the loads of the KS split partials are outstanding
// (8B, 32 rows: 5.2 us; reading it from a table 5.4).  KS = 0: the split count is
// taken from the arguments.
template <typename T, int KS>
__global__ __launch_bounds__(256) void qkv_finish_kernel(QkvArgs a) {
  const int m = blockIdx.x, hh = blockIdx.y * 4 + (threadIdx.x >> 6), j = threadIdx.x & 63;
  const int half = a.hd >> 1;
  if (j >= half || hh >= a.H + 2 * a.KVH) return;
  const size_t N = (size_t)(a.H + 2 * a.KVH) * a.hd, stride = (size_t)a.M * N;
  const size_t c = (size_t)m * N + (size_t)hh * a.hd + j;
  float x1 = 0.f, x2 = 0.f;
  double2 cs_sn = make_double2(1.0, 0.0);
  const RowInfo ri = a.rows[m];
  auto rotation = [&] {
    if (hh < a.H + a.KVH) rope_angle(ri.pos, j, a, &cs_sn.y, &cs_sn.x);  // V passes through
  };
  if constexpr (KS > 0) {
    float v1[KS], v2[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      v1[q] = a.P[(size_t)q * stride + c];
      v2[q] = a.P[(size_t)q * stride + c + half];
    }
    rotation();
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      x1 += v1[q];
      x2 += v2[q];
    }
  } else {
    rotation();
    for (int q = 0; q < a.ksplit; ++q) {
      x1 += a.P[(size_t)q * stride + c];
      x2 += a.P[(size_t)q * stride + c + half];
    }
  }
  const float sc = row_scale(a.ss, a.ss_stride, m, a.d, a.eps);  // RMSNorm of the input row
  qkv_store<T>(a, ri, m, hh, j, x1 * sc, x2 * sc, cs_sn.x, cs_sn.y);
}

// Rotations of the rows of a forward, computed once for all its layers: grid
// (M), one thread per pair.
__global__ __launch_bounds__(64) void rope_table_kernel(QkvArgs a) {
  const int m = blockIdx.x, j = threadIdx.x, half = a.hd >> 1;
  if (j >= half) return;
  double2 cs_sn;
  rope_angle(a.rows[m].pos, j, a, &cs_sn.y, &cs_sn.x);
  a.rope[(size_t)m * half + j] = cs_sn;
}

// The QKV finish with the rotations read from that table.  A work-group takes 16 consecutive rows and
// one KV head's share of them, its G query heads, its K head and its V head (or,
// where that leaves compute units idle, some of them).  Thread t holds row t / 16
// and the 8 dims from (t % 16) * 8 (hd 64: two heads' worth at a time), so the
// partials are read 32 bytes a thread, a pass ahead of their use; the
// rotations, the same for every head, stay in registers, and the rotation's
// other half comes from the lane hd / 16 away; Q terms and K go out 16 bytes a
// thread.  V, transposed in its pages, goes through LDS: 16 lanes then write 16
// tokens of one dim next to each other, where a row per work-group left every V
// page's 32-byte pieces to 16 work-groups on 8 XCDs (8B, 8188 rows: 134 us).
template <typename T, int HD, int KS>
__global__ __launch_bounds__(256) void qkv_finish_tile_kernel(QkvArgs a) {
  constexpr int TPH = HD / 8, HPP = 16 / TPH;  // threads of a row per head; heads per pass
  const int r = threadIdx.x >> 4, l = threadIdx.x & 15, sub = l / TPH, d0 = (l % TPH) * 8, half = HD / 2;
  const int m = blockIdx.x * 16 + r, g = blockIdx.y, G = a.H / a.KVH;
  const bool live = m < a.M;
  const int mm = live ? m : a.M - 1;  // rows past the end repeat the last one and store nothing
  const size_t N = (size_t)(a.H + 2 * a.KVH) * HD, stride = (size_t)a.M * N;
  __shared__ float vt[HD][17];
  // heads of this work-group: 0 .. G - 1 its queries, G the K head, G + 1 the V head
  auto head = [&](int h) { return h < G ? g * G + h : h == G ? a.H + g : a.H + a.KVH + g; };
  float4 v[KS][2];
  auto load = [&](int h0) {
    const float* p = a.P + (size_t)mm * N + (size_t)head(min(h0 + sub, G + 1)) * HD + d0;
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      v[q][0] = *(const float4*)(p + q * stride);
      v[q][1] = *(const float4*)(p + q * stride + 4);
    }
  };
  load(blockIdx.z * HPP);
  double2 rot[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) rot[e] = a.rope[(size_t)mm * half + d0 % half + e];
  const RowInfo ri = a.rows[mm];
  const int blk = ri.blk, t = ri.slot % kBlock;
  const float sc = row_scale(a.ss, a.ss_stride, mm, a.d, a.eps);  // RMSNorm of the input row
  const bool first = d0 < half;
  for (int h0 = blockIdx.z * HPP; h0 < G + 2; h0 += gridDim.z * HPP) {
    const int h = h0 + sub, hh = head(min(h, G + 1));
    float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      x[0] += v[q][0].x;
      x[1] += v[q][0].y;
      x[2] += v[q][0].z;
      x[3] += v[q][0].w;
      x[4] += v[q][1].x;
      x[5] += v[q][1].y;
      x[6] += v[q][1].z;
      x[7] += v[q][1].w;
    }
    if (h0 + (int)gridDim.z * HPP < G + 2) load(h0 + gridDim.z * HPP);
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      x[e] *= sc;
      const float o = __shfl_xor(x[e], TPH / 2, 64);  // the pair's other half
      const double x1 = first ? x[e] : o, x2 = first ? o : x[e];
      const float ro = first ? (float)(x1 * rot[e].x - x2 * rot[e].y) : (float)(x2 * rot[e].x + x1 * rot[e].y);
      y[e] = h <= G ? ro : x[e];  // V passes through
    }
    if (live && h < G) {
      const size_t o = ((size_t)m * a.H + hh) * HD + d0;
      if constexpr (sizeof(T) == 2) {
        // bf16 hi (truncated) + lo (rounded) terms for the attention MFMAs
        uint32_t hw[4], lw[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t u0 = __float_as_uint(y[2 * e]) >> 16, u1 = __float_as_uint(y[2 * e + 1]) >> 16;
          hw[e] = pack_bf16x2(u0, u1);
          lw[e] = pack_bf16x2(f2bf(y[2 * e] - __uint_as_float(u0 << 16)), f2bf(y[2 * e + 1] - __uint_as_float(u1 << 16)));
        }
        *(uint4*)(a.q_hi + o) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
        *(uint4*)(a.q_lo + o) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
      } else {
        float* q = (float*)a.q_hi + o;
        *(float4*)q = make_float4(y[0], y[1], y[2], y[3]);
        *(float4*)(q + 4) = make_float4(y[4], y[5], y[6], y[7]);
      }
    } else if (live && h == G) {
      T* kp = (T*)a.pool + k_off(a.layer_slot, blk, a.pool_blocks, a.KVH, HD, g, t, d0);
      if constexpr (sizeof(T) == 2) {
        *(uint4*)kp = make_uint4(pack_bf16x2(f2bf(y[0]), f2bf(y[1])), pack_bf16x2(f2bf(y[2]), f2bf(y[3])),
                                 pack_bf16x2(f2bf(y[4]), f2bf(y[5])), pack_bf16x2(f2bf(y[6]), f2bf(y[7])));
      } else {
        *(float4*)kp = make_float4(y[0], y[1], y[2], y[3]);
        *(float4*)(kp + 4) = make_float4(y[4], y[5], y[6], y[7]);
      }
    }
    if (h0 <= G + 1 && G + 1 < h0 + HPP) {  // uniform: this pass holds the V head
      if (h == G + 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) vt[d0 + e][r] = y[e];
      }
      __syncthreads();
      // lane -> token threadIdx.x % 16, dims threadIdx.x / 16, + 16, ...
      const int vr = threadIdx.x & 15, vm = blockIdx.x * 16 + vr;
      if (vm < a.M) {
        const RowInfo vi = a.rows[vm];
        T* vp = (T*)a.pool + v_off(a.layer_slot, vi.blk, a.pool_blocks, a.KVH, HD, g, vi.slot % kBlock, 0);
        for (int d = threadIdx.x >> 4; d < HD; d += 16) vp[(size_t)d * kBlock] = from_f<T>(vt[d][vr]);
      }
    }
  }
}

// Tier decision and gate walk for one sequence (App. B.1), one wave: lane j
// holds draft j (at most 64) with everything the walk may ask of it, loaded at
// once; the walk itself is wave-uniform, on ballots over the lanes and single
// lanes' values, so it waits for memory once and not at every node.
__global__ __launch_bounds__(64) void decide_kernel(DecideArgs a) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const StepSeq ss = a.seqs[b];
  const int D = a.max_drafts, B = a.batch;
  const int base = b * D;
  const bool have_full = a.f_row_max != nullptr && ss.full_ran;
  const bool live = lane < ss.n_drafts;
  int out = 0, parent = -2, tok = -1, s_arg = 0, f_arg = 0, tier = -1;
  float conf = 0.f, f_max = 0.f;
  if (live) {
    out = b * a.max_rows + a.draft_row[base + lane];
    parent = a.draft_parent[base + lane];
    tok = a.draft_tok[base + lane];
    s_arg = a.s_row_argmax[out];
    if (have_full) {
      f_max = a.f_row_max[out];
      f_arg = a.f_row_argmax[out];
    }
    conf = expf((a.s_draft_logit[base + lane] - a.s_row_max[out]) * a.inv_T);
    if (a.forced >= 0)
      tier = a.forced;
    else if (conf >= a.tau_acc)
      tier = 0;
    else if (conf >= a.tau_full)
      tier = 1;
    else
      tier = 2;  // also a NaN confidence
    a.conf[base + lane] = conf;
    a.tier[base + lane] = (int8_t)tier;
  }
  int* status = a.packed;
  int* kappa = a.packed + B;
  int* emit = a.packed + 2 * B;
  int* new_len = a.packed + 3 * B;
  int* path = a.packed + 4 * B + base;
  if (a.draft_probs) {
    // sampling rules (App. A), chain drafts in order: an accept-tier draft is
    // kept; a slim-tier position owes a sample of q'; an escalated draft x is
    // kept with probability min(1, q(x) / ((1 - alpha) p(x))) (Eq. A.2),
    // accepted iff its uniform is below that, else it owes a sample of the
    // A.3 residual.  The owed sample is drawn by the sampling kernels.
    bool keep = tier == 0, finite = true;
    if (tier == 2 && have_full) {
      finite = isfinite(f_max);
      if (finite) {
        const float qx = expf((a.f_draft_logit[base + lane] - f_max) * a.inv_T) / a.f_row_sumexp[out];
        const float px = a.draft_probs[(size_t)(base + lane) * a.vocab + tok];
        const float pk = px <= 0.f ? 1.f : fminf(1.f, qx / ((1.f - a.alpha) * px));
        keep = a.u[(size_t)(base + lane) * 3] < pk;
      }
    }
    const unsigned long long stop = __ballot(live && !keep);
    const int k = stop ? __ffsll((long long)stop) - 1 : ss.n_drafts;  // the first draft not kept
    for (int q = lane; q < D; q += 64) path[q] = q < k ? q : -1;
    if (lane != (stop ? k : 0)) return;
    SampleReq rq{0, 0, 0, 0.f};
    int st = 0;
    if (stop) {
      if (tier == 1)
        rq = SampleReq{1, out, k, a.u[(size_t)(base + k) * 3 + 1]};
      else if (!have_full)
        st = 1;
      else if (!finite)
        st = 2;
      else
        rq = SampleReq{2, out, k, a.u[(size_t)(base + k) * 3 + 2]};
    }
    a.req[b] = rq;
    status[b] = st;
    kappa[b] = k;
    emit[b] = -1;  // a sample owed is written by sample_pick_kernel
    new_len[b] = st == 2 ? ss.n : ss.n + k + (rq.kind ? 1 : 0);
    return;
  }
  // value v of draft j (wave-uniform)
  auto of = [](int v, int j) { return __builtin_amdgcn_readlane(v, j); };
  auto off = [](float v, int j) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j)); };
  int u = -1, k = 0, em = -1, st = 0, step = -1;  // lane i keeps path entry i in `step`
  for (;;) {
    const unsigned long long kids = __ballot(live && parent == u);  // children of u, in draft order
    if (!kids) break;                                               // leaf: whole path accepted, no emit
    const int first = __ffsll((long long)kids) - 1;
    int take = -1;
    float best = 0.f;
    for (unsigned long long acc = __ballot(live && parent == u && tier == 0); acc; acc &= acc - 1) {
      const int j = __ffsll((long long)acc) - 1;
      const float c = off(conf, j);
      if (take < 0 || c > best) {
        take = j;
        best = c;
      }
    }
    if (take < 0) {
      if (__ballot(live && parent == u && tier == 1)) {
        em = of(s_arg, first);
        break;
      }
      if (!have_full) {
        st = 1;
        break;
      }
      if (!isfinite(off(f_max, first))) {  // non-finite logits of q
        st = 2;
        break;
      }
      const int gtok = of(f_arg, first);
      const unsigned long long hit = __ballot(live && parent == u && tok == gtok);
      if (!hit) {
        em = gtok;
        break;
      }
      take = __ffsll((long long)hit) - 1;
    }
    if (lane == k) step = take;
    ++k;
    u = take;
  }
  const int ev = st == 0 ? em : -1;
  const int nv = st == 2 ? ss.n : ss.n + k + (st == 0 && em >= 0 ? 1 : 0);
  // the host mirror is written past the caches, so that it is in host memory
  // once the stream has been synchronised
  auto put = [&](int i, int v) {
    a.packed[i] = v;
    if (a.h_packed) __hip_atomic_store(a.h_packed + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  };
  if (lane < 4) put(lane * B + b, lane == 0 ? st : lane == 1 ? k : lane == 2 ? ev : nv);
  for (int q = lane; q < D; q += 64) put(4 * B + base + q, q < k ? step : -1);
}

// Tree compaction: copy the K/V of slot src to slot dst in every layer slot.
template <typename T>
__global__ __launch_bounds__(128) void kv_move_kernel(T* pool, int nblk, int KVH, int hd, const int32_t* btab,
                                                      const KvMove* moves, int n_moves) {
  const int l = blockIdx.y;  // layer slot
  for (int mv = 0; mv < n_moves; ++mv) {  // in order: destinations never overtake later sources
    const KvMove m = moves[mv];
    int sb = btab[m.bt + m.src / kBlock], st = m.src % kBlock;
    int db = btab[m.bt + m.dst / kBlock], dt = m.dst % kBlock;
    for (int e = threadIdx.x; e < KVH * hd; e += 128) {
      int g = e / hd, i = e % hd;
      pool[k_off(l, db, nblk, KVH, hd, g, dt, i)] = pool[k_off(l, sb, nblk, KVH, hd, g, st, i)];
      pool[v_off(l, db, nblk, KVH, hd, g, dt, i)] = pool[v_off(l, sb, nblk, KVH, hd, g, st, i)];
    }
    __syncthreads();
  }
}

}  // namespace

void launch_resid_add(bool bf16, float* X, const float* P, int ksplit, int M, int d, const void* g, void* Y, int MBn,
                      const RowInfo* rows, float* ss, int ss_stride, hipStream_t s, float* Xcopy, const void* E,
                      const RowInfo* erows) {
  const dim3 grid((d + kNormChunk - 1) / kNormChunk, M);
  if (bf16 && P && !rows && !E && M > kManyRows && ksplit == 1) {
    const dim3 rgrid((d + kNormChunk - 1) / kNormChunk, (M + 15) / 16);
    hipLaunchKernelGGL(resid_add_rows_kernel<kTerms>, rgrid, dim3(256), 0, s, X, P, M, d, (const uint16_t*)g, Y, MBn, ss,
                       ss_stride, Xcopy, erows);
    return;
  }
  if (!bf16) {  // one partial
    hipLaunchKernelGGL((resid_add_kernel<float, false, 1, 1>), grid, dim3(64), 0, s, X, P, ksplit, M, d,
                       (const float*)g, Y, MBn, rows, ss, ss_stride, Xcopy, (const float*)E, erows);
    return;
  }
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(64), 0, s, X, P, ksplit, M, d, (const uint16_t*)g, Y, MBn, rows, ss,
                       ss_stride, Xcopy, (const uint16_t*)E, erows);
  };
  // the split counts of the projections that feed it get their exact loads
  switch (P ? ksplit : 1) {
    case 1: go(resid_add_kernel<uint16_t, true, kTerms, 1>); break;
    case 2: go(resid_add_kernel<uint16_t, true, kTerms, 2>); break;
    case 4: go(resid_add_kernel<uint16_t, true, kTerms, 4>); break;
    case 8: go(resid_add_kernel<uint16_t, true, kTerms, 8>); break;
    default: go(resid_add_kernel<uint16_t, true, kTerms, 0>); break;
  }
}

void launch_rope_table(const QkvArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(rope_table_kernel, dim3(a.M), dim3(64), 0, s, a);
}

void launch_qkv_finish(bool bf16, const QkvArgs& a, hipStream_t s) {
  if (qkv_rope_table(a) && (a.ksplit == 1 || a.ksplit == 2 || a.ksplit == 4 || a.ksplit == 8)) {
    const int tiles = (a.M + 15) / 16, heads = a.H / a.KVH + 2, passes = a.hd == 128 ? heads : (heads + 1) / 2;
    const dim3 grid(tiles, a.KVH, std::min(passes, (256 + tiles * a.KVH - 1) / (tiles * a.KVH)));
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a); };
    auto by_size = [&](auto k128, auto k64) { a.hd == 128 ? go(k128) : go(k64); };
    if (!bf16)  // one partial
      by_size(qkv_finish_tile_kernel<float, 128, 1>, qkv_finish_tile_kernel<float, 64, 1>);
    else if (a.ksplit == 1)
      by_size(qkv_finish_tile_kernel<uint16_t, 128, 1>, qkv_finish_tile_kernel<uint16_t, 64, 1>);
    else if (a.ksplit == 2)
      by_size(qkv_finish_tile_kernel<uint16_t, 128, 2>, qkv_finish_tile_kernel<uint16_t, 64, 2>);
    else if (a.ksplit == 4)
      by_size(qkv_finish_tile_kernel<uint16_t, 128, 4>, qkv_finish_tile_kernel<uint16_t, 64, 4>);
    else
      by_size(qkv_finish_tile_kernel<uint16_t, 128, 8>, qkv_finish_tile_kernel<uint16_t, 64, 8>);
    return;
  }
  const dim3 grid(a.M, (a.H + 2 * a.KVH + 3) / 4);
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a); };
  if (bf16) {
    switch (a.ksplit) {
      case 1: go(qkv_finish_kernel<uint16_t, 1>); break;
      case 2: go(qkv_finish_kernel<uint16_t, 2>); break;
      case 4: go(qkv_finish_kernel<uint16_t, 4>); break;
      case 8: go(qkv_finish_kernel<uint16_t, 8>); break;
      default: go(qkv_finish_kernel<uint16_t, 0>); break;
    }
  } else {
    go(qkv_finish_kernel<float, 1>);
  }
}

namespace {

// Owed samples (App. A): the token a uniform u draws from weights w(v),
// v < V, is the first v in id order whose running sum exceeds u * sum(w)
// (the last token with weight when rounding leaves no crossing).  Weights:
// kind 1 the slim row's exp((l - max) / T); kind 2 the A.3 residual
// max(0, q / beta - p), q = exp((l - max) / T) / sum, or q itself when the
// residual has no mass.
//
// The vocabulary is cut into slices of kSampleThreads * E ids; thread t of a
// slice owns the E consecutive ids starting at t * E.  Sums are fp64 in one
// fixed grouping, shared by both kernels: a thread's ids in order; four
// consecutive threads in order per lane of wave 0; a 64-lane inclusive scan.
// sample_sums_kernel (one work-group per slice and sequence) writes each
// slice's residual and q sums; sample_pick_kernel (one per sequence) finds
// the crossing slice from them, rescans that slice with the same grouping,
// and walks the crossing lane, thread and id.
constexpr int kSampleThreads = 256;

struct SampleGeom {
  int E, slice, G;
};
__host__ __device__ inline SampleGeom sample_geom(int V) {
  int E = (V + kSampleSlices * kSampleThreads - 1) / (kSampleSlices * kSampleThreads);
  if (E < 1) E = 1;
  const int slice = E * kSampleThreads;
  return SampleGeom{E, slice, (V + slice - 1) / slice};
}

struct SampleRow {
  const float* lg;
  const float* p;
  float mx, inv_z, inv_T, inv_beta;
};
__device__ inline SampleRow sample_row(const DecideArgs& a, const SampleReq& r, int b) {
  const size_t V = (size_t)a.vocab;
  SampleRow w;
  w.lg = (r.kind == 1 ? a.s_logits : a.f_logits) + (size_t)r.out * V;
  w.p = a.draft_probs + (size_t)(b * a.max_drafts + r.j) * V;
  w.mx = r.kind == 1 ? a.s_row_max[r.out] : a.f_row_max[r.out];
  w.inv_z = r.kind == 2 ? 1.f / a.f_row_sumexp[r.out] : 1.f;
  w.inv_T = a.inv_T;
  w.inv_beta = 1.f / a.beta;
  return w;
}
// Inclusive scan of one fp64 value over the 64 lanes of a wave.
__device__ inline double wave_scan(double x, int lane) {
  for (int d = 1; d < 64; d <<= 1) {
    const double y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  return x;
}

// Weights of a slice's ids, eight a thread at a time (row stride 9: no bank
// conflicts): q, and for kind 2 the residual weight r.
struct SliceWeights {
  float q[kSampleThreads * 9], r[kSampleThreads * 9];
};
__device__ inline float q_weight(const SampleRow& w, float x) { return expf((x - w.mx) * w.inv_T) * w.inv_z; }
__device__ inline float r_weight(const SampleRow& w, float q, float p) { return fmaxf(0.f, q * w.inv_beta - p); }

// Thread sums of one slice (both weight kinds) into LDS; with probs, also the
// ids' probabilities, weight * inv_sum, to probs[v].  Thread t sums the ids
// [t * E, t * E + E) in order, but the work-group reads and weighs them side by
// side: thread by thread the eight loads and stores of a wave went to 64 cache
// lines each (sums and probabilities of 16 rows of 128256 ids: 12.3 -> 6.6 us,
// 3.2 us of it the bytes at the copy rate).
// Leaves the last eight ids a thread (all of them if E <= 8) in sw.
__device__ inline void slice_thread_sums(const SampleRow& w, int kind, int V, const SampleGeom& g, int slice_id,
                                         SliceWeights& sw, double* tq, double* tr, float* probs = nullptr,
                                         float inv_sum = 0.f) {
  const int t = threadIdx.x;
  const int id = t & 7, lo = slice_id * g.slice + (t >> 3) * g.E + id;
  double sq = 0.0, sr = 0.0;
  for (int e = 0; e < g.E; e += 8) {
    float x[8], p[8];
    bool in[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int v = lo + i * (kSampleThreads / 8) * g.E + e;
      in[i] = id + e < g.E && v < V;
      x[i] = in[i] ? w.lg[v] : 0.f;
      if (kind == 2) p[i] = in[i] ? w.p[v] : 0.f;
    }
    if (e) __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float q = in[i] ? q_weight(w, x[i]) : 0.f;
      const int o = (i * (kSampleThreads / 8) + (t >> 3)) * 9 + id;
      sw.q[o] = q;
      if (kind == 2) sw.r[o] = in[i] ? r_weight(w, q, p[i]) : 0.f;
      if (probs && in[i]) probs[lo + i * (kSampleThreads / 8) * g.E + e] = q * inv_sum;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      sq += (double)sw.q[t * 9 + i];
      if (kind == 2) sr += (double)sw.r[t * 9 + i];
    }
  }
  tq[t] = sq;
  tr[t] = sr;
}

// Lane sums (four threads in order) and their inclusive scan, wave 0.
__device__ inline double lane_scan(const double* ts, int lane, double* lane_sum) {
  const double x = ((ts[4 * lane] + ts[4 * lane + 1]) + ts[4 * lane + 2]) + ts[4 * lane + 3];
  *lane_sum = x;
  return wave_scan(x, lane);
}

// Requests: in device memory, or (kStaticSampleRows at most) in the kernel's arguments.
struct ReqArray {
  const SampleReq* r;
};
struct ReqArgs {
  SampleReq r[kStaticSampleRows];
};

// Slice sums of every request; with probs, also request b's softmax
// exp((l - max) / T) / sum as probs[b * ld + v], from the same loads.
template <typename R>
__global__ __launch_bounds__(kSampleThreads) void sample_sums_kernel(DecideArgs a, R req, float* probs, int ld) {
  const int b = blockIdx.y, g = blockIdx.x;
  const SampleReq r = req.r[b];
  if (r.kind == 0) return;  // uniform per work-group
  const SampleGeom geo = sample_geom(a.vocab);
  __shared__ double tq[kSampleThreads], tr[kSampleThreads];
  __shared__ SliceWeights sw;
  const SampleRow w = sample_row(a, r, b);
  if (probs)
    slice_thread_sums(w, r.kind, a.vocab, geo, g, sw, tq, tr, probs + (size_t)b * ld, 1.f / a.s_row_sumexp[r.out]);
  else
    slice_thread_sums(w, r.kind, a.vocab, geo, g, sw, tq, tr);
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  double ls;
  const double iq = lane_scan(tq, lane, &ls);
  const double ir = lane_scan(tr, lane, &ls);
  if (lane == 63) {
    double* out = a.slice_sum + ((size_t)b * kSampleSlices + g) * 2;
    out[0] = iq;
    out[1] = ir;
  }
}

template <typename R>
__global__ __launch_bounds__(kSampleThreads) void sample_pick_kernel(DecideArgs a, R req) {
  const int b = blockIdx.x;
  const SampleReq r = req.r[b];
  if (r.kind == 0) return;  // uniform per work-group
  const int V = a.vocab;
  const SampleGeom geo = sample_geom(V);
  const SampleRow w = sample_row(a, r, b);
  const int t = threadIdx.x, lane = t & 63;
  __shared__ double tq[kSampleThreads], tr[kSampleThreads];
  __shared__ SliceWeights sw;
  __shared__ int s_slice, s_last, s_resid;
  __shared__ double s_acc, s_target;
  if (t < 64) {
    // slice level: totals, the weights in use, the crossing slice
    const double* ssum = a.slice_sum + (size_t)b * kSampleSlices * 2;
    const double xq = lane < geo.G ? ssum[lane * 2] : 0.0, xr = lane < geo.G ? ssum[lane * 2 + 1] : 0.0;
    const double iq = wave_scan(xq, lane), ir = wave_scan(xr, lane);
    const double tot_r = __shfl(ir, 63, 64);
    const bool resid = r.kind == 2 && tot_r > 0.0;
    const double x = resid ? xr : xq, inc = resid ? ir : iq;
    const double tot = __shfl(inc, 63, 64);
    const double target = (double)r.u * tot;
    // crossings only at slices with weight (sums of zeros may round apart)
    const unsigned long long cross = __ballot(lane < geo.G && x > 0.0 && inc > target);
    const unsigned long long pos = __ballot(x > 0.0);
    if (lane == 0) {
      int c, last = 0;
      if (cross) {
        c = __ffsll((long long)cross) - 1;
      } else {
        c = pos ? 63 - __clzll((long long)pos) : 0;
        last = 1;
      }
      s_slice = c;
      s_last = last;
      s_resid = resid ? 1 : 0;
      s_target = target;
    }
    // running sum before the crossing slice: the previous lane's prefix
    const int c = cross ? __ffsll((long long)cross) - 1 : 0;
    const double before = __shfl(inc, c > 0 ? c - 1 : 0, 64);
    if (lane == 0) s_acc = c > 0 ? before : 0.0;
  }
  __syncthreads();
  const int c = s_slice;
  const bool resid = s_resid != 0;
  slice_thread_sums(w, resid ? 2 : 1, V, geo, c, sw, tq, tr);
  __syncthreads();
  if (t >= 64) return;
  const double* ts = resid ? tr : tq;
  double ls;
  const double inc = lane_scan(ts, lane, &ls);
  const double target = s_target;
  const double run0 = s_acc;
  bool last = s_last != 0;
  unsigned long long cross = last ? 0ull : __ballot(ls > 0.0 && run0 + inc > target);
  if (!cross) last = true;
  const unsigned long long pos = __ballot(ls > 0.0);
  int L;
  if (!last)
    L = __ffsll((long long)cross) - 1;
  else
    L = pos ? 63 - __clzll((long long)pos) : 0;
  if (lane != L) return;
  // the chosen lane: its four threads in order, then the chosen thread's ids
  double run = run0 + (inc - ls);
  int th = -1;
  if (!last) {
    for (int i = 0; i < 4; ++i) {
      const double v = ts[4 * L + i];
      if (v > 0.0 && run + v > target) {
        th = 4 * L + i;
        break;
      }
      run += v;
    }
  }
  bool take_last = th < 0;
  if (take_last) {
    th = 4 * L;
    for (int i = 3; i >= 0; --i)
      if (ts[4 * L + i] > 0.0) {
        th = 4 * L + i;
        break;
      }
  }
  const int lo = c * geo.slice + th * geo.E, hi = min(lo + geo.E, V);
  const float* wts = (resid ? sw.r : sw.q) + th * 9;  // these ids' weights, if E <= 8
  int tok = -1, lastpos = lo < V ? lo : V - 1;
  for (int v = lo; v < hi; ++v) {
    float wt;
    if (geo.E <= 8) {
      wt = wts[v - lo];
    } else {
      wt = q_weight(w, w.lg[v]);
      if (resid) wt = r_weight(w, wt, w.p[v]);
    }
    if (wt > 0.f) {
      lastpos = v;
      run += (double)wt;
      if (!take_last && run > target) {
        tok = v;
        break;
      }
    }
  }
  const int drawn = tok >= 0 ? tok : lastpos;
  if (a.tok_out)
    a.tok_out[b] = drawn;
  else
    a.packed[2 * a.batch + b] = drawn;
}

}  // namespace

template <typename R>
static void launch_draws(const DecideArgs& a, const R& req, float* probs, int probs_ld, hipStream_t s) {
  const SampleGeom g = sample_geom(a.vocab);
  hipLaunchKernelGGL(sample_sums_kernel<R>, dim3(g.G, a.batch), dim3(kSampleThreads), 0, s, a, req, probs, probs_ld);
  hipLaunchKernelGGL(sample_pick_kernel<R>, dim3(a.batch), dim3(kSampleThreads), 0, s, a, req);
}

void launch_decide(const DecideArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(decide_kernel, dim3(a.batch), dim3(64), 0, s, a);
  if (a.draft_probs) launch_draws(a, ReqArray{a.req}, nullptr, 0, s);
}

// Probabilities that may lie over the logits (n_logits floats) go out after
// the pick has read those; otherwise with the sums, which saves a launch.
template <typename R>
static void launch_rows(const DecideArgs& a, const R& req, size_t n_logits, float* probs, int probs_ld, hipStream_t s) {
  const uintptr_t p = (uintptr_t)probs, l = (uintptr_t)a.s_logits;
  const bool over = probs && p < l + n_logits * 4 && l < p + ((size_t)(a.batch - 1) * probs_ld + a.vocab) * 4;
  launch_draws(a, req, over ? nullptr : probs, probs_ld, s);
  if (!over) return;
  const SampleGeom g = sample_geom(a.vocab);
  hipLaunchKernelGGL(sample_sums_kernel<R>, dim3(g.G, a.batch), dim3(kSampleThreads), 0, s, a, req, probs, probs_ld);
}

void launch_sample_rows(const DecideArgs& a, int out_rows, float* probs, int probs_ld, hipStream_t s) {
  launch_rows(a, ReqArray{a.req}, (size_t)out_rows * a.vocab, probs, probs_ld, s);
}

// ---------------------------------------------------------------- draws without allocation
// Scratch of the draw entry point that allocates nothing (via_sample_rows_static):
// the per-slice sums [request][slice][2] (the requests are kernel arguments).
// Each GPU holds its own copy until the process ends; every call on a GPU reuses it.
namespace {
constexpr size_t kStaticScratchBytes = (size_t)kStaticSampleRows * kSampleSlices * 2 * sizeof(double);
static_assert(kStaticScratchBytes == 65536, "the size include/via.h states");
static __device__ __align__(256) char scratch[kStaticScratchBytes];
}  // namespace

hipError_t static_scratch(void** ptr, size_t* bytes) {
  // the array's device address, looked up once per device with that device current
  static std::mutex mu;
  static std::vector<void*> addr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  if ((size_t)dev >= addr.size()) addr.resize(dev + 1, nullptr);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  *bytes = kStaticScratchBytes;
  return hipSuccess;
}

void launch_sample_rows_static(DecideArgs a, int out_rows, const SampleReq* req, int n, void* scratch_ptr,
                               float* probs, int probs_ld, hipStream_t s) {
  ReqArgs q{};
  for (int i = 0; i < n; ++i) q.r[i] = req[i];
  a.slice_sum = (double*)scratch_ptr;
  a.batch = n;
  launch_rows(a, q, (size_t)out_rows * a.vocab, probs, probs_ld, s);
}

void launch_kv_moves(bool bf16, void* pool, int pool_blocks, int n_slots, int KVH, int hd, const int32_t* btab,
                     const KvMove* moves, int n_moves, hipStream_t s) {
  if (n_moves <= 0) return;
  if (bf16)
    hipLaunchKernelGGL(kv_move_kernel<uint16_t>, dim3(1, n_slots), dim3(128), 0, s, (uint16_t*)pool, pool_blocks,
                       KVH, hd, btab, moves, n_moves);
  else
    hipLaunchKernelGGL(kv_move_kernel<float>, dim3(1, n_slots), dim3(128), 0, s, (float*)pool, pool_blocks, KVH,
                       hd, btab, moves, n_moves);
}


namespace {

// Forward that starts after the layers the two routes share (route layer
// i == i for i < a.P): grid (M, P + 1).  y < P: the row's K and V of layer
// y, copied from the source cache (slot y) to the destination cache (slot y)
// at the row's position; y == P: the row's residual stream after layer
// P - 1.  A verify step's full forward copies slim -> full and takes the
// state from the state ring (saved there by the slim forward that fed the
// slot: this step's for window rows, an earlier one for lag rows); a
// prefill's slim forward copies full -> slim and takes the state its full
// forward saved for the same rows.
template <typename T>
__global__ __launch_bounds__(256) void prefix_copy_kernel(PrefixArgs a) {
  const int m = blockIdx.x, y = blockIdx.y;
  const PrefixXfer x = a.xfer[m];
  if (y == a.P) {
    const float* src = a.xstate + (size_t)x.src_row * a.d;
    float* dst = a.X + (size_t)m * a.d;
    for (int i = threadIdx.x; i < a.d; i += 256) dst[i] = src[i];
    return;
  }
  const T* sp = (const T*)a.src_pool;
  T* dp = (T*)a.dst_pool;
  const int n = a.KVH * a.hd;
  for (int e = threadIdx.x; e < 2 * n; e += 256) {
    const int g = (e % n) / a.hd, i = e % a.hd;
    if (e < n)
      dp[k_off(y, x.dst_blk, a.dst_blocks, a.KVH, a.hd, g, x.t, i)] =
          sp[k_off(y, x.src_blk, a.src_blocks, a.KVH, a.hd, g, x.t, i)];
    else
      dp[v_off(y, x.dst_blk, a.dst_blocks, a.KVH, a.hd, g, x.t, i)] =
          sp[v_off(y, x.src_blk, a.src_blocks, a.KVH, a.hd, g, x.t, i)];
  }
}

}  // namespace

void launch_prefix_copy(bool bf16, const PrefixArgs& a, hipStream_t s) {
  const dim3 grid(a.M, a.P + 1);
  if (bf16)
    hipLaunchKernelGGL(prefix_copy_kernel<uint16_t>, grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(prefix_copy_kernel<float>, grid, dim3(256), 0, s, a);
}

}  // namespace via
