// GEMMs of the verification forward: P[split][M][N] = X[M, K-slice] * W[N,
// K-slice]^T with M = fed rows and W packed.  gemm_path picks the kernel family
// by the number of rows: weights streamed past registers (up to 32 rows, with
// an LDS-staged kernel for the head), LDS-fed row tiles, 256 x 256 prefill
// tiles; fp32 models have one kernel of their own.
//
// LDS-staged head: a work-group of 8 waves owns a 256-column tile; each wave
// owns two 16-column blocks and streams their weights over all of K, two
// chunks of steps ahead of its multiply.  The activation fragments (X) of a
// chunk are loaded once per work-group into LDS (double-buffered) and read
// there by all eight waves, so X leaves L2 once per work-group and no
// cross-wave reduction is needed.
//
// The K slices of a tile ("splits") are written as separate fp32 partial tiles
// and summed, in split order, by the consumer kernel after the kernel boundary:
// handing partial sums between work-groups inside one kernel would need a
// device-scope release, which costs an L2 writeback on this GPU.  Every
// reduction has a fixed order, so results are bitwise reproducible.
//
// bf16 operands (v_mfma_f32_16x16x32_bf16): lane l holds row/column l%16 and
// K sub-block (l/16)*8 .. +7 of each 32-wide step.  Weights are pre-packed
// (via_pack_weight) and activations are written by their producer kernels
// as fragments (afrag_group), so every global load of a wave reads one
// contiguous 1 KB block and every LDS read is conflict-free.  fp32
// activations enter the matrix cores as kTerms bf16 terms (x = hi + lo, ~16
// significant bits).  Output register r of lane l is row (l/16)*4 + r, column
// l%16.  The head reduces its tile to per-row (max, second, sum-exp, argmax)
// partials and draft-token logits in place.
// fp32 models multiply in fp32 (v_mfma_f32_16x16x4_f32).
#include <hip/hip_ext.h>

#include "kernels.h"

namespace via {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;
constexpr int kNBW = 2;                // 16-column blocks per wave
constexpr int kTileN = 8 * 16 * kNBW;   // columns per work-group tile (8 waves)

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Work-group tile: the first 16*MB rows x (8 * 16 * NBW) columns over all of
// K.  Wave w owns NBW 16-column blocks and streams their packed W in chunks of
// C steps, two chunks ahead of the one it multiplies; the X fragments of a
// chunk are loaded one chunk ahead and staged once in LDS (double-buffered),
// where all eight waves read them: X leaves L2 once per work-group and no
// cross-wave reduction is needed.  Columns past N are computed from a clamped
// tile and never stored.
template <int MB, int NT, int NBW, int C>
struct TileShape {
  static constexpr int kCols = 8 * 16 * NBW;
  static constexpr int kXChunk = C * NT * MB * 64;   // uint4 per staged chunk
  static constexpr int kXPT = kXChunk / kThreads;     // uint4 staged per thread
};

// M32 (two 16-column blocks per wave, an even number of row blocks): the
// products run on v_mfma_f32_32x32x16_bf16, twice the rate of the 16x16x32
// form on this GPU.  Its operands are gathered from the same 1 KB
// fragments: lane l of a 32-row (or 32-column) x 16-K operand takes
// row (column) l%32 -- block (l/16)%2 of the pair, row l%16 -- and K group
// 2h + l/32 of the 32-wide step (half h), i.e. fragment lane
// (2h + l/32)*16 + l%16.  acc is then f32x16[MB/2]: 32-row tile i holds
// rows 32i + (r/4)*8 + (l/32)*4 + r%4, column l%32 of the wave's 32.
template <int MB, int NT, int NBW, int C, bool M32 = false, typename Acc>
__device__ void tile_bf16(const GemmArgs& a, int c0, uint4* sx, Acc& acc) {
  using TS = TileShape<MB, NT, NBW, C>;
  static_assert(TS::kXChunk % kThreads == 0, "chunk must split evenly over the threads");
  static_assert(!M32 || (NBW == 2 && MB % 2 == 0), "32x32 tiles need two column blocks and row-block pairs");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int S = a.K >> 5;
  const int t64 = (a.N + 63) >> 6;
  const int sel = (lane >> 4) & 1;                        // M32: block of the pair
  const int fl = M32 ? ((lane >> 5) * 16 + (lane & 15)) : lane;  // M32: fragment lane of half 0
  const uint4* wt[NBW];
#pragma unroll
  for (int j = 0; j < NBW; ++j) {
    // M32: wt[j] is K half j of the lane's block; otherwise block j, own lane
    const int blk = (c0 >> 4) + wave * NBW + (M32 ? sel : j);  // global 16-column block
    const int pt = min(blk >> 2, t64 - 1);
    wt[j] = (const uint4*)a.W + (size_t)pt * S * 256 + (blk & 3) * 64 + (M32 ? fl + j * 32 : lane);
  }
  const uint4* xg = (const uint4*)a.X;
  const size_t x_step = (size_t)a.MBn * 64, x_term = (size_t)S * x_step;
  if constexpr (M32) {
#pragma unroll
    for (int i = 0; i < MB / 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  } else {
#pragma unroll
    for (int j = 0; j < NBW; ++j)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[j][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int nch = (S + C - 1) / C;

#define TILE_LOAD_W(w, ch)                                                  \
  _Pragma("unroll") for (int sc = 0; sc < C; ++sc) {                        \
    const size_t st = (size_t)min((ch) * C + sc, S - 1);                    \
    _Pragma("unroll") for (int j = 0; j < NBW; ++j) w[sc][j] = wt[j][st * 256]; \
  }
#define TILE_LOAD_X(ch)                                                     \
  {                                                                         \
    _Pragma("unroll") for (int u = 0; u < TS::kXPT; ++u) {                  \
      const int e = threadIdx.x + u * kThreads; /* [step][term][mb][lane] */ \
      const int l = e & 63, mb = (e >> 6) % MB, q = (e / (64 * MB)) % NT, sc = e / (64 * MB * NT); \
      const size_t st = (size_t)min((ch) * C + sc, S - 1);                 \
      xs[u] = xg[q * x_term + st * x_step + mb * 64 + l];                   \
    }                                                                       \
  }
#define TILE_STORE_X(ch)                                                    \
  {                                                                         \
    uint4* d = sx + ((ch) & 1) * TS::kXChunk + threadIdx.x;                 \
    _Pragma("unroll") for (int u = 0; u < TS::kXPT; ++u) d[u * kThreads] = xs[u]; \
  }
#define TILE_COMPUTE(w, ch)                                                 \
  {                                                                         \
    const int valid = S - (ch) * C;                                         \
    if constexpr (M32) {                                                    \
      const uint4* xb = sx + ((ch) & 1) * TS::kXChunk + sel * 64 + fl;      \
      _Pragma("unroll") for (int sc = 0; sc < C; ++sc) {                    \
        if (sc < valid) {                                                   \
          _Pragma("unroll") for (int q = 0; q < NT; ++q)                    \
          _Pragma("unroll") for (int i = 0; i < MB / 2; ++i)                \
          _Pragma("unroll") for (int h = 0; h < 2; ++h) {                   \
            const uint4 xv = xb[((sc * NT + q) * MB + 2 * i) * 64 + h * 32]; \
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(xv), as_bf16x8(w[sc][h]), acc[i], 0, 0, 0); \
          }                                                                 \
        }                                                                   \
      }                                                                     \
    } else {                                                                \
      const uint4* xb = sx + ((ch) & 1) * TS::kXChunk + lane;               \
      _Pragma("unroll") for (int sc = 0; sc < C; ++sc) {                    \
        if (sc < valid) {                                                   \
          _Pragma("unroll") for (int q = 0; q < NT; ++q)                    \
          _Pragma("unroll") for (int mb = 0; mb < MB; ++mb) {               \
            const uint4 xv = xb[((sc * NT + q) * MB + mb) * 64];            \
            _Pragma("unroll") for (int j = 0; j < NBW; ++j)                 \
              acc[j][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(xv), as_bf16x8(w[sc][j]), acc[j][mb], 0, 0, 0); \
          }                                                                 \
        }                                                                   \
      }                                                                     \
    }                                                                       \
  }
  // one chunk: prefetch X(ch+1) and W(ch+2), multiply chunk ch, publish
  // X(ch+1).  Past the last chunk the prefetches repeat it (unconditional
  // code keeps the staging registers out of scratch memory); the buffer
  // they fill is never read.
#define TILE_CHUNK(wcur, wnext2, ch)                                        \
  {                                                                         \
    TILE_LOAD_X(min((ch) + 1, nch - 1));                                    \
    TILE_LOAD_W(wnext2, min((ch) + 2, nch - 1));                            \
    TILE_COMPUTE(wcur, ch);                                                 \
    TILE_STORE_X((ch) + 1);                                                 \
    __syncthreads();                                                        \
  }
  // buffer indices are compile-time constants (a runtime index would put
  // the buffers in scratch memory): the chunk loop is unrolled by three
  uint4 w0[C][NBW], w1[C][NBW], w2[C][NBW];
  uint4 xs[TS::kXPT];
  TILE_LOAD_X(0);
  TILE_LOAD_W(w0, 0);
  TILE_LOAD_W(w1, min(1, nch - 1));
  TILE_STORE_X(0);
  __syncthreads();
  for (int ch = 0; ch < nch; ch += 3) {
    TILE_CHUNK(w0, w2, ch);
    if (ch + 1 >= nch) break;
    TILE_CHUNK(w1, w0, ch + 1);
    if (ch + 2 >= nch) break;
    TILE_CHUNK(w2, w1, ch + 2);
  }
#undef TILE_CHUNK
#undef TILE_COMPUTE
#undef TILE_STORE_X
#undef TILE_LOAD_X
#undef TILE_LOAD_W
}

// (max, argmax, second) merge with lowest-index tie break
__device__ __forceinline__ void merge3(float& mx, int& am, float& sc, float mx2, int am2, float sc2) {
  if (mx2 > mx || (mx2 == mx && am2 < am)) {
    sc = fmaxf(sc2, mx);
    mx = mx2;
    am = am2;
  } else {
    sc = fmaxf(sc, mx2);
  }
}

// Head tile epilogue, per head row: partial (max, second, sum-exp at the tile
// max, argmax), the logit of each draft token inside the tile, and the
// optional fp32 logits dump.  16 threads per row take every 16th column (no
// bank conflicts) and leave the scaled logits in the tile; the dump is written
// a row per wave, 256 contiguous bytes a store (8B, 256 rows: 590 -> 470 us).
template <int MB, int TN = kTileN, int LDC = TN, int THR = kThreads>
__device__ void epi_stats(const GemmArgs& a, int tile, int m0, float* lds) {
  const int grp = threadIdx.x >> 4, gl = threadIdx.x & 15;  // THR / 16 groups of 16 threads
  const int c0 = tile * TN;
  for (int r = grp; r < 16 * MB; r += THR / 16) {
    const int m = m0 + r;
    if (m >= a.M) continue;  // uniform within the group
    // the row's final RMSNorm scale (the head is linear in it)
    const float rs = row_scale(a.ss, a.ss_stride, m, a.K, a.eps);
    float mx = -INFINITY, sc = -INFINITY;
    int am = 0x7fffffff;
    constexpr int CPT = TN / 16;
    float v[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = gl + 16 * i;
      v[i] = lds[r * LDC + c] * rs;
      lds[r * LDC + c] = v[i];
      if (c0 + c < a.N) merge3(mx, am, sc, v[i], c0 + c, -INFINITY);
    }
    for (int o = 1; o < 16; o <<= 1) {
      const float mx2 = __shfl_xor(mx, o, 64), sc2 = __shfl_xor(sc, o, 64);
      const int am2 = __shfl_xor(am, o, 64);
      merge3(mx, am, sc, mx2, am2, sc2);
    }
    float se = 0.f;
#pragma unroll
    for (int i = 0; i < CPT; ++i)
      if (c0 + gl + 16 * i < a.N) se += expf((v[i] - mx) * a.inv_T);
    for (int o = 1; o < 16; o <<= 1) se += __shfl_xor(se, o, 64);
    if (gl == 0) {
      float* p = a.lm_part + ((size_t)tile * a.M + m) * 4;
      p[0] = mx;
      p[1] = sc;
      p[2] = se;
      p[3] = __int_as_float(am);
    }
    if (gl < min(a.lm[m].n_drafts, kMaxChildren)) {
      const int tk = a.lm[m].draft_tok[gl];
      // (the columns of a row belong to one wave: its writes above are in order)
      if (tk >= c0 && tk < c0 + TN) a.draft_logit[a.lm[m].draft_idx[gl]] = lds[r * LDC + tk - c0];
    }
  }
  if (!a.logits) return;
  __syncthreads();
  for (int r = threadIdx.x >> 6; r < 16 * MB; r += THR / 64) {
    const int m = m0 + r;
    if (m >= a.M) break;
    float* o = a.logits + (size_t)a.lm[m].out * a.N + c0;
    for (int c = threadIdx.x & 63; c < TN; c += 64)
      if (c0 + c < a.N) o[c] = lds[r * LDC + c];
  }
}

// Head of up to 32 rows (bf16): tiles of 256 columns over all of K.
template <int MB, int C>
__global__ __launch_bounds__(kThreads) void gemm_head(GemmArgs a) {
  using TS = TileShape<MB, kTerms, kNBW, C>;
  constexpr int kLdsX = 2 * TS::kXChunk * 16;               // bytes of the X double buffer
  constexpr int kLdc = kTileN + 4, kLdsT = 16 * MB * kLdc * 4;  // bytes of an fp32 output tile (rows padded)
  constexpr int kLds = kLdsX > kLdsT ? kLdsX : kLdsT;
  __shared__ __align__(16) unsigned char smem[kLds];
  float* lds = (float*)smem;
  const int tile = blockIdx.x, c0 = tile * kTileN, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if constexpr (MB % 2 == 0) {
    // 32x32x16 MFMAs: tile i, register r of lane l is row 32i + (r/4)*8 + (l/32)*4 + r%4,
    // column wave*32 + l%32 of the work-group's tile
    f32x16 acc[MB / 2];
    tile_bf16<MB, kTerms, kNBW, C, true>(a, c0, (uint4*)smem, acc);
    const int cl = wave * 32 + (lane & 31), rl = (lane >> 5) * 4;
    __syncthreads();  // the X buffers become the output tile
#pragma unroll
    for (int i = 0; i < MB / 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) lds[(i * 32 + (r >> 2) * 8 + rl + (r & 3)) * kLdc + cl] = acc[i][r];
  } else {
    f32x4 acc[kNBW][MB];
    tile_bf16<MB, kTerms, kNBW, C>(a, c0, (uint4*)smem, acc);
    const int n = lane & 15, g = lane >> 4;
    __syncthreads();  // the X buffers become the output tile
#pragma unroll
    for (int j = 0; j < kNBW; ++j)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) lds[(mb * 16 + g * 4 + r) * kLdc + (wave * kNBW + j) * 16 + n] = acc[j][mb][r];
  }
  __syncthreads();
  epi_stats<MB, kTileN, kLdc>(a, tile, 0, lds);
}

// Every projection of fp32 models, on v_mfma_f32_16x16x4_f32 (fp32 products
// and sums).  The packed layouts give lane l of a 16-row (column) block the 8
// consecutive k's (l/16)*8 .. +7 of each 32-wide step, so element e of all
// lanes is one MFMA operand over the k's {e, 8 + e, 16 + e, 24 + e}.  These
// models are small, so latency is the cost: a work-group owns NB column blocks
// of 16 MB rows over all of K, its 8 waves interleave the K steps (one step of
// loads ahead) and their partial tiles are added in LDS in wave order.  A K of
// 256 is one step per wave: 14 us for the serial vector-ALU loop, now 4.
enum class Epi { kPart, kSwiglu, kStats };  // what is done with a tile
template <int MB, int NB, Epi EPI>
__global__ __launch_bounds__(kThreads) void gemm_f32(GemmArgs a) {
  constexpr int kCols = NB * 16, kStride = kCols + 4;
  __shared__ __align__(16) float red[kWaves][16 * MB][kStride];
  const int blk0 = blockIdx.x * NB, m0 = blockIdx.y * 16 * MB;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int S = a.K >> 5, t64 = (a.N + 63) >> 6;
  const float4* wt[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int blk = min(blk0 + j, t64 * 4 - 1);  // columns past N: never stored
    wt[j] = (const float4*)a.W + ((size_t)(blk >> 2) * S * 256 + (blk & 3) * 64 + lane) * 2;
  }
  const float4* xt[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
    xt[i] = (const float4*)a.X + ((size_t)min((m0 >> 4) + i, a.MBn - 1) * 64 + lane) * 2;
  f32x4 acc[NB][MB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < MB; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nst = max(0, (S - wave + kWaves - 1) / kWaves);  // steps of this wave
  float4 w[2][NB][2], x[2][MB][2];
  auto load = [&](int buf, int i) {
    const size_t st = (size_t)(wave + min(i, nst - 1) * kWaves);
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) w[buf][j][h] = wt[j][st * 512 + h];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int h = 0; h < 2; ++h) x[buf][m][h] = xt[m][st * a.MBn * 128 + h];
  };
  auto compute = [&](int buf) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          const float4 xv = x[buf][m][h], wv = w[buf][j][h];
          acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv.x, wv.x, acc[j][m], 0, 0, 0);
          acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv.y, wv.y, acc[j][m], 0, 0, 0);
          acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv.z, wv.z, acc[j][m], 0, 0, 0);
          acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv.w, wv.w, acc[j][m], 0, 0, 0);
        }
  };
  if (nst > 0) {
    load(0, 0);
    for (int i = 0; i < nst; i += 2) {
      load(1, i + 1);
      compute(0);
      if (i + 1 >= nst) break;
      load(0, i + 2);
      compute(1);
    }
  }
  const int n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][i * 16 + g * 4 + r][j * 16 + n] = acc[j][i][r];
  __syncthreads();
  if constexpr (EPI == Epi::kSwiglu) {
    for (int e = threadIdx.x; e < 16 * MB * NB; e += kThreads) {
      const int r = e / NB, j = e - r * NB, m = m0 + r;
      if (m >= a.M || blk0 + j >= a.N >> 4) continue;
      const float sc = row_scale(a.ss, a.ss_stride, m, a.K, a.eps);  // RMSNorm of the input row
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float gt = 0.f, up = 0.f;
#pragma unroll
        for (int wv = 0; wv < kWaves; ++wv) {
          gt += red[wv][r][j * 16 + i];
          up += red[wv][r][j * 16 + 8 + i];
        }
        gt *= sc;
        up *= sc;
        v[i] = gt / (1.0f + expf(-gt)) * up;
      }
      put_afrag<false, 1>(a.H, m, (blk0 + j) * 8, v, a.F >> 5, a.MBn);
    }
  } else {
    for (int e = threadIdx.x; e < 16 * MB * kCols; e += kThreads) {
      const int r = e / kCols, c = e - r * kCols, m = m0 + r, col = blk0 * 16 + c;
      float v = 0.f;
#pragma unroll
      for (int wv = 0; wv < kWaves; ++wv) v += red[wv][r][c];
      if constexpr (EPI == Epi::kStats)
        red[0][r][c] = v;
      else if (m < a.M && col < a.N)
        a.part[(size_t)m * a.N + col] = v;
    }
    if constexpr (EPI == Epi::kStats) {
      __syncthreads();
      epi_stats<MB, kCols, kStride>(a, blockIdx.x, m0, &red[0][0][0]);
    }
  }
}

// Gate/up with SwiGLU for up to 32 rows, K-interleaved: wave w multiplies
// K steps w, w + 8, w + 16, ... of all a.nb (<= 8) column blocks of the
// work-group, loading its X fragments straight from global memory (each is
// used by one wave only, so neither LDS staging nor a barrier sits in the
// main loop), one step of loads ahead of its MFMAs.  Weights are read with
// non-temporal loads: streamed once, they should not displace X from the
// caches.  The eight waves' partial tiles are summed in LDS in wave order
// (fixed, so the result is reproducible) and the epilogue writes h as the
// down projection's fragments.
__device__ __forceinline__ uint4 load_stream(const uint4* p) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

template <int MB>
__global__ __launch_bounds__(kThreads) void gemm_gate_up_ki(GemmArgs a) {
  constexpr int NT = 2, NBM = kWaves;
  __shared__ __align__(16) float red[kWaves][16 * MB][NBM * 16 + 4];
  const int nblocks = a.N >> 4;
  const int blk0 = blockIdx.x * a.nb;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int nb = min(a.nb, nblocks - blk0);
  const int S = a.K >> 5, t64 = (a.N + 63) >> 6;
  const uint4* wt[NBM];
#pragma unroll
  for (int j = 0; j < NBM; ++j) {
    const int blk = blk0 + min(j, nb - 1);
    wt[j] = (const uint4*)a.W + (size_t)min(blk >> 2, t64 - 1) * S * 256 + (blk & 3) * 64 + lane;
  }
  const uint4* xg = (const uint4*)a.X + lane;
  const size_t x_step = (size_t)a.MBn * 64, x_term = (size_t)S * x_step;
  f32x4 acc[NBM][MB];
#pragma unroll
  for (int j = 0; j < NBM; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[j][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nst = max(0, (S - wave + kWaves - 1) / kWaves);  // steps of this wave
  uint4 w[2][NBM], x[2][NT][MB];
  // loads of the wave's i-th step into buffer `buf` (past the last step the
  // last one is loaded again and never used)
  auto load = [&](int buf, int i) {
    const size_t st = (size_t)(wave + min(i, nst - 1) * kWaves);
#pragma unroll
    for (int j = 0; j < NBM; ++j)
      if (j < nb) w[buf][j] = load_stream(wt[j] + st * 256);
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) x[buf][q][mb] = xg[q * x_term + st * x_step + mb * 64];
  };
  auto compute = [&](int buf) {
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < NBM; ++j)
          if (j < nb)
            acc[j][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x[buf][q][mb]), as_bf16x8(w[buf][j]),
                                                                 acc[j][mb], 0, 0, 0);
  };
  if (nst > 0) {
    load(0, 0);
    for (int i = 0; i < nst; i += 2) {
      load(1, i + 1);
      compute(0);
      if (i + 1 >= nst) break;
      load(0, i + 2);
      compute(1);
    }
  }
  const int n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int j = 0; j < NBM; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][mb * 16 + g * 4 + r][j * 16 + n] = acc[j][mb][r];
  __syncthreads();
  for (int e = threadIdx.x; e < 16 * MB * nb; e += kThreads) {
    const int r = e / nb, j = e - r * nb;
    if (r >= a.M) continue;
    const float sc = row_scale(a.ss, a.ss_stride, r, a.K, a.eps);  // RMSNorm of the input row
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float gt = 0.f, up = 0.f;
#pragma unroll
      for (int wv = 0; wv < kWaves; ++wv) {
        gt += red[wv][r][j * 16 + i];
        up += red[wv][r][j * 16 + 8 + i];
      }
      gt *= sc;
      up *= sc;
      v[i] = gt / (1.0f + expf(-gt)) * up;
    }
    put_afrag<true, NT>(a.H, r, (blk0 + j) * 8, v, a.F >> 5, a.MBn);
  }
}

// With timing events the launch carries them in its dispatch, so they
// bracket the kernel itself rather than the stream around it.
template <typename K>
void launch_timed(K kernel, dim3 grid, int threads, const GemmArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (e0)
    hipExtLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, e0, e1, 0, a);
  else
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, a);
}
void launch_head(const GemmArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(gemm_head_tiles(true, a.M, a.N, a.K));
  if (a.M <= 16)
    launch_timed(gemm_head<1, 4>, grid, kThreads, a, s, e0, e1);
  else
    launch_timed(gemm_head<2, 4>, grid, kThreads, a, s, e0, e1);
}
void launch_gate_up_ki(const GemmArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(((a.N >> 4) + a.nb - 1) / a.nb);
  if (a.M <= 16)
    launch_timed(gemm_gate_up_ki<1>, grid, kThreads, a, s, e0, e1);
  else
    launch_timed(gemm_gate_up_ki<2>, grid, kThreads, a, s, e0, e1);
}
void launch_f32(GemmRole role, const GemmArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  // one 16-row block as far as it goes, else 64 rows; one column block per
  // work-group until there are 256 of them with four
  const int rows = a.M <= 16 ? 16 : 64, groups = (a.M + rows - 1) / rows;
  const bool wide = role == GemmRole::kHead || (rows == 64 && (a.N + 63) / 64 * groups >= 256);
  const dim3 grid(wide ? (a.N + 63) / 64 : (a.N + 15) / 16, groups);
  auto go = [&](auto kernel) { launch_timed(kernel, grid, kThreads, a, s, e0, e1); };
  if (role == GemmRole::kHead)
    rows == 16 ? go(gemm_f32<1, 4, Epi::kStats>) : go(gemm_f32<4, 4, Epi::kStats>);
  else if (role == GemmRole::kGateUp)
    rows == 16 ? go(gemm_f32<1, 1, Epi::kSwiglu>) : wide ? go(gemm_f32<4, 4, Epi::kSwiglu>) : go(gemm_f32<4, 1, Epi::kSwiglu>);
  else
    rows == 16 ? go(gemm_f32<1, 1, Epi::kPart>) : wide ? go(gemm_f32<4, 4, Epi::kPart>) : go(gemm_f32<4, 1, Epi::kPart>);
}


// QKV, O and down projections of forwards of up to 32 rows (bf16): the
// weight-streaming decomposition of the gate/up kernel with split-K partials.
// A work-group owns a.nb 16-column blocks and K split blockIdx.x % a.ksplit (a.ksplit
// equal ranges of 32-wide steps); its 8 waves interleave the split's steps
// (wave w takes steps w, w+8, ...) over all its blocks, loading X fragments
// straight from global memory (each is used by one wave; they stay in L2)
// and weights with non-temporal loads, one step ahead.  The 8 wave partial
// tiles are summed in LDS in wave order and written to
// a.part[split][M][N], which the consumer sums in split order.  Fewer,
// longer splits (4-8, not 10-16) write a quarter of the partials.
template <int MB, int NT>
__global__ __launch_bounds__(kThreads) void gemm_ki_part(GemmArgs a) {
  constexpr int NBM = kWaves;
  __shared__ __align__(16) float red[kWaves][16 * MB][NBM * 16 + 4];
  const int nblocks = a.N >> 4;
  const int split = blockIdx.x % a.ksplit;
  const int blk0 = (blockIdx.x / a.ksplit) * a.nb;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int nb = min(a.nb, nblocks - blk0);
  const int S = a.K >> 5, t64 = (a.N + 63) >> 6;
  const int per = (S + a.ksplit - 1) / a.ksplit;
  const int s_beg = min(S, split * per), s_end = min(S, s_beg + per);
  const uint4* wt[NBM];
#pragma unroll
  for (int j = 0; j < NBM; ++j) {
    const int blk = blk0 + min(j, nb - 1);
    wt[j] = (const uint4*)a.W + (size_t)min(blk >> 2, t64 - 1) * S * 256 + (blk & 3) * 64 + lane;
  }
  const uint4* xg = (const uint4*)a.X + lane;
  const size_t x_step = (size_t)a.MBn * 64, x_term = (size_t)S * x_step;
  f32x4 acc[NBM][MB];
#pragma unroll
  for (int j = 0; j < NBM; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[j][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nst = max(0, (s_end - s_beg - wave + kWaves - 1) / kWaves);  // steps of this wave
  uint4 w[2][NBM], x[2][NT][MB];
  // loads of the wave's i-th step into buffer `buf` (past the last step the
  // last one is loaded again and never used)
  auto load = [&](int buf, int i) {
    const size_t st = (size_t)(s_beg + wave + min(i, nst - 1) * kWaves);
#pragma unroll
    for (int j = 0; j < NBM; ++j)
      if (j < nb) w[buf][j] = load_stream(wt[j] + st * 256);
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) x[buf][q][mb] = xg[q * x_term + st * x_step + mb * 64];
  };
  auto compute = [&](int buf) {
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < NBM; ++j)
          if (j < nb)
            acc[j][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x[buf][q][mb]), as_bf16x8(w[buf][j]),
                                                                 acc[j][mb], 0, 0, 0);
  };
  if (nst > 0) {
    load(0, 0);
    for (int i = 0; i < nst; i += 2) {
      load(1, i + 1);
      compute(0);
      if (i + 1 >= nst) break;
      load(0, i + 2);
      compute(1);
    }
  }
  const int n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int j = 0; j < NBM; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][mb * 16 + g * 4 + r][j * 16 + n] = acc[j][mb][r];
  __syncthreads();
  float* P = a.part + (size_t)split * a.M * a.N;
  const int cols = nb * 16;
  for (int e = threadIdx.x; e < 16 * MB * cols; e += kThreads) {
    const int r = e / cols, c = e - r * cols;
    if (r >= a.M) continue;
    float v = 0.f;
#pragma unroll
    for (int wv = 0; wv < kWaves; ++wv) v += red[wv][r][c];
    P[(size_t)r * a.N + blk0 * 16 + c] = v;
  }
}

// The same decomposition at a fixed shape: NB blocks per work-group and
// exactly NSW steps per wave, fully unrolled, with the loads of DEPTH steps
// in flight (a ring of DEPTH register buffers) instead of one.  Used when
// the K split and the column blocks divide evenly.
template <int MB, int NT, int NB, int NSW, int DEPTH>
__global__ __launch_bounds__(kThreads) void gemm_ki_fixed(GemmArgs a) {
  __shared__ __align__(16) float red[kWaves][16 * MB][NB * 16 + 4];
  const int split = blockIdx.x % a.ksplit;
  const int blk0 = (blockIdx.x / a.ksplit) * NB;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int S = a.K >> 5, t64 = (a.N + 63) >> 6;
  const int s_beg = split * NSW * kWaves;
  const uint4* wt[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int blk = blk0 + j;
    wt[j] = (const uint4*)a.W + (size_t)min(blk >> 2, t64 - 1) * S * 256 + (blk & 3) * 64 + lane;
  }
  const uint4* xg = (const uint4*)a.X + lane;
  const size_t x_step = (size_t)a.MBn * 64, x_term = (size_t)S * x_step;
  f32x4 acc[NB][MB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[j][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint4 w[DEPTH][NB], x[DEPTH][NT][MB];
  // iteration i multiplies step i - DEPTH (its buffer) and then loads step i into it
#pragma unroll
  for (int i = 0; i < NSW + DEPTH; ++i) {
    if (i >= DEPTH) {
      const int b = (i - DEPTH) % DEPTH;
#pragma unroll
      for (int q = 0; q < NT; ++q)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[j][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x[b][q][mb]), as_bf16x8(w[b][j]),
                                                                 acc[j][mb], 0, 0, 0);
    }
    if (i < NSW) {
      const int b = i % DEPTH;
      const size_t st = (size_t)(s_beg + wave + i * kWaves);
#pragma unroll
      for (int j = 0; j < NB; ++j) w[b][j] = load_stream(wt[j] + st * 256);
#pragma unroll
      for (int q = 0; q < NT; ++q)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) x[b][q][mb] = xg[q * x_term + st * x_step + mb * 64];
    }
  }
  const int n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][mb * 16 + g * 4 + r][j * 16 + n] = acc[j][mb][r];
  __syncthreads();
  float* P = a.part + (size_t)split * a.M * a.N;
  constexpr int cols = NB * 16;
  for (int e = threadIdx.x; e < 16 * MB * cols; e += kThreads) {
    const int r = e / cols, c = e - r * cols;
    if (r >= a.M) continue;
    float v = 0.f;
#pragma unroll
    for (int wv = 0; wv < kWaves; ++wv) v += red[wv][r][c];
    P[(size_t)r * a.N + blk0 * 16 + c] = v;
  }
}

void launch_ki_part(const GemmArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  // split-major order: work-group i takes K split i % ksplit, so with the
  // round-robin dispatch of work-groups over the 8 XCDs each XCD's
  // work-groups share 8 / ksplit splits (one for 8 splits) and its L2 holds
  // only their slices of the activations
  const dim3 grid((((a.N >> 4) + a.nb - 1) / a.nb) * a.ksplit);
  auto go = [&](auto kernel) { launch_timed(kernel, grid, kThreads, a, s, e0, e1); };
  // fixed shapes (the 8B and 1B projections): even K splits and column blocks
  const int S = a.K >> 5, per = S / a.ksplit, nsw = per / kWaves;
  if (S % a.ksplit == 0 && per % kWaves == 0 && (a.N >> 4) % a.nb == 0) {
#define VIA_KI_FIXED(NB_, NSW_)                                                   \
  if (a.nb == NB_ && nsw == NSW_) {                                              \
    if (a.M <= 16)                                                               \
      go(gemm_ki_fixed<1, kTerms, NB_, NSW_, 2>);                                    \
    else                                                                         \
      go(gemm_ki_fixed<2, kTerms, NB_, NSW_, 2>);                                    \
    return;                                                                      \
  }
    VIA_KI_FIXED(6, 4)
    VIA_KI_FIXED(4, 4)
    VIA_KI_FIXED(8, 7)
    VIA_KI_FIXED(2, 4)
    VIA_KI_FIXED(1, 4)
#undef VIA_KI_FIXED
  }
  if (a.M <= 16)
    go(gemm_ki_part<1, kTerms>);
  else
    go(gemm_ki_part<2, kTerms>);
}

// ---------------------------------------------------------------- head stats
// One work-group per head row; reductions by lane shuffles, then the four
// waves in order.
__global__ __launch_bounds__(256) void lm_finalize_kernel(const LmRow* lm, const float* part, int M, int ntiles,
                                                          float inv_T, int32_t* row_argmax, float* row_max,
                                                          float* row_sumexp, float* row_gap) {
  __shared__ float s_mx[4], s_sc[4], s_se[4];
  __shared__ int s_am[4];
  const int m = blockIdx.x, t = threadIdx.x, w = t >> 6;
  const int out = lm[m].out;
  float mx = -INFINITY, sc = -INFINITY;
  int am = 0x7fffffff;
  for (int tl = t; tl < ntiles; tl += 256) {
    const float4 p = *(const float4*)(part + ((size_t)tl * M + m) * 4);
    merge3(mx, am, sc, p.x, __float_as_int(p.w), p.y);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float mx2 = __shfl_xor(mx, o, 64), sc2 = __shfl_xor(sc, o, 64);
    const int am2 = __shfl_xor(am, o, 64);
    merge3(mx, am, sc, mx2, am2, sc2);
  }
  if ((t & 63) == 0) {
    s_mx[w] = mx;
    s_sc[w] = sc;
    s_am[w] = am;
  }
  __syncthreads();
  mx = s_mx[0];
  sc = s_sc[0];
  am = s_am[0];
#pragma unroll
  for (int i = 1; i < 4; ++i) merge3(mx, am, sc, s_mx[i], s_am[i], s_sc[i]);
  float se = 0.f;
  for (int tl = t; tl < ntiles; tl += 256) {
    const float* p = part + ((size_t)tl * M + m) * 4;
    se += p[2] * expf((p[0] - mx) * inv_T);
  }
  se = wave_sum(se);
  if ((t & 63) == 0) s_se[w] = se;
  __syncthreads();
  if (t == 0) {
    row_max[out] = mx;
    row_argmax[out] = am;
    row_sumexp[out] = ((s_se[0] + s_se[1]) + s_se[2]) + s_se[3];
    if (row_gap) row_gap[out] = mx - sc;
  }
}

// Row-major [rows, cols] -> packed tiles; one thread per 8-element group.
template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(const T* src, T* dst, int rows, int cols, int ffn, size_t groups) {
  const size_t gidx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (gidx >= groups) return;
  const int steps = cols >> 5;
  const int lane = (int)(gidx & 63);
  size_t q = gidx >> 6;
  const int nb = (int)(q & 3);
  q >>= 2;
  const int st = (int)(q % steps);
  const size_t tile = q / steps;
  const size_t r = tile * 64 + nb * 16 + (lane & 15);
  const size_t c = (size_t)st * 32 + (lane >> 4) * 8;
  // gate/up interleave: packed row 16 b + i <- gate row 8 b + i, or up row 8 b + i - 8
  const size_t sr = ffn > 0 ? ((r & 8) ? (size_t)ffn : 0) + (r >> 4) * 8 + (r & 7) : r;
#pragma unroll
  for (int e = 0; e < 8; ++e) dst[gidx * 8 + e] = r < (size_t)rows ? src[sr * cols + c + e] : T(0);
}

// ------------------------------------------------------------- prefill GEMM
// Many-row GEMM (prefill-sized M): C[M, N] = sum over the NT activation terms
// of X_q[M, K] W[N, K]^T, fp32, written as one partial tile (split 1) so the
// consumers of the verify GEMMs read it unchanged.  Compute-bound: a
// work-group of 8 waves owns a 256 x 256 tile; wave (wm, wn) computes rows
// wm*128 .. +128 and columns wn*64 .. +64 with v_mfma_f32_16x16x32_bf16.  A
// stage is one 32-wide K step of the tile: 16 row blocks of X and 16 column
// blocks of W, each a contiguous 1 KB fragment in both layouts, copied
// verbatim into LDS by global_load_lds_dwordx4 (16 bytes per lane written at
// m0 + 16 * lane).  Four stages rotate in LDS, two K steps per barrier:
// stage s is copied two to four steps ahead, read into registers during step
// s - 1 and multiplied in step s, so a wave's products never wait for LDS
// after a barrier; the reads of the next step are pinned between the
// products (one read per two MFMAs) so that the compiler cannot sink them
// next to their use again.  The copies are issued
// by inline asm with wave-uniform bases in SGPRs (one lane-offset VGPR for
// all of them) so that the compiler, which would otherwise make every LDS
// read wait for all outstanding copies, leaves their completion to the
// explicit vmcnt waits below.  Work-groups are dispatched
// round-robin over the 8 XCDs; XCD x takes a contiguous range of tiles, taken
// in groups of 8 row tiles so that co-resident work-groups share operand
// blocks in its L2.
//
// SWIGLU (the gate/up projection): instead of the fp32 product the tile's
// epilogue writes h = silu(g s) * (u s) with the input row's RMSNorm scale
// s, as 2-term fragments of the down projection's input.  A 16-column block
// of the packed gate/up weight holds the gate (columns 0-7) and up (8-15)
// rows of the same 8 FFN indices, so lane n < 8 of an output block takes its
// up value from lane n + 8; h of the tile's 128 FFN indices is staged in LDS
// (the freed operand stages) and written 8 indices per fragment group.
constexpr int kPfStages = 4, kPfStage = 32 * 1024;
constexpr int kPfGroupM = 8;
constexpr int kPfHStride = kPfBN / 2 + 4;  // fp32 per staged h row (padded: no bank conflicts)
constexpr int kPfLds = kPfStages * kPfStage > kPfBM * kPfHStride * 4 ? kPfStages * kPfStage : kPfBM * kPfHStride * 4;

// 16 bytes per lane from base + voff to LDS at lds + 16 * lane (base wave-uniform)
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds) : "memory", "m0");
}

// The same, streamed past the caches.
__device__ __forceinline__ void lds_dma16_stream(const void* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(base), "s"(lds) : "memory", "m0");
}

template <bool SWIGLU, bool PAIR>
__global__ __launch_bounds__(kThreads, 1) void gemm_prefill(GemmArgs a, int nt) {
  __shared__ __align__(1024) unsigned char smem[SWIGLU ? kPfLds : kPfStages * kPfStage];
  const int S = a.K >> 5, t64 = (a.N + 63) >> 6;
  const int tiles_n = (a.N + kPfBN - 1) / kPfBN, tiles_m = (a.M + kPfBM - 1) / kPfBM;
  const int ntiles = tiles_m * tiles_n;
  const int per = (ntiles + 7) / 8;
  const int tile = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (tile >= ntiles) return;  // uniform
  const int grp = tile / (kPfGroupM * tiles_n), in = tile % (kPfGroupM * tiles_n);
  const int gm = min(kPfGroupM, tiles_m - grp * kPfGroupM);
  const int m0 = (grp * kPfGroupM + in % gm) * kPfBM, n0 = (in / gm) * kPfBN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  // K32 steps over all terms.  PAIR (two terms): step it is term it % 2 of
  // K step it / 2, so a K step's two terms run back to back and the second
  // reuses the first's W operands (no W copy or W read for it); otherwise
  // term-major, step it is term it / S of K step it % S.
  const int iters = nt * S;
  // wave w copies row blocks w, w + 8 and column blocks w, w + 8 of each stage;
  // blocks past the matrix are clamped (their products are never stored)
  const uint4* xs[2];
  const uint4* ws[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    xs[h] = (const uint4*)a.X + (size_t)min((m0 >> 4) + h * 8 + wave, a.MBn - 1) * 64;
    const int cb = (n0 >> 4) + h * 8 + wave;
    ws[h] = (const uint4*)a.W + (size_t)min(cb >> 2, t64 - 1) * S * 256 + (cb & 3) * 64;
  }
  const size_t xstep = (size_t)a.MBn * 64;
  const uint32_t voff = lane * 16;
  const uint32_t lds_base =
      __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) void*)(smem + wave * 1024));
  auto issue = [&](int it) {
    const int q = PAIR ? (it & 1) : it / S, ks = PAIR ? it >> 1 : it - q * S;
    const uint32_t d = lds_base + (it % kPfStages) * kPfStage;
    lds_dma16(xs[0] + ((size_t)q * S + ks) * xstep, voff, d);
    lds_dma16(xs[1] + ((size_t)q * S + ks) * xstep, voff, d + 8 * 1024);
    if (!PAIR || q == 0) {
      lds_dma16(ws[0] + (size_t)ks * 256, voff, d + 16 * 1024);
      lds_dma16(ws[1] + (size_t)ks * 256, voff, d + 24 * 1024);
    }
  };
  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < kPfStages - 1; ++p) issue(min(p, iters - 1));
  // SwiGLU: the RMSNorm scales of the tile's input rows, read while the
  // first stages are in flight
  __shared__ float rscale[SWIGLU ? kPfBM : 1];
  if constexpr (SWIGLU)
    for (int r = threadIdx.x; r < kPfBM; r += kThreads)
      rscale[r] = m0 + r < a.M ? row_scale(a.ss, a.ss_stride, m0 + r, a.K, a.eps) : 0.f;
  // operands of one step: 8 row blocks of X, 4 column blocks of W
  uint4 pa[8], pb[4], qa[8], qb[4];
  auto read = [&](int it, uint4* A, uint4* B) {  // B null: X only
    const uint4* st = (const uint4*)(smem + (it % kPfStages) * kPfStage);
#pragma unroll
    for (int i = 0; i < 8; ++i) A[i] = st[(wm * 8 + i) * 64 + lane];
    if (B)
#pragma unroll
      for (int j = 0; j < 4; ++j) B[j] = st[(16 + wn * 4 + j) * 64 + lane];
  };
  auto mma = [&](const uint4* A, const uint4* B) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(A[i]), as_bf16x8(B[j]), acc[i][j], 0, 0, 0);
  };
  // the products of one step with the reads of the next (NR of them) pinned
  // between them
#define VIA_PF_PIN(NR)                                                                 \
  _Pragma("unroll") for (int g = 0; g < (NR); ++g) {                                   \
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0); /* 2 MFMAs */                   \
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); /* 1 LDS read */                \
  }                                                                                    \
  __builtin_amdgcn_sched_group_barrier(0x008, 32 - 2 * (NR), 0);
  // stage 0 in LDS (the oldest 4 copies of the 12, PAIR: of 10) and in registers
  __builtin_amdgcn_s_waitcnt((PAIR ? 6 : 4 * (kPfStages - 2)) | (0x7 << 4) | (0xF << 8));
  __builtin_amdgcn_s_barrier();
  read(0, pa, pb);
  // two steps per barrier, it and it + 1, with the register sets swapped: at
  // the barrier every copy has landed (stages it + 1 and it + 2 are read in
  // this trip) and every wave's reads of stages it - 1 and it are back
  // (lgkmcnt 0), so their buffers take stages it + 3 and it + 4 (past the end
  // the last stage is copied again into a buffer nothing reads).  One exit
  // only: an exit between the halves makes the compiler spill.
  int it = 0;
  for (; it + 1 < iters; it += 2) {
    __builtin_amdgcn_s_waitcnt(0x0 | (0x7 << 4) | (0x0 << 8));
    __builtin_amdgcn_s_barrier();
    issue(min(it + 3, iters - 1));
    issue(min(it + 4, iters - 1));
    // PAIR: step it + 1 (second term) multiplies its X with step it's W
    // (pb), and the next K step's W goes to qb, moved to pb afterwards
    read(min(it + 1, iters - 1), qa, PAIR ? nullptr : qb);
    mma(pa, pb);
    VIA_PF_PIN(PAIR ? 8 : 12)
    read(min(it + 2, iters - 1), pa, PAIR ? qb : pb);
    mma(qa, PAIR ? pb : qb);
    VIA_PF_PIN(12)
    if constexpr (PAIR)
#pragma unroll
      for (int j = 0; j < 4; ++j) pb[j] = qb[j];
  }
#undef VIA_PF_PIN
  if (it < iters) mma(pa, pb);  // odd step count (not PAIR): the last stage is in pa, pb
  __builtin_amdgcn_s_waitcnt(0);  // the trailing copies land before the work-group ends
  const int n = lane & 15, g = lane >> 4;
  if constexpr (SWIGLU) {
    __syncthreads();  // every wave's copies have landed and its stage reads are done
    float* hl = (float*)smem;  // [row][FFN index of the tile]
    // lane n < 8 of a 16-lane row holds the gate value of FFN index n, lane
    // n + 8 its up value (rows g * 4 + r).  The pair swaps its four values
    // with a DPP rotate by 8 within the row (xor 8: no LDS round trip), and
    // lane n < 8 computes h for rows r = 0, 1, lane n + 8 for rows 2, 3, so
    // every lane runs the same instructions.
    const bool lo8 = n < 8;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float other[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          other[r] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc[i][j][r]), 0x128, 0xf, 0xf, false));
#pragma unroll
        for (int rr = 0; rr < 2; ++rr) {
          const float gv = lo8 ? acc[i][j][rr] : other[rr + 2];
          const float uv = lo8 ? other[rr] : acc[i][j][rr + 2];
          const int rl = wm * 128 + i * 16 + g * 4 + rr + (lo8 ? 0 : 2);
          const float sc = rscale[rl], gt = gv * sc, u = uv * sc;
          hl[rl * kPfHStride + wn * 32 + j * 8 + (n & 7)] = gt / (1.0f + expf(-gt)) * u;
        }
      }
    __syncthreads();
    // consecutive lanes take consecutive rows of one 8-index group: 16 of
    // them write 256 contiguous bytes of a fragment term
    const int f0 = n0 >> 1;
    for (int e = threadIdx.x; e < kPfBM * (kPfBN / 16); e += kThreads) {
      const int rl = e % kPfBM, gq = e / kPfBM, m = m0 + rl, f = f0 + gq * 8;
      if (m >= a.M || f >= a.F) continue;
      float v[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = hl[rl * kPfHStride + gq * 8 + t];
      put_afrag<true, 2>(a.H, m, f, v, a.F >> 5, a.MBn);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = n0 + wn * 64 + j * 16 + n;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = m0 + wm * 128 + i * 16 + g * 4 + r;
          if (row < a.M && col < a.N) a.part[(size_t)row * a.N + col] = acc[i][j][r];
        }
      }
  }
}

// ----------------------------------------------------------- row-tile GEMM
// bf16 projections and head of forwards between the weight-streaming kernels
// (up to 32 rows) and the 256 x 256 prefill tiles: C[M, N] = sum over the two
// activation terms of X_q[M, K] W[N, K]^T.  A work-group owns a tile of 16 MB
// rows x 64 WN columns and one K split.  Everything reaches the matrix cores
// through LDS: each 32-wide K step's X blocks (both terms) and W blocks are
// copied verbatim by global_load_lds_dwordx4 into rings, and a step is read
// into registers while the one before it is multiplied, so after a barrier no
// product waits for LDS.  A wave multiplies 8 MB rows x 64 columns.
//
// What bounds it is the copies in flight: a compute unit returns them in order,
// so X (an L2 hit) waits behind W (from HBM) and the two together move about
// 46 GB/s per compute unit at ~110 KB in flight, all that the rings hold.
// Half the waves copy W, SW trips deep, the other half X, SX deep, each
// waiting on its own count before the barrier.
//
// WN = 2, KG = 2 (128 columns): up to 128 rows it keeps ~256 work-groups on the
// weight stream, above it is taken where 256 columns would leave compute
// units idle; waves 0-3 multiply the even and 4-7 the odd K steps and the two
// halves are added in LDS.  WN = 2, KG = 1: the same tiles with four waves that
// take every K step, in the order of the 256-column and the prefill tiles, for
// forwards of more than kFixedOrderRows rows; the copies bound both (1B shape,
// 1023 rows, down projection: 58 us without a K split; with four, which make the
// order follow the row count, 40 and 3 more in the residual update).  WN = 4, KG = 1 (256 columns): the fewest copied
// bytes per product.
//
// kPart writes one fp32 partial per split, kSwiglu (the gate/up projection)
// writes h as the down projection's fragments, kStats the head's row statistics.
// s_waitcnt operand: at most vm vector-memory and lgkm LDS operations outstanding
constexpr int waitcnt_imm(int vm, int lgkm) { return (vm & 15) | (7 << 4) | (lgkm << 8) | ((vm >> 4) << 14); }

template <int MB, int WN, int KG, int SX, int SW>
struct RtShape {
  static constexpr int kBN = 64 * WN, kStride = kBN + 4;  // columns; fp32 per row of an output tile in LDS
  static constexpr int kXTrip = KG * 2 * MB * 1024, kWTrip = KG * 4 * WN * 1024;  // bytes per trip (KG K steps)
  static constexpr int kRing = SX * kXTrip + SW * kWTrip;
  static constexpr int kTile = 16 * MB * kStride * 4;
  static constexpr int kLds = kRing > kTile ? kRing : kTile;
  static constexpr int kThreads = 128 * WN * KG;
  static_assert(kLds <= 160 * 1024, "LDS of a compute unit");
  static_assert(MB % 2 == 0 && (2 * MB) % WN == 0 && (WN == 2 || WN == 4), "wave split");
};

template <int MB, int WN, int KG, int SX, int SW, Epi EPI>
__global__ __launch_bounds__(128 * WN * KG, 1) void gemm_row_tile(GemmArgs a) {
  using SH = RtShape<MB, WN, KG, SX, SW>;
  constexpr int HB = MB / 2;  // row blocks of a wave
  constexpr int kThr = SH::kThreads, kBN = SH::kBN, kStride = SH::kStride;
  __shared__ __align__(1024) unsigned char smem[SH::kLds];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int S = a.K >> 5, t64 = (a.N + 63) >> 6;
  // XCD x (work-groups go round robin over the 8) takes a contiguous range of
  // tiles; row tiles of one column tile are neighbours, so they share W in its L2
  const int tiles_m = (a.M + 16 * MB - 1) / (16 * MB), tiles_n = (a.N + kBN - 1) / kBN;
  const int ntiles = tiles_m * tiles_n * a.ksplit, perx = (ntiles + 7) >> 3;
  const int tile = (blockIdx.x & 7) * perx + (blockIdx.x >> 3);
  if (tile >= ntiles) return;  // uniform
  const int tm = tile % tiles_m, tc = tile / tiles_m, split = tc / tiles_n, tn = tc - split * tiles_n;
  const int m0 = tm * 16 * MB, n0 = tn * kBN;
  // K steps of the split: KG of them per trip
  const int per = (S + a.ksplit * KG - 1) / (a.ksplit * KG) * KG;
  const int s_beg = min(S, split * per), s_end = min(S, s_beg + per);
  const int T = (s_end - s_beg + KG - 1) / KG;
  const uint32_t voff = lane * 16;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) void*)smem);
  const uint32_t ldsW = lds0 + SX * SH::kXTrip;
  const size_t xstep = (size_t)a.MBn * 64;
  const uint4* const X = (const uint4*)a.X;
  // block b of a K step and term of X (rows past the fragments repeat the last
  // block, columns past N the last tile: their products are never stored)
  auto copy_x = [&](int ks, int q, int b, uint32_t dst) {
    lds_dma16(X + ((size_t)q * S + ks) * xstep + (size_t)min((m0 >> 4) + b, a.MBn - 1) * 64, voff, dst);
  };
  auto copy_w = [&](int ks, int b, uint32_t dst) {
    const int pt = min((n0 >> 6) + (b >> 2), t64 - 1);
    lds_dma16_stream((const uint4*)a.W + ((size_t)pt * S + ks) * 256 + (b & 3) * 64, voff, dst);
  };
  // this wave's copies of trip t: a 64-column W tile, or a share of one term of
  // X, of one K step (past the end the last K step again, into buffers nothing
  // reads, so that every trip issues the same number)
  constexpr int kNW = 4, kNX = 2 * MB / WN;
  const bool copies_w = wave < KG * WN;
  const int ckk = wave / WN % KG, cr = wave % WN;
  auto issue = [&](int t, int sx, int sw) {
    const int ks = min(s_beg + t * KG + ckk, s_end - 1);
    if (copies_w) {
#pragma unroll
      for (int i = 0; i < kNW; ++i) copy_w(ks, cr * 4 + i, ldsW + ((sw * KG + ckk) * 4 * WN + cr * 4 + i) * 1024);
    } else {
      const int q = cr & 1, b0 = (cr >> 1) * kNX;
#pragma unroll
      for (int b = 0; b < kNX; ++b) copy_x(ks, q, b0 + b, lds0 + (((sx * KG + ckk) * 2 + q) * MB + b0 + b) * 1024);
    }
  };
  f32x4 acc[HB][4];
#pragma unroll
  for (int i = 0; i < HB; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int kg = wave / (2 * WN), wm = wave / WN & 1, wn = wave % WN;
  struct Ops {
    uint4 x[2][HB], w[4];
  };
  auto read = [&](int sx, int sw, Ops& o) {
    const uint4* xb = (const uint4*)(smem + ((sx * KG + kg) * 2 * MB + wm * HB) * 1024) + lane;
    const uint4* wb = (const uint4*)(smem + SX * SH::kXTrip + ((sw * KG + kg) * WN + wn) * 4096) + lane;
#pragma unroll
    for (int j = 0; j < 4; ++j) o.w[j] = wb[j * 64];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < HB; ++i) o.x[q][i] = xb[(q * MB + i) * 64];
  };
  auto mma = [&](const Ops& o) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < HB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(o.x[q][i]), as_bf16x8(o.w[j]), acc[i][j], 0, 0, 0);
  };
  // every wave's copies of trip t + 1 have landed and its reads of trip t are
  // back: the buffers of trip t take trip t + SX (SW)
  auto arrive = [&]() {
    if (copies_w)
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(kNW * (SW - 2), 0));
    else
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(kNX * (SX - 2), 0));
    __builtin_amdgcn_s_barrier();
  };
  static_assert(kNW * (SW - 1) < 64 && kNX * (SX - 1) < 64, "vmcnt");
  constexpr int kReads = 2 * HB + 4, kMma = 8 * HB;  // per K step
#define VIA_RT_PIN()                                                     \
  _Pragma("unroll") for (int g_ = 0; g_ < kReads; ++g_) {               \
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); /* 1 LDS read */ \
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0); /* 2 MFMAs */    \
  }                                                                      \
  if constexpr (kMma > 2 * kReads) __builtin_amdgcn_sched_group_barrier(0x008, kMma - 2 * kReads, 0);
  // 256 columns, up to kFixedOrderRows rows: every kFlush K steps the products so
  // far go to a second set of sums.  With fewer K splits than the kernels before
  // and no K halves, up to 224 products added to one accumulator made the logits of
  // 8B windows of 320 to 512 rows 10% less exact; so they are what they were, for
  // 0-1% of the window.  (The gate/up projection never had splits; the head's
  // and the longer forwards' order is fixed.)
  constexpr bool kSums = WN == 4 && EPI == Epi::kPart;
  constexpr int kFlush = 16;
  const bool flush = kSums && a.M <= kFixedOrderRows;
  f32x4 sum[kSums ? HB : 1][4];
#pragma unroll
  for (int i = 0; i < (kSums ? HB : 1); ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  int sx = 0, sw = 0;  // ring positions of the trip in registers
  auto next = [](int s, int n) { return s + 1 == n ? 0 : s + 1; };
  Ops pa, pb;
  // one trip: multiply `cur` (trip t), read trip t + 1 into `nxt`
#define VIA_RT_TRIP(cur, nxt)                  \
  {                                             \
    arrive();                                   \
    issue(t + (copies_w ? SW : SX), sx, sw);    \
    sx = next(sx, SX);                          \
    sw = next(sw, SW);                          \
    read(sx, sw, nxt);                          \
    mma(cur);                                   \
    VIA_RT_PIN()                                \
    ++t;                                        \
  }
  if (T > 0) {
#pragma unroll
    for (int p = 0; p < (SX > SW ? SX : SW); ++p)
      if (copies_w ? p < SW : p < SX) issue(p, p % SX, p % SW);
    // trip 0 in LDS: all but the SX (SW) - 1 youngest trips
    if (copies_w)
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(kNW * (SW - 1), 15));
    else
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(kNX * (SX - 1), 15));
    __builtin_amdgcn_s_barrier();
    read(0, 0, pa);
    int t = 0;
    for (; t + 2 < T;) {
      VIA_RT_TRIP(pa, pb)
      VIA_RT_TRIP(pb, pa)
      if constexpr (kSums)
        if (flush && t % kFlush == 0) {
#pragma unroll
          for (int i = 0; i < HB; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              sum[i][j] += acc[i][j];
              acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
    }
    if constexpr (kSums)
      if (flush)
#pragma unroll
        for (int i = 0; i < HB; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = sum[i][j] + acc[i][j];
    // one or two trips left; the last one of an odd split has no second K step
    const bool tail = s_beg + (T - 1) * KG + kg < s_end;
    if (T - t == 2) {
      VIA_RT_TRIP(pa, pb)
      if (tail) mma(pb);
    } else if (tail) {
      mma(pa);
    }
  }
#undef VIA_RT_TRIP
#undef VIA_RT_PIN
  __builtin_amdgcn_s_waitcnt(0);  // the trailing copies land before LDS is reused or the work-group ends
  const int n = lane & 15, g = lane >> 4;
  float* tl = (float*)smem;
  if constexpr (EPI == Epi::kPart && KG == 1) {
    float* P = a.part + (size_t)split * a.M * a.N;
#pragma unroll
    for (int i = 0; i < HB; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = n0 + wn * 64 + j * 16 + n;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + (wm * HB + i) * 16 + g * 4 + r;
          if (m < a.M && col < a.N) P[(size_t)m * a.N + col] = acc[i][j][r];
        }
      }
    return;
  }
  __syncthreads();
  auto cell = [&](int i, int j, int r) -> float& {
    return tl[((wm * HB + i) * 16 + g * 4 + r) * kStride + wn * 64 + j * 16 + n];
  };
  if (KG == 1 || kg == 1) {
#pragma unroll
    for (int i = 0; i < HB; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) cell(i, j, r) = acc[i][j][r];
  }
  __syncthreads();
  if constexpr (KG == 2) {
    if (kg == 0) {  // even K steps + odd K steps
#pragma unroll
      for (int i = 0; i < HB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) cell(i, j, r) = acc[i][j][r] + cell(i, j, r);
    }
    __syncthreads();
  }
  if constexpr (EPI == Epi::kPart) {
    float* P = a.part + (size_t)split * a.M * a.N;
    const int c = threadIdx.x % (kBN / 4) * 4;
    for (int r = threadIdx.x / (kBN / 4); r < 16 * MB; r += kThr / (kBN / 4)) {
      const int m = m0 + r, col = n0 + c;
      if (m >= a.M) break;
      if (col < a.N) *(float4*)(P + (size_t)m * a.N + col) = *(const float4*)(tl + r * kStride + c);  // N % 4 == 0
    }
  } else if constexpr (EPI == Epi::kSwiglu) {
    for (int e = threadIdx.x; e < 16 * MB * (kBN / 16); e += kThr) {
      const int r = e % (16 * MB), j = e / (16 * MB), m = m0 + r, f = (n0 >> 1) + j * 8;
      if (m >= a.M || f >= a.F) continue;
      const float* t = tl + r * kStride + j * 16;
      const float sc = row_scale(a.ss, a.ss_stride, m, a.K, a.eps);  // RMSNorm of the input row
      float v[8];
      {
        // h is rounded before its terms are split, as in gemm_prefill (which
        // holds it in LDS): a product fused into the split's subtraction gives
        // another last bit, and forwards of many rows take either kernel
#pragma clang fp contract(off)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float gt = t[i] * sc, up = t[8 + i] * sc;
          v[i] = gt / (1.0f + expf(-gt)) * up;
        }
      }
      put_afrag<true, 2>(a.H, m, f, v, a.F >> 5, a.MBn);
    }
  } else {
    epi_stats<MB, kBN, kStride, kThr>(a, tn, m0, tl);
  }
}

void launch_row_tile(GemmRole role, const GemmArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const RtPlan p = row_tile_plan(role, a.M, a.N, a.K);
  const int ntiles = ((a.M + p.rows - 1) / p.rows) * ((a.N + p.cols - 1) / p.cols) * a.ksplit;
  const dim3 grid((ntiles + 7) / 8 * 8);
  // 128 columns: one K group where the order of summation is fixed
  const bool one = a.M > kFixedOrderRows && p.cols == 128;
  const int threads = one ? 256 : 512;
  auto pick = [&](auto part, auto swiglu, auto stats) {
    launch_timed(role == GemmRole::kGateUp ? swiglu : role == GemmRole::kHead ? stats : part, grid, threads, a, s, e0, e1);
  };
#define VIA_RT_PICK(...)                                                                        \
  pick(gemm_row_tile<__VA_ARGS__, Epi::kPart>, gemm_row_tile<__VA_ARGS__, Epi::kSwiglu>,   \
       gemm_row_tile<__VA_ARGS__, Epi::kStats>)
  if (p.cols == 256 && p.rows == 96)
    VIA_RT_PICK(6, 4, 1, 5, 6);
  else if (p.cols == 256)
    VIA_RT_PICK(8, 4, 1, 5, 5);
  else if (one && p.rows == 64)
    VIA_RT_PICK(4, 2, 1, 6, 12);
  else if (one && p.rows == 96)
    VIA_RT_PICK(6, 2, 1, 5, 12);
  else if (one)
    VIA_RT_PICK(8, 2, 1, 5, 10);
  else if (p.rows == 64)
    VIA_RT_PICK(4, 2, 2, 3, 6);
  else if (p.rows == 96)
    VIA_RT_PICK(6, 2, 2, 4, 3);
  else
    VIA_RT_PICK(8, 2, 2, 3, 4);
#undef VIA_RT_PICK
}

void launch_prefill(const GemmArgs& a, int nt, bool swiglu, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const int ntiles = ((a.M + kPfBM - 1) / kPfBM) * ((a.N + kPfBN - 1) / kPfBN);
  const dim3 grid((ntiles + 7) / 8 * 8);
  auto go = [&](auto kernel) {
    if (e0)
      hipExtLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, e0, e1, 0, a, nt);
    else
      hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, a, nt);
  };
  if (swiglu)
    go(gemm_prefill<true, true>);
  else if (nt == 2)
    go(gemm_prefill<false, true>);
  else
    go(gemm_prefill<false, false>);
}

}  // namespace

void launch_pack(bool bf16, const void* src, void* dst, int rows, int cols, int ffn, hipStream_t s) {
  const size_t groups = (size_t)((rows + 63) / 64) * 64 * (cols / 8);
  const dim3 grid((unsigned)((groups + 255) / 256));
  if (bf16)
    hipLaunchKernelGGL(pack_kernel<uint16_t>, grid, dim3(256), 0, s, (const uint16_t*)src, (uint16_t*)dst, rows, cols,
                       ffn, groups);
  else
    hipLaunchKernelGGL(pack_kernel<float>, grid, dim3(256), 0, s, (const float*)src, (float*)dst, rows, cols, ffn,
                       groups);
}

void launch_gemm(bool bf16, GemmRole role, const GemmArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  switch (gemm_path(bf16, role, a.M, a.N, a.K)) {
    case GemmPath::kPrefill:
      // the compute-bound tile kernel (one partial, ksplit 1; the gate/up projection writes h itself)
      launch_prefill(a, 2, role == GemmRole::kGateUp, s, e0, e1);
      break;
    case GemmPath::kRowTile:
      launch_row_tile(role, a, s, e0, e1);
      break;
    case GemmPath::kStream:
      if (role == GemmRole::kGateUp)
        launch_gate_up_ki(a, s, e0, e1);
      else
        launch_ki_part(a, s, e0, e1);
      break;
    case GemmPath::kHead: launch_head(a, s, e0, e1); break;
    case GemmPath::kF32: launch_f32(role, a, s, e0, e1); break;
  }
}

void launch_gemm_bf16(const GemmArgs& a, hipStream_t s) { launch_prefill(a, 1, false, s, nullptr, nullptr); }

void launch_lm_finalize(const LmRow* lm, const float* lm_part, int n_lm, int ntiles, float inv_T, int32_t* row_argmax,
                        float* row_max, float* row_sumexp, float* row_gap, hipStream_t s) {
  hipLaunchKernelGGL(lm_finalize_kernel, dim3(n_lm), dim3(256), 0, s, lm, lm_part, n_lm, ntiles, inv_T, row_argmax,
                     row_max, row_sumexp, row_gap);
}

}  // namespace via
