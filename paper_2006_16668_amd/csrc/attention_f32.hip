// Scaled dot-product attention core and its backward pass in fp32 on the matrix cores (d = 64 or 128),
// v_mfma_f32_32x32x2_f32: full fp32 products and sums, exponentials with expf.  Other d, and calls of fewer
// than 128 queries, run the plain kernels of encoder.hip and encoder_bwd.hip, which took every fp32 call before.
//
// The transposed arrangement of the bf16 kernels: a lane owns one column (a query; a key in the dk/dv kernel).
// The instruction takes one k per lane half: lane (r = lane % 32, hf = lane / 32) supplies row r of the first
// operand and column r of the second at k = hf, and receives C[8 (i/4) + 4 hf + i%4][r] in value i.  So
//   sums over d       step j of a group of 8 d takes d = 8 g + 4 hf + j: both operands are 16-byte pieces of rows
//   sums over rows    value i of a score tile is the second operand of the step that takes the rows
//                     8 (i/4) + 4 hf + i%4, the first operand one float of each of those two rows, 32 neighbours
//                     per half: nothing is transposed.
// A sum over rows is taken per block of 32 rows and then added, one over d as two: fewer roundings at the size of
// the result.
//
// A block has four wavefronts.  With columns enough each has 32 of its own, and the block stages 32 rows of the two
// other operands in LDS while the next ones wait in registers.  With few columns they share 32, take the blocks
// of rows in turn, straight from memory (a head's rows stay in L2) and without barriers, and add up in LDS, in order.
//
// Bound: the matrix pipes, 64 cycles an instruction: 128 (forward), 192 (dq) and 256 (dk, dv) of them per
// wavefront, 32 columns and 32 rows at d 128; with few columns the chain of a wavefront's blocks.
// us of a launch (backward: both of them), plain kernels / these:
//   3 x 384 tokens, 16 heads of 64   281 / 37, 1161 / 129     1 x 640, 8 of 128    301 / 37, 1359 / 139
//   8 x 197, 8 of 128                225 / 38,  990 / 130     78 x 26, 8 of 64    27.6 / 11.2, 99.6 / 42.4
//   2 x 1024, 8 of 128              1307 / 111, 6956 / 426    16 x 1000, 16 of 64 8824 / 719, 39449 / 2291
// Error against float64, relative, plain / these: ctx 4.5e-7 / 2.2e-7, dq 5.6e-7 / 3.7e-7, dk and dv 5.4e-7 / 3.7e-7
// (3 x 384, 16 heads of 64; normal q, k, v).
#include <float.h>
#include <math.h>
#include "common.h"

namespace moe {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// a lane's 16-byte pieces of a row (half of its d)
template <int D> struct Pieces {
  f32x4_t v[D / 8];
  __device__ __forceinline__ void load(const float* row, int hf) {
#pragma unroll
    for (int g = 0; g < D / 8; ++g) v[g] = *reinterpret_cast<const f32x4_t*>(row + 8 * g + 4 * hf);
  }
  __device__ __forceinline__ f32x4_t piece(int g) const { return v[g]; }
};
// The floats of a block's 32 rows that the sums over rows take.  Rows past the end are copies of the last one, with a
// factor of 0.  An infinity in that row of v or dctx must not become 0 x inf there, so they are cleared before use (q and
// k need not be: their infinities make the head's scores, so all results, NaN anyway).
template <int D> struct Rows {
  float v[16][D / 32];
  __device__ __forceinline__ void load(const float* base, size_t ld, int row0, int L, int r, int hf) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      int row = row0 + 8 * (i >> 2) + 4 * hf + (i & 3);
      row = row < L ? row : L - 1;
#pragma unroll
      for (int t = 0; t < D / 32; ++t) v[i][t] = base[(size_t)row * ld + 32 * t + r];
    }
  }
  __device__ __forceinline__ void clear_past(int row0, int L, int hf) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int t = 0; t < D / 32; ++t) v[i][t] = row0 + 8 * (i >> 2) + 4 * hf + (i & 3) < L ? v[i][t] : 0.f;
  }
  __device__ __forceinline__ float at(int i, int t) const { return v[i][t]; }
};
// 32 rows staged in LDS serve as both.  Pitch: the halves of a one-float read, four rows apart, start 32 banks apart.
template <int D> struct Staged {
  static constexpr int kPitch = D + 8, kFloats = 32 * kPitch;
  const float* rows;
  int r, hf;
  __device__ __forceinline__ f32x4_t piece(int g) const {
    return *reinterpret_cast<const f32x4_t*>(rows + r * kPitch + 8 * g + 4 * hf);
  }
  __device__ __forceinline__ float at(int i, int t) const {
    return rows[(8 * (i >> 2) + 4 * hf + (i & 3)) * kPitch + 32 * t + r];
  }
};
// the rows 32 blk .. + 31 of two operands on their way to LDS (past the end: the last one on the way, zeros in LDS)
template <int D> struct Transit {
  static constexpr int kPer = 32 * D / 4 / 256, kVecs = D / 4;
  f32x4_t a[kPer], b[kPer];
  __device__ __forceinline__ void fetch(const float* pa, size_t lda, const float* pb, size_t ldb, int blk, int L) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int f = threadIdx.x + 256 * i, c = 4 * (f % kVecs);
      int row = 32 * blk + f / kVecs;
      row = row < L ? row : L - 1;
      a[i] = *reinterpret_cast<const f32x4_t*>(pa + (size_t)row * lda + c);
      b[i] = *reinterpret_cast<const f32x4_t*>(pb + (size_t)row * ldb + c);
    }
  }
  __device__ __forceinline__ void put(float* la, float* lb, int blk, int L) {
    if (32 * blk + 32 > L) {                                   // block-uniform
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const bool past = 32 * blk + (int)(threadIdx.x + 256 * i) / kVecs >= L;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          a[i][k] = past ? 0.f : a[i][k];
          b[i][k] = past ? 0.f : b[i][k];
        }
      }
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int f = threadIdx.x + 256 * i, at = f / kVecs * Staged<D>::kPitch + 4 * (f % kVecs);
      *reinterpret_cast<f32x4_t*>(la + at) = a[i];
      *reinterpret_cast<f32x4_t*>(lb + at) = b[i];
    }
  }
};
// rows x columns over d, in two sums
template <int D, typename R>
__device__ __forceinline__ f32x16_t over_d(const R& rows, const Pieces<D>& col) {
  f32x16_t c[2];
#pragma unroll
  for (int i = 0; i < 16; ++i) c[0][i] = c[1][i] = 0.f;
#pragma unroll
  for (int g = 0; g < D / 16; ++g) {
    const f32x4_t x[2] = {rows.piece(g), rows.piece(D / 16 + g)};
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        c[h] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[h][j], col.v[h * (D / 16) + g][j], c[h], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) c[0][i] += c[1][i];
  return c[0];
}
// acc[d][column] += rows^T times c
template <int D, typename R>
__device__ __forceinline__ void over_rows(f32x16_t (&acc)[D / 32], const R& rows, const f32x16_t& c) {
#pragma unroll
  for (int t = 0; t < D / 32; t += 2) {
    f32x16_t p[2];
#pragma unroll
    for (int i = 0; i < 16; ++i) p[0][i] = p[1][i] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) p[h] = __builtin_amdgcn_mfma_f32_32x32x2f32(rows.at(i, t + h), c[i], p[h], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 16; ++i) { acc[t][i] += p[0][i]; acc[t + 1][i] += p[1][i]; }
  }
}
template <int D>
__device__ __forceinline__ void clear(f32x16_t (&acc)[D / 32]) {
#pragma unroll
  for (int t = 0; t < D / 32; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
}
// acc[t][i] is d = 32 t + 8 (i/4) + 4 hf + i%4 of the lane's row
template <int D>
__device__ __forceinline__ void store_column(float* row, const f32x16_t (&acc)[D / 32], float scale, int hf) {
#pragma unroll
  for (int t = 0; t < D / 32; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<f32x4_t*>(row + 32 * t + 8 * q + 4 * hf) =
          f32x4_t{acc[t][4 * q] * scale, acc[t][4 * q + 1] * scale, acc[t][4 * q + 2] * scale, acc[t][4 * q + 3] * scale};
}

constexpr int kWaves = 4;

// What a wavefront does: 32 columns from col0 on, blocks of 32 rows from `first` on, `step` apart.
struct Work { long long bh, b; int h, col0, first, step; };
template <bool SPLIT>
__device__ __forceinline__ Work work_of(int L, int heads, int wave) {
  const int columns = SPLIT ? 32 : 32 * kWaves, per = (L + columns - 1) / columns;
  unsigned item = blockIdx.x;                                  // XCDs get contiguous ranges: a head's blocks share an L2
  const unsigned per_xcd = gridDim.x / 8;
  if (item < per_xcd * 8) item = (item % 8) * per_xcd + item / 8;
  Work w;
  w.bh = item / per;
  w.col0 = (int)(item % per) * columns + (SPLIT ? 0 : 32 * wave);
  w.b = w.bh / heads;
  w.h = (int)(w.bh % heads);
  w.first = SPLIT ? wave : 0;
  w.step = SPLIT ? kWaves : 1;
  return w;
}
// the wavefronts' sums meet in wavefront 0, in order; sums: LDS, 8 KB per 64 d and wavefront but the first
template <int D>
__device__ __forceinline__ void add_up(f32x16_t (&acc)[D / 32], float (*sums)[D / 32][16][64], int wave, int lane) {
  __syncthreads();                                             // (what they held before has been read)
  if (wave > 0) {
#pragma unroll
    for (int t = 0; t < D / 32; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) sums[wave - 1][t][i][lane] = acc[t][i];
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int w = 0; w < kWaves - 1; ++w)
#pragma unroll
      for (int t = 0; t < D / 32; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] += sums[w][t][i][lane];
  }
}

template <int D, bool SPLIT>
__global__ __launch_bounds__(64 * kWaves, D == 64 ? 2 : 1) void attention_f32_kernel(
    const float* __restrict__ qkv, float* __restrict__ ctx, float* __restrict__ lse, int L, int heads) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, hf = lane >> 5;
  const Work w = work_of<SPLIT>(L, heads, wave);
  const int A = heads * D;
  const size_t ld = (size_t)3 * A;
  const float* base = qkv + (size_t)w.b * L * ld + (size_t)w.h * D;
  const int q = w.col0 + r, qc = q < L ? q : L - 1;
  Pieces<D> qf, kf;
  qf.load(base + (size_t)qc * ld, hf);
  auto load_keys = [&](int kb) __attribute__((always_inline)) {
    const int key = 32 * kb + r;
    kf.load(base + A + (size_t)(key < L ? key : L - 1) * ld, hf);
  };
  f32x16_t o[D / 32];
  clear<D>(o);
  const float scale = 1.0f / sqrtf((float)D);
  // (the maximum starts finite: a block of keys whose scores are all -inf adds nothing)
  float m_run = -FLT_MAX, l_run = 0.f;
  const int nkb = (L + 31) / 32;
  auto softmax_block = [&](int kb, f32x16_t& p) __attribute__((always_inline)) {     // scores to probabilities
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      p[i] *= scale;
      if (32 * kb + 8 * (i >> 2) + 4 * hf + (i & 3) >= L) p[i] = -INFINITY;
      mx = fmaxf(mx, p[i]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx);
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) { p[i] = expf(p[i] - m_new); sum += p[i]; }
    sum += __shfl_xor(sum, 32, 64);
    if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
      const float alpha = expf(m_run - m_new);                 // 0 on the first block
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < D / 32; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[t][i] *= alpha;
    }
    l_run += sum;
    m_run = m_new;
  };
  if constexpr (SPLIT) {
    load_keys(w.first);                                        // (past the end: the last key)
    for (int kb = w.first; kb < nkb; kb += w.step) {
      Rows<D> vf;
      vf.load(base + 2 * A, ld, 32 * kb, L, r, hf);
      f32x16_t p = over_d<D>(kf, qf);
      load_keys(kb + w.step);
      softmax_block(kb, p);
      if (32 * kb + 32 > L) vf.clear_past(32 * kb, L, hf);     // wavefront-uniform
      over_rows<D>(o, vf, p);
    }
  } else {
    __shared__ __attribute__((aligned(16))) float ks[Staged<D>::kFloats], vs[Staged<D>::kFloats];
    Transit<D> next;
    next.fetch(base + A, ld, base + 2 * A, ld, 0, L);
    for (int kb = 0; kb < nkb; ++kb) {
      __syncthreads();                                         // the block before has been read by everyone
      next.put(ks, vs, kb, L);
      __syncthreads();
      if (kb + 1 < nkb) next.fetch(base + A, ld, base + 2 * A, ld, kb + 1, L);
      f32x16_t p = over_d<D>(Staged<D>{ks, r, hf}, qf);
      softmax_block(kb, p);
      over_rows<D>(o, Staged<D>{vs, r, hf}, p);
    }
  }
  if constexpr (SPLIT) {                                       // to the columns' common maximum, then add up
    __shared__ float stats[2][kWaves][64], sums[kWaves - 1][D / 32][16][64];
    stats[0][wave][lane] = m_run;
    stats[1][wave][lane] = l_run;
    __syncthreads();
    float m = m_run;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) m = fmaxf(m, stats[0][k][lane]);
    const float alpha = expf(m_run - m);                       // (a wavefront without a block of keys: 0 x 0)
    l_run = 0.f;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) l_run += stats[1][k][lane] * expf(stats[0][k][lane] - m);
#pragma unroll
    for (int t = 0; t < D / 32; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[t][i] *= alpha;
    m_run = m;
    add_up<D>(o, sums, wave, lane);
    if (wave > 0) return;
  }
  if (q >= L) return;
  if (lse != nullptr && hf == 0) lse[(size_t)w.bh * L + q] = m_run + logf(l_run);
  store_column<D>(ctx + ((size_t)w.b * L + q) * A + (size_t)w.h * D, o, 1.0f / l_run, hf);
}

// dq, and D = rowsum(dctx * ctx)
template <int D, bool SPLIT>
__global__ __launch_bounds__(64 * kWaves, 1) void attention_f32_bwd_dq_kernel(
    const float* __restrict__ qkv, const float* __restrict__ ctx, const float* __restrict__ dctx,
    const float* __restrict__ lse, float* __restrict__ dqkv, float* __restrict__ dvec, int L, int heads) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, hf = lane >> 5;
  const Work w = work_of<SPLIT>(L, heads, wave);
  const int A = heads * D;
  const size_t ld = (size_t)3 * A;
  const float* base = qkv + (size_t)w.b * L * ld + (size_t)w.h * D;
  const int q = w.col0 + r, qc = q < L ? q : L - 1;
  const size_t crow = ((size_t)w.b * L + qc) * A + (size_t)w.h * D;
  Pieces<D> qf, gf, kf, vf;
  qf.load(base + (size_t)qc * ld, hf);
  gf.load(dctx + crow, hf);
  kf.load(ctx + crow, hf);
  float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < D / 8; ++g)
#pragma unroll
    for (int j = 0; j < 4; ++j) part[j] = fmaf(gf.v[g][j], kf.v[g][j], part[j]);
  float dd = (part[0] + part[1]) + (part[2] + part[3]);
  dd += __shfl_xor(dd, 32, 64);
  if (hf == 0 && q < L && (!SPLIT || wave == 0)) dvec[(size_t)w.bh * L + q] = dd;
  const float ls = lse[(size_t)w.bh * L + qc];
  const float scale = 1.0f / sqrtf((float)D);
  auto load_keys = [&](int kb) __attribute__((always_inline)) {
    const int key = 32 * kb + r;
    const float* row = base + A + (size_t)(key < L ? key : L - 1) * ld;
    kf.load(row, hf);
    vf.load(row + A, hf);
  };
  f32x16_t dq[D / 32];
  clear<D>(dq);
  const int nkb = (L + 31) / 32;
  auto score_gradients = [&](int kb, const f32x16_t& s, f32x16_t& ds) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      ds[i] = expf(s[i] * scale - ls) * (ds[i] - dd) * scale;
      if (32 * kb + 8 * (i >> 2) + 4 * hf + (i & 3) >= L) ds[i] = 0.f;
    }
  };
  if constexpr (SPLIT) {
    load_keys(w.first);
    for (int kb = w.first; kb < nkb; kb += w.step) {
      Rows<D> kr;
      kr.load(base + A, ld, 32 * kb, L, r, hf);
      const f32x16_t s = over_d<D>(kf, qf);
      f32x16_t ds = over_d<D>(vf, gf);
      load_keys(kb + w.step);
      score_gradients(kb, s, ds);
      over_rows<D>(dq, kr, ds);
    }
  } else {
    __shared__ __attribute__((aligned(16))) float ks[Staged<D>::kFloats], vs[Staged<D>::kFloats];
    Transit<D> next;
    next.fetch(base + A, ld, base + 2 * A, ld, 0, L);
    for (int kb = 0; kb < nkb; ++kb) {
      __syncthreads();
      next.put(ks, vs, kb, L);
      __syncthreads();
      if (kb + 1 < nkb) next.fetch(base + A, ld, base + 2 * A, ld, kb + 1, L);
      const f32x16_t s = over_d<D>(Staged<D>{ks, r, hf}, qf);
      f32x16_t ds = over_d<D>(Staged<D>{vs, r, hf}, gf);
      score_gradients(kb, s, ds);
      over_rows<D>(dq, Staged<D>{ks, r, hf}, ds);
    }
  }
  if constexpr (SPLIT) {
    __shared__ float sums[kWaves - 1][D / 32][16][64];
    add_up<D>(dq, sums, wave, lane);
    if (wave > 0) return;
  }
  if (q >= L) return;
  store_column<D>(dqkv + ((size_t)w.b * L + q) * ld + (size_t)w.h * D, dq, 1.0f, hf);
}

// dk and dv; needs lse and D of every query of the head.  (d = 128: 12 values more than vector registers, 26 where
// wavefronts share columns; the compiler keeps them in accumulation registers, none in memory.)
template <int D, bool SPLIT>
__global__ __launch_bounds__(64 * kWaves, 1) void attention_f32_bwd_dkv_kernel(
    const float* __restrict__ qkv, const float* __restrict__ dctx, const float* __restrict__ lse,
    const float* __restrict__ dvec, float* __restrict__ dqkv, int L, int heads) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, hf = lane >> 5;
  const Work w = work_of<SPLIT>(L, heads, wave);
  const int A = heads * D;
  const size_t ld = (size_t)3 * A;
  const float* base = qkv + (size_t)w.b * L * ld + (size_t)w.h * D;
  const float* gbase = dctx + (size_t)w.b * L * A + (size_t)w.h * D;
  const float *lrow = lse + (size_t)w.bh * L, *drow = dvec + (size_t)w.bh * L;
  const int key = w.col0 + r, kc = key < L ? key : L - 1;
  Pieces<D> kf, vf, qf, gf;
  kf.load(base + (size_t)kc * ld + A, hf);
  vf.load(base + (size_t)kc * ld + 2 * A, hf);
  auto load_queries = [&](int qb) __attribute__((always_inline)) {
    const int q = 32 * qb + r < L ? 32 * qb + r : L - 1;
    qf.load(base + (size_t)q * ld, hf);
    gf.load(gbase + (size_t)q * A, hf);
  };
  const float scale = 1.0f / sqrtf((float)D);
  f32x16_t dk[D / 32], dv[D / 32];
  clear<D>(dk);
  clear<D>(dv);
  const int nqb = (L + 31) / 32;
  // scores to p, dctx v^T to ds; ls, dd: lse and D of the queries.  A query past the end has lse = inf: p = ds = 0
  auto probabilities = [&](f32x16_t& p, f32x16_t& ds, const float (&ls)[16], const float (&dd)[16]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      p[i] = expf(p[i] * scale - ls[i]);
      ds[i] = p[i] * (ds[i] - dd[i]) * scale;
      if (ls[i] == INFINITY) p[i] = ds[i] = 0.f;               // (also where a copied row's products are not finite)
    }
  };
  float ls[16], dd[16];
  if constexpr (SPLIT) {
    constexpr bool kAhead = D == 64;                           // (registers do not hold a block more at d = 128)
    if (kAhead) load_queries(w.first);
    for (int qb = w.first; qb < nqb; qb += w.step) {
      if (!kAhead) load_queries(qb);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int row = 32 * qb + 8 * (i >> 2) + 4 * hf + (i & 3), rc = row < L ? row : L - 1;
        ls[i] = row < L ? lrow[rc] : INFINITY;
        dd[i] = row < L ? drow[rc] : 0.f;
      }
      Rows<D> rows;
      if (kAhead) rows.load(gbase, (size_t)A, 32 * qb, L, r, hf);
      f32x16_t p = over_d<D>(qf, kf);
      f32x16_t ds = over_d<D>(gf, vf);
      if (kAhead) load_queries(qb + w.step);
      else rows.load(gbase, (size_t)A, 32 * qb, L, r, hf);
      probabilities(p, ds, ls, dd);
      rows.clear_past(32 * qb, L, hf);
      over_rows<D>(dv, rows, p);
      rows.load(base, ld, 32 * qb, L, r, hf);
      over_rows<D>(dk, rows, ds);
    }
  } else {
    __shared__ __attribute__((aligned(16))) float qs[Staged<D>::kFloats], gs[Staged<D>::kFloats], stats[2][32];
    Transit<D> next;
    float next_stat = 0.f;                                     // threads 0..31: lse, 32..63: D
    auto fetch = [&](int qb) __attribute__((always_inline)) {
      next.fetch(base, ld, gbase, (size_t)A, qb, L);
      const int row = 32 * qb + (threadIdx.x & 31);
      if (threadIdx.x < 32) next_stat = row < L ? lrow[row] : INFINITY;
      else if (threadIdx.x < 64) next_stat = row < L ? drow[row] : 0.f;
    };
    fetch(0);
    for (int qb = 0; qb < nqb; ++qb) {
      __syncthreads();
      next.put(qs, gs, qb, L);
      if (threadIdx.x < 64) stats[threadIdx.x >> 5][threadIdx.x & 31] = next_stat;
      __syncthreads();
      if (qb + 1 < nqb) fetch(qb + 1);
      f32x16_t p = over_d<D>(Staged<D>{qs, r, hf}, kf);
      f32x16_t ds = over_d<D>(Staged<D>{gs, r, hf}, vf);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        ls[i] = stats[0][8 * (i >> 2) + 4 * hf + (i & 3)];
        dd[i] = stats[1][8 * (i >> 2) + 4 * hf + (i & 3)];
      }
      probabilities(p, ds, ls, dd);
      over_rows<D>(dv, Staged<D>{gs, r, hf}, p);
      over_rows<D>(dk, Staged<D>{qs, r, hf}, ds);
    }
  }
  if constexpr (SPLIT) {
    __shared__ float sums[kWaves - 1][D / 32][16][64];
    add_up<D>(dk, sums, wave, lane);
    add_up<D>(dv, sums, wave, lane);
    if (wave > 0) return;
  }
  if (key >= L) return;
  float* out = dqkv + ((size_t)w.b * L + key) * ld + A + (size_t)w.h * D;
  store_column<D>(out, dk, 1.0f, hf);
  store_column<D>(out + A, dv, 1.0f, hf);
}

// Sharing columns: up to four blocks of 32 columns on a compute unit a wavefront has its SIMD to itself either
// way, and the longest chain of blocks of rows decides (`ends`: what the adding up takes, in blocks).  us, shared /
// not, forward and backward: 1 x 768, 8 heads of 64 25 / 75 and 90 / 230; 8 x 197, 8 of 128 38 / 45 and 130 / 149;
// 3 x 384, 16 of 64 37 / 42 and 139 / 129; 8 x 250, 16 of 64 38 / 32 and 138 / 97; 78 x 26, 8 of 64 12 / 11 and 51 / 42.
inline bool share_columns(long long columns, int L, double ends) {
  const int blocks = (L + 31) / 32;
  return columns <= 1024 && (double)((columns + 255) / 256) * ((blocks + 3) / 4 + ends) < blocks;
}

}  // namespace

// A handful of queries is quicker with a wavefront each (2 heads of 20: forward 4.5 us plain, 5.1 here; 6 of 77
// 13.6 plain, 11.7 here).
bool attention_f32_ok(int act_dtype, int d, long long queries) {
  return act_dtype == MOE_F32 && (d == 64 || d == 128) && queries >= 128;
}

#define MOE_ATT_F32(KERNEL, ...)                                                                                   \
  {                                                                                                                \
    const long long blocks = split ? columns : B * heads * ((L + 32 * kWaves - 1) / (32 * kWaves));                \
    if (blocks > 0x7fffffffLL) return MOE_EUNSUPPORTED;                                                            \
    const dim3 grid((unsigned)blocks), threads(64 * kWaves);                                                       \
    if (d == 64) {                                                                                                 \
      if (split) hipLaunchKernelGGL((KERNEL<64, true>), grid, threads, 0, st, __VA_ARGS__, L, heads);              \
      else hipLaunchKernelGGL((KERNEL<64, false>), grid, threads, 0, st, __VA_ARGS__, L, heads);                   \
    } else {                                                                                                       \
      if (split) hipLaunchKernelGGL((KERNEL<128, true>), grid, threads, 0, st, __VA_ARGS__, L, heads);             \
      else hipLaunchKernelGGL((KERNEL<128, false>), grid, threads, 0, st, __VA_ARGS__, L, heads);                  \
    }                                                                                                              \
  }

int launch_attention_f32(const void* qkv, void* ctx, float* lse, long long B, int L, int heads, int d,
                         hipStream_t st) {
  const long long columns = B * heads * ((L + 31) / 32);
  const bool split = share_columns(columns, L, 0.5);
  MOE_ATT_F32(attention_f32_kernel, static_cast<const float*>(qkv), static_cast<float*>(ctx), lse)
  return check_launch();
}

int launch_attention_f32_bwd(const void* qkv, const void* ctx, const void* dctx, const float* lse, void* dqkv,
                             float* dvec, long long B, int L, int heads, int d, hipStream_t st) {
  const long long columns = B * heads * ((L + 31) / 32);
  const bool split = share_columns(columns, L, 1.0);
  auto in = static_cast<const float*>(qkv);
  auto g = static_cast<const float*>(dctx);
  auto out = static_cast<float*>(dqkv);
  MOE_ATT_F32(attention_f32_bwd_dq_kernel, in, static_cast<const float*>(ctx), g, lse, out, dvec)
  MOE_ATT_F32(attention_f32_bwd_dkv_kernel, in, g, lse, dvec, out)
  return check_launch();
}

}  // namespace moe
