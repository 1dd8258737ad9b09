// The Transformer encoder sub-layers around the MoE layer (Section 2.1 of the paper: a
// self-attention layer and a position-wise feed-forward layer per encoder layer, with
// residual connections and layer normalisation; every other feed-forward layer is the MoE
// layer).  This file holds the pieces that are not GEMMs:
//
//   add_layer_norm   s = x (+ delta);  n = gamma * (s - mean) / sqrt(var + eps) + beta
//   attention core   ctx[b,l,h,:] = softmax_l'( q[b,l,h,:] . k[b,l',h,:] / sqrt(d) ) v[b,l',h,:]
//                    on the output of the fused Q|K|V projection, qkv [tokens, 3*heads*d]
//
// The attention core has a plain one-wavefront-per-query kernel here, for other d than 64 and 128 and for fp32 calls of
// fewer than 128 queries; those on the matrix cores are in attention_mfma.hip (bf16) and attention_f32.hip.
#include <math.h>
#include "common.h"

namespace moe {
namespace {

// ---------------------------------------------------------------- layer normalisation
// one wavefront per row; the row lives in registers between the two passes
template <typename T, int VPL>   // VPL: 16-byte vectors per lane (row <= 64 * VPL vectors)
__global__ __launch_bounds__(256) void add_layer_norm_kernel(
    const uint4* __restrict__ x, const uint4* __restrict__ delta, const float* __restrict__ gamma,
    const float* __restrict__ beta, uint4* __restrict__ sum_out, uint4* __restrict__ norm_out,
    int M, int vec_per_row, long long rows, float eps) {
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int lane = threadIdx.x & 63;
  constexpr int K = Vec16<T>::kElts;
  float v[VPL][K];
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < VPL; ++j) {
    const int vi = lane + 64 * j;
#pragma unroll
    for (int i = 0; i < K; ++i) v[j][i] = 0.f;
    if (vi < vec_per_row) {
      Vec16<T>::unpack(x[row * vec_per_row + vi], v[j]);
      if (delta != nullptr) {
        float d[K];
        Vec16<T>::unpack(delta[row * vec_per_row + vi], d);
#pragma unroll
        for (int i = 0; i < K; ++i) v[j][i] += d[i];
        const uint4 packed = Vec16<T>::pack(v[j]);
        sum_out[row * vec_per_row + vi] = packed;
        Vec16<T>::unpack(packed, v[j]);               // normalise the stored (rounded) sum
      }
#pragma unroll
      for (int i = 0; i < K; ++i) s += v[j][i];
    }
  }
  const float mean = wave_sum(s) / (float)M;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < VPL; ++j)
    if (lane + 64 * j < vec_per_row)
#pragma unroll
      for (int i = 0; i < K; ++i) q += (v[j][i] - mean) * (v[j][i] - mean);
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)M + eps);
#pragma unroll
  for (int j = 0; j < VPL; ++j) {
    const int vi = lane + 64 * j;
    if (vi < vec_per_row) {
      float o[K];
#pragma unroll
      for (int i = 0; i < K; ++i)
        o[i] = gamma[vi * K + i] * ((v[j][i] - mean) * rstd) + beta[vi * K + i];
      norm_out[row * vec_per_row + vi] = Vec16<T>::pack(o);
    }
  }
}

// y = a + b, 16 bytes per thread
template <typename T>
__global__ __launch_bounds__(256) void add_rows_kernel(const uint4* __restrict__ a,
                                                       const uint4* __restrict__ b,
                                                       uint4* __restrict__ y, long long vecs) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= vecs) return;
  constexpr int K = Vec16<T>::kElts;
  float fa[K], fb[K];
  Vec16<T>::unpack(a[i], fa);
  Vec16<T>::unpack(b[i], fb);
#pragma unroll
  for (int k = 0; k < K; ++k) fa[k] += fb[k];
  y[i] = Vec16<T>::pack(fa);
}

// ---------------------------------------------------------------- attention, plain form
// One wavefront per (sequence, head, query).  Scores of the whole row sit in LDS.
template <typename T>
__global__ __launch_bounds__(256) void attention_rows_kernel(
    const T* __restrict__ qkv, T* __restrict__ ctx, float* __restrict__ lse, int L, int heads, int d,
    long long queries) {
  extern __shared__ float att_smem[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float* sc = att_smem + (size_t)wave * (L + d);        // [L] scores, then [d] the query row
  float* qs = sc + L;
  const long long id = (long long)blockIdx.x * 4 + wave;   // (b * heads + h) * L + l
  if (id >= queries) return;
  const int l = (int)(id % L);
  const long long bh = id / L;
  const int h = (int)(bh % heads);
  const long long b = bh / heads;
  const int A = heads * d;
  const size_t ld = (size_t)3 * A;
  const T* qrow = qkv + ((size_t)b * L + l) * ld + (size_t)h * d;
  const T* kbase = qkv + (size_t)b * L * ld + A + (size_t)h * d;
  const T* vbase = kbase + A;
  for (int i = lane; i < d; i += 64) qs[i] = Elt<T>::load(qrow + i);
  __builtin_amdgcn_wave_barrier();
  const float scale = 1.0f / sqrtf((float)d);
  float mx = -INFINITY;
  for (int k0 = 0; k0 < L; k0 += 64) {
    const int key = k0 + lane;
    if (key < L) {
      const T* kr = kbase + (size_t)key * ld;
      float dot = 0.f;
      for (int i = 0; i < d; ++i) dot = fmaf(qs[i], Elt<T>::load(kr + i), dot);
      dot *= scale;
      sc[key] = dot;
      mx = fmaxf(mx, dot);
    }
  }
  mx = wave_max(mx);
  float sum = 0.f;
  for (int key = lane; key < L; key += 64) {
    const float p = expf(sc[key] - mx);
    sc[key] = p;
    sum += p;
  }
  sum = wave_sum(sum);
  if (lse != nullptr && lane == 0) lse[id] = mx + logf(sum);   // log sum_k exp(score), for the backward pass
  __builtin_amdgcn_wave_barrier();
  const float inv = 1.0f / sum;
  T* out = ctx + ((size_t)b * L + l) * A + (size_t)h * d;
  for (int i = lane; i < d; i += 64) {
    float acc = 0.f;
    for (int key = 0; key < L; ++key) acc = fmaf(sc[key], Elt<T>::load(vbase + (size_t)key * ld + i), acc);
    Elt<T>::store(out + i, acc * inv);
  }
}

}  // namespace

int launch_add_layer_norm(int act_dtype, const void* x, const void* delta, const float* gamma,
                          const float* beta, void* sum_out, void* norm_out, long long rows, int M,
                          hipStream_t st) {
  const int elt = act_dtype == MOE_F32 ? 4 : 2;
  const int vec_per_row = M * elt / 16;
  const int vpl = (vec_per_row + 63) / 64;
  if (vpl > 8) return MOE_EUNSUPPORTED;        // rows of more than 8192 bytes per lane set
  const unsigned grid = (unsigned)((rows + 3) / 4);
  const float eps = 1e-6f;
#define MOE_LN_CASE(T, V)                                                                     \
  hipLaunchKernelGGL((add_layer_norm_kernel<T, V>), dim3(grid), dim3(256), 0, st,             \
                     static_cast<const uint4*>(x), static_cast<const uint4*>(delta), gamma,   \
                     beta, static_cast<uint4*>(sum_out), static_cast<uint4*>(norm_out), M,    \
                     vec_per_row, rows, eps)
  if (act_dtype == MOE_F32) {
    if (vpl <= 1) MOE_LN_CASE(float, 1); else if (vpl <= 2) MOE_LN_CASE(float, 2);
    else if (vpl <= 4) MOE_LN_CASE(float, 4); else MOE_LN_CASE(float, 8);
  } else {
    if (vpl <= 1) MOE_LN_CASE(bf16_t, 1); else if (vpl <= 2) MOE_LN_CASE(bf16_t, 2);
    else if (vpl <= 4) MOE_LN_CASE(bf16_t, 4); else MOE_LN_CASE(bf16_t, 8);
  }
#undef MOE_LN_CASE
  return check_launch();
}

int launch_add_rows(int act_dtype, const void* a, const void* b, void* y, long long elems,
                    hipStream_t st) {
  const int elt = act_dtype == MOE_F32 ? 4 : 2;
  const long long vecs = elems * elt / 16;
  const unsigned grid = (unsigned)((vecs + 255) / 256);
  if (act_dtype == MOE_F32)
    hipLaunchKernelGGL(add_rows_kernel<float>, dim3(grid), dim3(256), 0, st,
                       static_cast<const uint4*>(a), static_cast<const uint4*>(b),
                       static_cast<uint4*>(y), vecs);
  else
    hipLaunchKernelGGL(add_rows_kernel<bf16_t>, dim3(grid), dim3(256), 0, st,
                       static_cast<const uint4*>(a), static_cast<const uint4*>(b),
                       static_cast<uint4*>(y), vecs);
  return check_launch();
}

// ctx [B*L, heads*d] from qkv [B*L, 3*heads*d]
int launch_attention_core(int act_dtype, const void* qkv, void* ctx, float* lse, long long B, int L,
                          int heads, int d, hipStream_t st) {
  if (attention_mfma_ok(act_dtype, L, heads, d)) return launch_attention_mfma(qkv, ctx, lse, B, L, heads, d, st);
  const size_t shm = (size_t)4 * (L + d) * sizeof(float);
  if (shm > 64 * 1024) return MOE_EUNSUPPORTED;          // sequences of more than ~4000 tokens
  if (attention_f32_ok(act_dtype, d, B * heads * L)) return launch_attention_f32(qkv, ctx, lse, B, L, heads, d, st);
  const long long queries = B * heads * L;
  const long long blocks = (queries + 3) / 4;
  if (blocks > 0x7fffffffLL) return MOE_EUNSUPPORTED;
  if (act_dtype == MOE_F32)
    hipLaunchKernelGGL(attention_rows_kernel<float>, dim3((unsigned)blocks), dim3(256), shm, st,
                       static_cast<const float*>(qkv), static_cast<float*>(ctx), lse, L, heads, d, queries);
  else
    hipLaunchKernelGGL(attention_rows_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), shm, st,
                       static_cast<const bf16_t*>(qkv), static_cast<bf16_t*>(ctx), lse, L, heads, d, queries);
  return check_launch();
}

}  // namespace moe
