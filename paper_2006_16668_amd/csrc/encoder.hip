// The Transformer encoder sub-layers around the MoE layer (Section 2.1 of the paper: a
// self-attention layer and a position-wise feed-forward layer per encoder layer, with
// residual connections and layer normalisation; every other feed-forward layer is the MoE
// layer).  This file holds the pieces that are not GEMMs:
//
//   add_layer_norm   s = x (+ delta);  n = gamma * (s - mean) / sqrt(var + eps) + beta
//   attention core   ctx[b,l,h,:] = softmax_l'( q[b,l,h,:] . k[b,l',h,:] / sqrt(d) ) v[b,l',h,:]
//                    on the output of the fused Q|K|V projection, qkv [tokens, 3*heads*d]
//
// The attention core has two forms here: a flash-style MFMA kernel (bf16, d = 64 or 128) and a plain
// one-wavefront-per-query kernel for other d and for fp32 calls of fewer than 128 queries; the fp32 one on the matrix
// cores is in attention_f32.hip.
#include <float.h>
#include <math.h>
#include <type_traits>
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

// ---------------------------------------------------------------- attention, MFMA form
// Block = 128 queries of one (sequence, head); wavefront w owns queries 32 w .. 32 w + 31.
// Everything is computed transposed so that a lane owns ONE query column:
//   S^T = K . Q^T  (keys x queries): MFMA A operand = 32 keys x 16 d, B operand = Q^T, both
//         read as 16 contiguous bytes of a qkv row.  In the result a lane holds, per 32-key
//         tile, the 16 scores of its query for the keys 8 (i/4) + 4 (lane/32) + i%4.
//   online softmax over the keys: in-lane over those scores plus one exchange with the
//         partner lane (lane ^ 32), running maximum m and sum l per query.
//   O^T += V^T . P^T (d x queries): P^T is the B operand straight from the score registers
//         (acc values 8 s .. 8 s + 7 of a tile are the 8 keys of MFMA step s); V^T is the A
//         operand, fetched with the transposing LDS read from the V block staged as
//         [keys][d] with the key rows stored in the matching order (bits 2 and 3 of the key
//         index swapped inside each 32-key tile).
// The K and V blocks (64 keys x D each) are staged through LDS once per block and step, double
// buffered, the next block waiting in registers while the current one is multiplied.  K runs one block
// ahead of V: a step multiplies the scores of the next block between the exponentials of this one, and
// requests fragments two products before their use.  Matrix pipes, vector ALU and LDS were each busy
// 25 to 45 % of the time, so what bounds the kernel is how far they overlap; two wavefronts per SIMD
// (registers allow no more) left them taking turns.  Same sums in the same order.  Self-attention
// sub-layer, 16 heads of 128, 16 x 1024 tokens: 462 -> 447 us; 4 heads of 128, 2 x 1024 tokens (one
// block per compute unit): 50 -> 44.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// RAGGED: L is no multiple of 128.  Query and key rows past the end are read from row L - 1, the
// scores of such keys become -inf before the softmax (the last key block always holds a real key),
// such queries are not stored, and a wavefront that has none but those only stages.  The
// probabilities stay fp32, as in the plain kernel that served these lengths first: P^T enters the
// product as three bf16 terms (split_bf16x8), so ctx differs from a float64 evaluation by its own
// rounding and at most 2e-7 of the sum's magnitude.  L % 128 == 0 keeps the form without these tests,
// whose probabilities are rounded to bf16 (1e-3 of that magnitude).  Self-attention sub-layer, M 1024,
// plain / one bf16 term / three: 16 x 1000 tokens, 16 heads of 128 11.2 ms / 479 us / 564 us; 4 x 1000,
// 16 of 64 1508 / 75.5 / 88.2 us; M 512, 16 x 200, 4 of 128 206 / 33.1 / 36.8 us.
template <int D, bool RAGGED>
__global__ __launch_bounds__(256, 2) void attention_mfma_kernel(
    const bf16_t* __restrict__ qkv, bf16_t* __restrict__ ctx, float* __restrict__ lse, int L,
    int heads) {
  constexpr int KS = D / 16;                 // MFMA steps over d for the scores
  constexpr int DT = D / 32;                 // 32-row tiles of O^T
  // Row pitches of the staged blocks, chosen for the 64 LDS banks: the 16-byte K reads of 16
  // consecutive rows must start 4 banks apart (pitch = 4 words mod 64), the transposing 8-byte V
  // reads of a half-wavefront touch 4 rows x 16 words (pitch = 16 words mod 64).
  constexpr int kKPitch = D * 2 + 16, kVPitch = D * 2 + 64;
  constexpr int kKTile = 64 * kKPitch;       // one staged K block of 64 keys (the V block follows it)
  constexpr int kStage = kKTile + 64 * kVPitch;
  __shared__ __attribute__((aligned(16))) unsigned char kvs[2][kStage];      // stage: K block, V block
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 31, hf = lane >> 5;
  const int qblocks = RAGGED ? (L + 127) / 128 : L / 128;
  // Consecutive workgroups go to different XCDs (8, each with its own L2): give every XCD a
  // contiguous range of work items, so the query blocks of one (sequence, head), which read
  // the same K and V rows, run under one L2.
  unsigned work = blockIdx.x;
  const unsigned per_xcd = gridDim.x / 8;
  if (work < per_xcd * 8) work = (work % 8) * per_xcd + work / 8;
  const int qb = work % qblocks;
  const long long bh = work / qblocks;
  const int h = (int)(bh % heads);
  const long long b = bh / heads;
  const int A = heads * D;
  const size_t ld = (size_t)3 * A;
  const bf16_t* base = qkv + (size_t)b * L * ld + (size_t)h * D;
  const bf16_t* kbase = base + A;
  const bf16_t* vbase = base + 2 * A;

  // Q^T fragments of this wavefront's 32 queries: lane (r, hf) holds d = 16 s + 8 hf .. + 7
  const int q = qb * 128 + wave * 32 + r;
  const bool live = !RAGGED || qb * 128 + __builtin_amdgcn_readfirstlane(wave) * 32 < L;
  const bf16_t* qrow = base + (size_t)(RAGGED && q >= L ? L - 1 : q) * ld;
  u32x4_t qf[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) qf[s] = *reinterpret_cast<const u32x4_t*>(qrow + 16 * s + 8 * hf);

  f32x16_t o[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[t][i] = 0.f;
  // running maximum (in log2 units) and sum; the maximum starts finite, so that a block of keys whose scores
  // are all -inf adds nothing
  float m_run = -FLT_MAX, l_run = 0.f;
  const float sl2 = 1.4426950408889634f / sqrtf((float)D);

  // cooperative staging of a block of 64 keys: K rows as they are, V rows in the order the
  // P^T operand needs (bits 2 and 3 of the key index swapped); 64 * D / 8 16-byte vectors each.
  // The block after the current one waits in registers while the current one is multiplied.
  constexpr int VV = 64 * D / 8 / 256;       // vectors per thread and operand
  constexpr int VPR = D / 8;                 // vectors per row
  u32x4_t kreg[VV], vreg[VV];
#define MOE_ATT_LOAD(reg, src, kb)                                                            \
  _Pragma("unroll") for (int i = 0; i < VV; ++i) {                                            \
    const int f = tid + 256 * i, c = f % VPR;                                                 \
    int key = (kb) * 64 + f / VPR;                                                            \
    if (RAGGED) key = key < L ? key : L - 1;                                                  \
    reg[i] = *reinterpret_cast<const u32x4_t*>(src + (size_t)key * ld + 8 * c);               \
  }
#define MOE_ATT_STORE_K(stage)                                                                \
  _Pragma("unroll") for (int i = 0; i < VV; ++i) {                                            \
    const int f = tid + 256 * i, key = f / VPR, c = f % VPR;                                  \
    *reinterpret_cast<u32x4_t*>(&kvs[stage][key * kKPitch + 16 * c]) = kreg[i];               \
  }
#define MOE_ATT_STORE_V(stage)                                                                \
  _Pragma("unroll") for (int i = 0; i < VV; ++i) {                                            \
    const int f = tid + 256 * i, key = f / VPR, c = f % VPR;                                  \
    const int pos = (key & ~12) | ((key & 4) << 1) | ((key & 8) >> 1); /* swap bits 2, 3 */   \
    *reinterpret_cast<u32x4_t*>(&kvs[stage][kKTile + pos * kVPitch + 16 * c]) = vreg[i];      \
  }
  const int nkb = RAGGED ? (L + 63) / 64 : L / 64;
  MOE_ATT_LOAD(kreg, kbase, 0)
  MOE_ATT_LOAD(vreg, vbase, 0)
  MOE_ATT_STORE_K(0)
  MOE_ATT_STORE_V(0)
  if (nkb > 1) {
    MOE_ATT_LOAD(kreg, kbase, 1)
    MOE_ATT_STORE_K(1)
  }
  __syncthreads();

  typedef s16x4_t __attribute__((address_space(3))) * lds_s16x4_ptr;
  typedef u32x4_t __attribute__((address_space(3))) * lds_u4_ptr;
  typedef unsigned char __attribute__((address_space(3))) * lds_ptr;
  const uint32_t kvs0 = (uint32_t)(uintptr_t)((lds_ptr)&kvs[0][0]);
  const int p16 = lane & 15, bb = lane >> 4;
  const int krow0 = 8 * (bb >> 1) + (p16 >> 2);          // staged key row inside a 16-row step
  // scores S^T of the 64 keys staged at kst: two 32-key tiles; lane (r, hf) reads 16 bytes of key row r
  f32x16_t sacc[2];
  auto scores = [&](f32x16_t (&acc)[2], uint32_t kst) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const u32x4_t kf = *(lds_u4_ptr)(uintptr_t)(kst + (32 * t + r) * kKPitch + 32 * s + 16 * hf);
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, kf),
                                                         __builtin_bit_cast(bf16x8_t, qf[s]),
                                                         acc[t], 0, 0, 0);
      }
    }
  };
  if (live) scores(sacc, kvs0);
  if (nkb > 2) __syncthreads();              // step 0 writes K block 2 where these scores read block 0
  // One block of keys.  LAST: no block follows.
  auto step = [&](int kb, auto last) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last)::value;
    if (!LAST) {
      if (kb + 2 < nkb) MOE_ATT_LOAD(kreg, kbase, kb + 2)
      MOE_ATT_LOAD(vreg, vbase, kb + 1)
    }
    const uint32_t vst = kvs0 + (kb & 1) * kStage + kKTile;
    if (live) {
      f32x16_t snext[2];
      if (!LAST) scores(snext, kvs0 + ((kb + 1) & 1) * kStage);
      if (RAGGED && LAST && kb * 64 + 64 > L) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (kb * 64 + 32 * t + 8 * (i >> 2) + 4 * hf + (i & 3) >= L) sacc[t][i] = -INFINITY;
      }
      // ---- online softmax for this lane's query (partner lane ^ 32 holds the other keys)
      float mx = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sacc[t][i]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * sl2;        // sl2 > 0: scaling commutes with max
      const float m_new = fmaxf(m_run, mx);
      float psum = 0.f;
      u32x4_t pf[2][2];                                    // P^T fragments: tile t, MFMA step s
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x16_t& p = sacc[t];                             // probabilities in the scores' place
#pragma unroll
        for (int i = 0; i < 16; ++i) { p[i] = __builtin_amdgcn_exp2f(fmaf(p[i], sl2, -m_new)); psum += p[i]; }
        if (RAGGED) continue;                              // (split where they are multiplied)
#pragma unroll
        for (int s = 0; s < 2; ++s)
          pf[t][s] = u32x4_t{pack_bf16x2(p[8 * s], p[8 * s + 1]), pack_bf16x2(p[8 * s + 2], p[8 * s + 3]),
                             pack_bf16x2(p[8 * s + 4], p[8 * s + 5]), pack_bf16x2(p[8 * s + 6], p[8 * s + 7])};
      }
      if (!LAST) {
        // a product of the next block's scores every few vector instructions of this block's softmax,
        // its fragment requested two products ahead
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
        for (int i = 0; i < 2 * KS; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 112 / KS, 0);
        }
      }
      psum += __shfl_xor(psum, 32, 64);
      // the running maximum rarely moves after the first blocks: rescale only when some query
      // of the wavefront needs it (alpha == 1 exactly otherwise)
      if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on the first block
        l_run *= alpha;
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
          for (int i = 0; i < 16; ++i) o[t][i] *= alpha;
      }
      l_run += psum;
      m_run = m_new;
      // ---- O^T += V^T . P^T: MFMA step (t, s) covers staged key rows 32 t + 16 s .. + 15
      constexpr int TERMS = RAGGED ? 3 : 1;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          bf16x8_bits_t pt[3];
          if (RAGGED) split_bf16x8(sacc[t], 8 * s, pt);
          else pt[0] = pf[t][s];
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            // lane needs V^T[d = 32 dt + lane%32][8 consecutive staged keys of its half]:
            // 16-lane block bb reads rows krow0 (+4), columns 32 dt + 16 (bb&1) + 4 (p16&3) .. +3
            const int col = 32 * dt + 16 * (bb & 1) + 4 * (p16 & 3);
            const uint32_t pv = vst + (32 * t + 16 * s + krow0) * kVPitch + 2 * col;
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)pv);
            const s16x4_t hi =
                __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(pv + 4 * kVPitch));
            const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int k = TERMS - 1; k >= 0; --k)           // smallest term first
              o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8_t, pt[k]),
                                                              o[dt], 0, 0, 0);
          }
        }
      if (!RAGGED) {
        // fragments of V two products ahead (three products per fragment leave time enough without)
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int i = 0; i < 4 * DT; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
      }
      if (!LAST) { sacc[0] = snext[0]; sacc[1] = snext[1]; }
    }
    // What the stores overwrite was last read one step ago, before the previous barrier: V block kb - 1,
    // and K block kb, whose scores step kb - 1 multiplied (the prologue before step 0, hence its barrier).
    if (!LAST) {
      if (kb + 2 < nkb) MOE_ATT_STORE_K(kb & 1)
      MOE_ATT_STORE_V((kb + 1) & 1)
      __syncthreads();
    }
  };
  for (int kb = 0; kb + 1 < nkb; ++kb) step(kb, std::false_type{});
  step(nkb - 1, std::true_type{});
#undef MOE_ATT_LOAD
#undef MOE_ATT_STORE_K
#undef MOE_ATT_STORE_V
  // o[dt][i]: d = 32 dt + 8 (i/4) + 4 hf + i%4 of query r: four consecutive d per 8-byte store
  const float inv = 1.0f / l_run;
  // row statistic for the backward pass: log sum_k exp(score) in natural-log units
  if (RAGGED && q >= L) return;
  if (lse != nullptr && hf == 0)
    lse[(size_t)bh * L + q] = (m_run + log2f(l_run)) * 0.6931471805599453f;
  bf16_t* orow = ctx + ((size_t)b * L + q) * A + (size_t)h * D;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
      const u32x2_t w = {pack_bf16x2(o[dt][4 * q4] * inv, o[dt][4 * q4 + 1] * inv),
                         pack_bf16x2(o[dt][4 * q4 + 2] * inv, o[dt][4 * q4 + 3] * inv)};
      *reinterpret_cast<u32x2_t*>(orow + 32 * dt + 8 * q4 + 4 * hf) = w;
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
  if (act_dtype == MOE_BF16 && (d == 64 || d == 128)) {
    const long long blocks = B * heads * ((L + 127) / 128);
    if (blocks > 0x7fffffffLL) return MOE_EUNSUPPORTED;
#define MOE_ATT_CASE(D, RAGGED)                                                                      \
  hipLaunchKernelGGL((attention_mfma_kernel<D, RAGGED>), dim3((unsigned)blocks), dim3(256), 0, st,  \
                     static_cast<const bf16_t*>(qkv), static_cast<bf16_t*>(ctx), lse, L, heads)
    const bool ragged = L % 128 != 0;
    if (d == 64) { if (ragged) MOE_ATT_CASE(64, true); else MOE_ATT_CASE(64, false); }
    else if (ragged) MOE_ATT_CASE(128, true);
    else MOE_ATT_CASE(128, false);
#undef MOE_ATT_CASE
    return check_launch();
  }
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
