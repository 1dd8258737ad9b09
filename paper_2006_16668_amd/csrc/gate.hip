// Top2Gating (Algorithm 1 of the paper, for G independent groups) in three kernels:
//
//   gate_topk_kernel    per token: logits x.wg, softmax, top-2, renormalised gates,
//                       the random-routing decision; per 64-token chunk: histogram of
//                       first choices / sampled second choices and the gate sums
//   gate_scan_kernel    per group: exclusive scan of the chunk histograms over the
//                       chunks (the running counters c_E of Algorithm 1 at chunk
//                       boundaries), c1, mean gates m_E, fill, empty slots
//   gate_slots_kernel   per chunk: stable rank of every token among the earlier
//                       tokens of its chunk with the same expert + the chunk base
//                       = position in the expert buffer; capacity test; combine
//                       weights; inverse map slot -> token; l_aux
//
// Calls of few chunks run the last two as one (gate_route_kernel).
//
// bf16 activations take the MFMA form of the first kernel (gate_mfma_*): x is
// exactly bf16, so with wg split into three bf16 terms (hi + mid + lo = all 24
// mantissa bits) every product is exact in fp32 and only the accumulation order
// differs from a plain fp32 dot product.  wg is repacked (by the caller once per
// weight update, else once per call) into the lane order of the
// v_mfma_f32_32x32x16_bf16 B operand, so each B load is one contiguous 1 KB read.
// Gates that leave compute units idle and fp32 gates take gate_chunk_kernel (one chunk
// per block, the features split over its wavefronts).  Gates wider than 512 experts and
// fp32 gates wider than 128 with GEMM-friendly shapes get their logits from the
// persistent GEMM kernel; everything else keeps the plain FMA kernel.
//
// Positions never come from atomics: they are exact counts of earlier tokens, so
// the result equals the sequential two-pass loop of Algorithm 1 bit for bit.
#include <limits.h>
#include <math.h>
#include "common.h"

namespace moe {

namespace {

__device__ __forceinline__ void argmax_merge(float& bv, int& bi, float ov, int oi) {
  if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
}
__device__ __forceinline__ void wave_argmax(float& bv, int& bi) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    float ov = __shfl_xor(bv, o, 64);
    int oi = __shfl_xor(bi, o, 64);
    argmax_merge(bv, bi, ov, oi);
  }
}

// A token with fewer than two logits above -inf (infinities or NaN in its row of x, or overflow): what is
// missing of its two choices goes to the lowest other index, as a tie would.  Every later kernel addresses
// memory with these indices, so they are valid whatever x holds.
__device__ __forceinline__ void complete_choices(int& e1, int& e2) {
  if (e1 == INT_MAX) e1 = 0;
  if (e2 == INT_MAX) e2 = e1 == 0 ? 1 : 0;
}

// One block = one chunk of 64 tokens of one group; wave w takes tokens w, w+4, ...
// Lane l owns experts l, l+64, ... (EPL of them).
// PRE: the logits were computed beforehand on the matrix cores (very wide gates): zpre
// [tokens, cols] holds, for expert e, the three partial logits x . (hi, mid, lo term of wg) in
// columns 3e, 3e+1, 3e+2; they are added smallest term first.
template <typename T, int EPL, bool PRE>
__global__ __launch_bounds__(256) void gate_topk_kernel(
    const T* __restrict__ x, const float* __restrict__ wg, const float* __restrict__ u,
    const float* __restrict__ zpre, int cols, int S, int M, int E, int nch,
    int32_t* __restrict__ expert_idx, int32_t* __restrict__ slot, float* __restrict__ weight,
    float* __restrict__ gates_opt,
    int32_t* __restrict__ hist1, int32_t* __restrict__ hist2, float* __restrict__ msum) {
  extern __shared__ unsigned char smem[];
  const int g = blockIdx.x / nch, ch = blockIdx.x % nch;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float* xs = reinterpret_cast<float*>(smem) + (size_t)wave * M;  // this wave's token row
  float* msum_l = reinterpret_cast<float*>(smem) + (PRE ? 0 : (size_t)4 * M);  // [4][E]
  int* h1 = reinterpret_cast<int*>(msum_l + (size_t)4 * E);
  int* h2 = h1 + E;
  for (int e = threadIdx.x; e < E; e += 256) { h1[e] = 0; h2[e] = 0; }

  float macc[EPL];
#pragma unroll
  for (int j = 0; j < EPL; ++j) macc[j] = 0.f;

  for (int it = 0; it < kChunk / 4; ++it) {
    const int s = ch * kChunk + it * 4 + wave;
    const bool valid = s < S;
    const size_t n = (size_t)g * S + (valid ? s : 0);
    __syncthreads();  // previous row fully consumed (also orders the histogram zeroing)
    if (!PRE)
      for (int m = lane; m < M; m += 64) xs[m] = Elt<T>::load(x + n * M + m);
    __syncthreads();
    if (!valid) continue;  // both barriers of the next iteration are still reached

    float z[EPL];
#pragma unroll
    for (int j = 0; j < EPL; ++j) z[j] = 0.f;
    if (PRE) {
      const float* zp = zpre + n * cols;
#pragma unroll
      for (int j = 0; j < EPL; ++j) {
        const int e = lane + 64 * j;
        if (e < E) z[j] = (zp[3 * e + 2] + zp[3 * e + 1]) + zp[3 * e];
      }
    } else {
      for (int m = 0; m < M; ++m) {
        const float xv = xs[m];
        const float* wrow = wg + (size_t)m * E;
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
          const int e = lane + 64 * j;
          if (e < E) z[j] = fmaf(xv, wrow[e], z[j]);
        }
      }
    }
    // top-2 on the logits (softmax is monotone); ties go to the lowest index
    float v1 = -INFINITY; int e1 = INT_MAX;
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      const int e = lane + 64 * j;
      if (e < E) argmax_merge(v1, e1, z[j], e);
    }
    wave_argmax(v1, e1);
    float v2 = -INFINITY; int e2 = INT_MAX;
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      const int e = lane + 64 * j;
      if (e < E && e != e1) argmax_merge(v2, e2, z[j], e);
    }
    wave_argmax(v2, e2);
    complete_choices(e1, e2);

    // softmax over all experts (needed for the mean gates m_E)
    float p[EPL], psum = 0.f;
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      const int e = lane + 64 * j;
      p[j] = (e < E) ? expf(z[j] - v1) : 0.f;
      psum += p[j];
    }
    psum = wave_sum(psum);
    const float inv = 1.0f / psum;
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      const int e = lane + 64 * j;
      const float gate = p[j] * inv;
      macc[j] += gate;
      if (gates_opt != nullptr && e < E) gates_opt[n * E + e] = gate;
    }
    // g1/(g1+g2) and g2/(g1+g2): the softmax denominator cancels
    const float p2 = expf(v2 - v1);
    const float g1n = 1.0f / (1.0f + p2);
    const float g2n = p2 / (1.0f + p2);
    const bool sampled = 2.0f * g2n > u[n];
    if (lane == 0) {
      expert_idx[2 * n] = e1;
      expert_idx[2 * n + 1] = e2;
      weight[2 * n] = g1n;          // provisional: zeroed later if the slot is lost
      weight[2 * n + 1] = g2n;
      slot[2 * n + 1] = sampled ? 0 : MOE_SLOT_NOT_SAMPLED;
      atomicAdd(&h1[e1], 1);
      if (sampled) atomicAdd(&h2[e2], 1);
    }
  }

#pragma unroll
  for (int j = 0; j < EPL; ++j) {
    const int e = lane + 64 * j;
    if (e < E) msum_l[(size_t)wave * E + e] = macc[j];
  }
  __syncthreads();
  const size_t base = ((size_t)g * nch + ch) * E;
  for (int e = threadIdx.x; e < E; e += 256) {
    msum[base + e] = ((msum_l[e] + msum_l[E + e]) + msum_l[2 * (size_t)E + e]) + msum_l[3 * (size_t)E + e];
    hist1[base + e] = h1[e];
    hist2[base + e] = h2[e];
  }
}

// ----------------------------------------------------------------------------
// MFMA form for bf16 activations
// ----------------------------------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// K order inside a block of 64 model features: MFMA step j (0..3), lane half h,
// element i  <->  feature 32 h + 8 j + i.  A lane of the A operand then owns 64
// contiguous bytes of its token row per block (four 16-byte loads).
//
// wgP[ks][t][split][lane] (uint4 = 8 bf16): B operand of step ks = 4 kb + j for
// the 32 experts of column tile t; lane = 32 h + c holds expert 32 t + c.
__global__ __launch_bounds__(256) void gate_pack_wg_kernel(
    const float* __restrict__ wg, uint4* __restrict__ wgP, int M, int E, int T, int total) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const int lane = idx & 63, t = (idx >> 6) % T, ks = (idx >> 6) / T;
  const int h = lane >> 5, col = 32 * t + (lane & 31);
  const int m0 = (ks >> 2) * 64 + 32 * h + 8 * (ks & 3);
  uint32_t w[3][4];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int m = m0 + i;
    const float v = (m < M && col < E) ? wg[(size_t)m * E + col] : 0.f;
    const bf16_t hi = f32_to_bf16(v);
    const float r1 = v - bf16_to_f32(hi);          // exact
    const bf16_t mid = f32_to_bf16(r1);
    const float r2 = r1 - bf16_to_f32(mid);        // exact
    const bf16_t lo = f32_to_bf16(r2);
    const bf16_t parts[3] = {hi, mid, lo};
#pragma unroll
    for (int sp = 0; sp < 3; ++sp) {
      if (i & 1) w[sp][i >> 1] |= (uint32_t)parts[sp] << 16;
      else w[sp][i >> 1] = parts[sp];
    }
  }
#pragma unroll
  for (int sp = 0; sp < 3; ++sp)
    wgP[((size_t)(ks * T + t) * 3 + sp) * 64 + lane] = uint4{w[sp][0], w[sp][1], w[sp][2], w[sp][3]};
}

struct Top2 { float v1; int e1; float v2; int e2; };

__device__ __forceinline__ bool better(float a, int ia, float b, int ib) {
  return a > b || (a == b && ia < ib);
}
__device__ __forceinline__ Top2 top2_merge(const Top2& a, const Top2& b) {
  // winner = better first entry; runner-up = better of the loser's first and the winner's second
  const bool bw = better(b.v1, b.e1, a.v1, a.e1);
  const float wv1 = bw ? b.v1 : a.v1, lv1 = bw ? a.v1 : b.v1, wv2 = bw ? b.v2 : a.v2;
  const int we1 = bw ? b.e1 : a.e1, le1 = bw ? a.e1 : b.e1, we2 = bw ? b.e2 : a.e2;
  const bool lb = better(lv1, le1, wv2, we2);
  Top2 r;
  r.v1 = wv1; r.e1 = we1;
  r.v2 = lb ? lv1 : wv2; r.e2 = lb ? le1 : we2;
  return r;
}

// Softmax / top-2 / random routing / chunk statistics for the 64 tokens of one chunk whose
// logits sit in LDS (zs, row pitch `pitch` floats, pitch = 8 mod 64).  NT threads, TPT = NT/64
// per token; a wavefront holds 64/TPT tokens (lane % (64/TPT)) and thread `sub` = lane / (64/TPT)
// of a token owns the 4-expert groups sub, sub + TPT, ...: its 16-byte reads and those of the
// 15 lanes around it fall into different banks.  A token's logits are processed in registers
// and its gates written back for the column sums.  EXACT: library exponentials (fp32 layers).  Must be
// called by all threads of the block; ends with a barrier.
template <int NT, int EPAD, bool EXACT = false>
__device__ __forceinline__ void gate_chunk_epilogue(
    float* zs, int pitch, int g, int ch, int S, int E, int nch, const float* __restrict__ u,
    int32_t* __restrict__ expert_idx, int32_t* __restrict__ slot, float* __restrict__ weight,
    float* __restrict__ gates_opt, int32_t* __restrict__ hist1, int32_t* __restrict__ hist2,
    float* __restrict__ msum, int* h1, int* h2) {
  constexpr int TPT = NT / 64, TPW = 64 / TPT, EPT = EPAD / TPT, NG = EPT / 4;
  static_assert(EPT % 4 == 0 && EPT >= 4, "whole 4-expert groups per thread");
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  __shared__ float mpart[8 * EPAD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tk = wave * TPW + lane % TPW, sub = lane / TPW;
  const int s = ch * kChunk + tk;
  const bool valid = s < S;
  const size_t n = (size_t)g * S + (valid ? s : 0);
  const float u_n = u[n];                              // needed last: its latency hides below
  for (int e = tid; e < E; e += NT) { h1[e] = 0; h2[e] = 0; }
  float* zr = zs + (size_t)tk * pitch;
  float z[EPT];
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const f32x4_t v = *reinterpret_cast<const f32x4_t*>(zr + 4 * (sub + TPT * i));
#pragma unroll
    for (int k = 0; k < 4; ++k) z[4 * i + k] = v[k];
  }
  Top2 t2{-INFINITY, INT_MAX, -INFINITY, INT_MAX};
#pragma unroll
  for (int i = 0; i < NG; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int e = 4 * (sub + TPT * i) + k;
      const float zv = z[4 * i + k];
      if (e < E) {   // a thread meets its experts in ascending order: strict > keeps the lowest index of a tie
        if (zv > t2.v1) { t2.v2 = t2.v1; t2.e2 = t2.e1; t2.v1 = zv; t2.e1 = e; }
        else if (zv > t2.v2) { t2.v2 = zv; t2.e2 = e; }
      }
    }
#pragma unroll
  for (int o = TPW; o < 64; o <<= 1) {
    Top2 other;
    other.v1 = __shfl_xor(t2.v1, o, 64); other.e1 = __shfl_xor(t2.e1, o, 64);
    other.v2 = __shfl_xor(t2.v2, o, 64); other.e2 = __shfl_xor(t2.e2, o, 64);
    t2 = top2_merge(t2, other);
  }
  complete_choices(t2.e1, t2.e2);
  // softmax (bulk exponentials: the hardware exp2 path, relative error ~1e-6 at most over the
  // range a softmax tail can reach); rows past the end of the group count as zeros
  float psum = 0.f;
#pragma unroll
  for (int i = 0; i < NG; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float d = z[4 * i + k] - t2.v1;
      const float p = 4 * (sub + TPT * i) + k < E ? (EXACT ? expf(d) : __expf(d)) : 0.f;
      z[4 * i + k] = p;
      psum += p;
    }
#pragma unroll
  for (int o = TPW; o < 64; o <<= 1) psum += __shfl_xor(psum, o, 64);
  const float inv = valid ? 1.0f / psum : 0.f;
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    f32x4_t v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = z[4 * i + k] * inv;
    *reinterpret_cast<f32x4_t*>(zr + 4 * (sub + TPT * i)) = v;
    if (gates_opt != nullptr && valid) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (4 * (sub + TPT * i) + k < E) gates_opt[n * E + 4 * (sub + TPT * i) + k] = v[k];
    }
  }
  __syncthreads();                                     // histograms cleared, gates in LDS
  if (sub == 0 && valid) {
    const float p2 = expf(t2.v2 - t2.v1);
    const float g1n = 1.0f / (1.0f + p2);
    const float g2n = p2 / (1.0f + p2);
    const bool sampled = 2.0f * g2n > u_n;
    expert_idx[2 * n] = t2.e1;
    expert_idx[2 * n + 1] = t2.e2;
    weight[2 * n] = g1n;            // provisional: zeroed later if the slot is lost
    weight[2 * n + 1] = g2n;
    slot[2 * n + 1] = sampled ? 0 : MOE_SLOT_NOT_SAMPLED;
    atomicAdd(&h1[t2.e1], 1);
    if (sampled) atomicAdd(&h2[t2.e2], 1);
  }
  const size_t base = ((size_t)g * nch + ch) * E;
  // Gate sums of the chunk in a fixed order: eight interleaved partial sums over the 64 rows
  // (partial q takes rows q, q + 8, ...), then a tree.  tpe = 8, 4, 2 or 1 threads share the
  // partial sums of one expert.
  int tpe = 8;
  while (tpe * E > NT) tpe >>= 1;
  {
    const int e = tid / tpe, j = tid - e * tpe;
    if (e < E)
      for (int q = j; q < 8; q += tpe) {
        float part = 0.f;
#pragma unroll
        for (int r0 = 0; r0 < kChunk; r0 += 8) part += zs[(size_t)(r0 + q) * pitch + e];
        mpart[8 * e + q] = part;
      }
  }
  __syncthreads();
  for (int e = tid; e < E; e += NT) {
    const float* pp = mpart + 8 * e;
    msum[base + e] = ((pp[0] + pp[1]) + (pp[2] + pp[3])) + ((pp[4] + pp[5]) + (pp[6] + pp[7]));
    hist1[base + e] = h1[e];
    hist2[base + e] = h2[e];
  }
  __syncthreads();
}

#define MOE_GATE_MFMA(A, B, C) __builtin_amdgcn_mfma_f32_32x32x16_bf16( \
    __builtin_bit_cast(bf16x8_t, A), __builtin_bit_cast(bf16x8_t, B), C, 0, 0, 0)

// Narrow gates (E <= 64), two chunks per block: 128 tokens, wavefront w owns quarter w of the feature
// dimension and all four 32-token row tiles, so that one fetch of a packed weight fragment
// (3 KB per MFMA step from L2) feeds 12 MFMAs instead of 3: with one chunk per block the
// weight fragments cost three times the L2 traffic of x itself.  x goes from global memory
// straight into the A operand, two 64-feature blocks ahead, re-requested row tile by row tile
// as the MFMAs free the registers; the four partial sums meet in LDS.  The epilogue works in
// registers: two lanes per token read the four partial sums of half a row each (added in a fixed
// order), so softmax, top-2 and the routing decision need no further pass over LDS; the chunk's
// gate sums are wavefront butterflies over the 32 tokens of a wavefront, then one addition of
// the chunk's two wavefronts.
template <int ET>
__global__ __launch_bounds__(256) void gate_mfma_rows_kernel(
    const bf16_t* __restrict__ x, const uint4* __restrict__ wgP, const float* __restrict__ u,
    int S, int M, int E, int nch,
    int32_t* __restrict__ expert_idx, int32_t* __restrict__ slot, float* __restrict__ weight,
    float* __restrict__ gates_opt,
    int32_t* __restrict__ hist1, int32_t* __restrict__ hist2, float* __restrict__ msum) {
  // pitch = 4 mod 32 floats: the 16-byte reads of 16 lanes (16 token rows, same columns) fall
  // into 16 different bank groups
  constexpr int Epad = 32 * ET, pitch = Epad + 4, PD = 2, EPT = Epad / 2;
  extern __shared__ __attribute__((aligned(16))) unsigned char gate_smem[];
  float* part = reinterpret_cast<float*>(gate_smem);            // [4][128 * pitch]
  float* msw = part + 4 * 128 * pitch;                           // [4 wavefronts][Epad] gate sums
  int* hh = reinterpret_cast<int*>(msw + 4 * Epad);              // [2 chunks][2][Epad] histograms
  const int npair = (nch + 1) / 2;
  const int g = blockIdx.x / npair, pr = blockIdx.x % npair;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 31, h = lane >> 5;
  // epilogue role: token 32 wave + (lane % 16) + 16 (lane / 32), half (lane / 16) % 2 of its experts;
  // its random number is requested before everything else
  const int tk = 32 * wave + (lane & 15) + 16 * (lane >> 5), sub = (lane >> 4) & 1;
  const int s_ep = pr * 128 + tk;
  const bool valid = s_ep < S;
  const size_t n_ep = (size_t)g * S + (valid ? s_ep : 0);
  const float u_n = u[n_ep];
  for (int i = threadIdx.x; i < 4 * Epad; i += 256) hh[i] = 0;   // ordered by the barrier after the K loop

  const bf16_t* xrow[4];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) {
    int s = pr * 128 + 32 * rt + r;
    s = s < S ? s : S - 1;                            // clamp: surplus rows are ignored later
    xrow[rt] = x + ((size_t)g * S + s) * M;
  }
  const int KB = (M + 63) / 64, KBq = (KB + 3) / 4;
  const int kb0 = wave * KBq < KB ? wave * KBq : KB;
  const int kb1 = kb0 + KBq < KB ? kb0 + KBq : KB;

  f32x16_t acc[4][ET];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int t = 0; t < ET; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[rt][t][i] = 0.f;

  // Loads are unconditional: a block index past this wavefront's range is clamped (its
  // data is never multiplied) and features past M read the row start instead (they meet
  // zero weights in the packed operand).
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  u32x4_t a[PD][4][4];
#define MOE_GATE_LOAD_XROW(P, KBI, rt)                                                \
  {                                                                                   \
    int kbc_ = (KBI) < kb1 ? (KBI) : kb1 - 1;                                         \
    kbc_ = kbc_ < 0 ? 0 : kbc_;                                                       \
    _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                   \
      const int col_ = kbc_ * 64 + 32 * h + 8 * j;                                    \
      a[P][rt][j] = *reinterpret_cast<const u32x4_t*>(xrow[rt] + (col_ < M ? col_ : 0)); \
    }                                                                                 \
  }
  // (two column tiles leave no registers for a pinned schedule: the compiler places the loads)
#define MOE_GATE_FENCE if (ET == 1) __builtin_amdgcn_sched_barrier(0);
  // Vector loads come back in the order they were issued, so a weight fragment requested
  // just before its MFMA would wait behind every x row requested earlier (HBM latency each
  // time).  The weight fragments of a whole super-block of SB feature blocks are therefore
  // requested first (they hit in L2), then the x rows, PD blocks ahead of their use.  The
  // fences keep the compiler from moving the loads to their uses.
  constexpr int SB = 4 / ET;
  for (int sb0 = kb0; sb0 < kb1; sb0 += SB) {
    u32x4_t b[SB][4][ET * 3];
#pragma unroll
    for (int q = 0; q < SB; ++q) {
      const int cur = sb0 + q < kb1 ? sb0 + q : kb1 - 1;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u32x4_t* bp = reinterpret_cast<const u32x4_t*>(wgP) + (size_t)((cur * 4 + j) * ET) * 3 * 64 + lane;
#pragma unroll
        for (int t = 0; t < ET * 3; ++t) b[q][j][t] = bp[t * 64];
      }
    }
#pragma unroll
    for (int p = 0; p < PD; ++p)
#pragma unroll
      for (int rt = 0; rt < 4; ++rt) MOE_GATE_LOAD_XROW(p, sb0 + p, rt)
    MOE_GATE_FENCE
#pragma unroll
    for (int q = 0; q < SB; ++q) {
      const bool live = sb0 + q < kb1;                // wave-uniform
#pragma unroll
      for (int rt = 0; rt < 4; ++rt) {
        if (live) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < ET; ++t) {
              acc[rt][t] = MOE_GATE_MFMA(a[q % PD][rt][j], b[q][j][t * 3 + 2], acc[rt][t]);
              acc[rt][t] = MOE_GATE_MFMA(a[q % PD][rt][j], b[q][j][t * 3 + 1], acc[rt][t]);
              acc[rt][t] = MOE_GATE_MFMA(a[q % PD][rt][j], b[q][j][t * 3 + 0], acc[rt][t]);
            }
        }
        MOE_GATE_FENCE
        if (q + PD < SB) MOE_GATE_LOAD_XROW(q % PD, sb0 + q + PD, rt)
        MOE_GATE_FENCE
      }
    }
  }
#undef MOE_GATE_LOAD_XROW
#undef MOE_GATE_FENCE
  // acc[rt][t][i]: token row 32 rt + 8 (i/4) + 4 h + i%4, expert 32 t + r
  float* dst = part + (size_t)wave * 128 * pitch;
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int t = 0; t < ET; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        dst[(32 * rt + 8 * (i >> 2) + 4 * h + (i & 3)) * pitch + 32 * t + r] = acc[rt][t][i];
  __syncthreads();

  // ---- epilogue: logits of experts [EPT sub, EPT sub + EPT) of token tk, in registers
  float z[EPT];
  {
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    const float* zr = part + (size_t)tk * pitch + EPT * sub;
#pragma unroll
    for (int i4 = 0; i4 < EPT / 4; ++i4) {
      const f32x4_t p0 = *reinterpret_cast<const f32x4_t*>(zr + 4 * i4);
      const f32x4_t p1 = *reinterpret_cast<const f32x4_t*>(zr + 128 * pitch + 4 * i4);
      const f32x4_t p2 = *reinterpret_cast<const f32x4_t*>(zr + 2 * 128 * pitch + 4 * i4);
      const f32x4_t p3 = *reinterpret_cast<const f32x4_t*>(zr + 3 * 128 * pitch + 4 * i4);
#pragma unroll
      for (int k = 0; k < 4; ++k) z[4 * i4 + k] = (p0[k] + p1[k]) + (p2[k] + p3[k]);
    }
  }
  const int ebase = EPT * sub;
  Top2 t2{-INFINITY, INT_MAX, -INFINITY, INT_MAX};
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int e = ebase + k;
    if (e < E) {     // ascending order: strict > keeps the lowest index of a tie
      if (z[k] > t2.v1) { t2.v2 = t2.v1; t2.e2 = t2.e1; t2.v1 = z[k]; t2.e1 = e; }
      else if (z[k] > t2.v2) { t2.v2 = z[k]; t2.e2 = e; }
    }
  }
  {
    Top2 other;
    other.v1 = __shfl_xor(t2.v1, 16, 64); other.e1 = __shfl_xor(t2.e1, 16, 64);
    other.v2 = __shfl_xor(t2.v2, 16, 64); other.e2 = __shfl_xor(t2.e2, 16, 64);
    t2 = top2_merge(t2, other);
  }
  complete_choices(t2.e1, t2.e2);
  // softmax numerators (bulk exponentials: the hardware exp2 path, relative error ~1e-6 at most
  // over the range a softmax tail can reach)
  float psum = 0.f;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    z[k] = ebase + k < E ? __expf(z[k] - t2.v1) : 0.f;
    psum += z[k];
  }
  psum += __shfl_xor(psum, 16, 64);
  const float inv = valid ? 1.0f / psum : 0.f;        // rows past the end of the group count as zeros
#pragma unroll
  for (int k = 0; k < EPT; ++k) z[k] *= inv;          // the gates
  if (gates_opt != nullptr && valid) {
#pragma unroll
    for (int k = 0; k < EPT; ++k)
      if (ebase + k < E) gates_opt[n_ep * E + ebase + k] = z[k];
  }
  int* h1 = hh + (wave >> 1) * 2 * Epad;              // the histograms of this wavefront's chunk
  int* h2 = h1 + Epad;
  if (sub == 0 && valid) {
    const float p2 = expf(t2.v2 - t2.v1);
    const float g1n = 1.0f / (1.0f + p2);
    const float g2n = p2 / (1.0f + p2);
    const bool sampled = 2.0f * g2n > u_n;
    expert_idx[2 * n_ep] = t2.e1;
    expert_idx[2 * n_ep + 1] = t2.e2;
    weight[2 * n_ep] = g1n;          // provisional: zeroed later if the slot is lost
    weight[2 * n_ep + 1] = g2n;
    slot[2 * n_ep + 1] = sampled ? 0 : MOE_SLOT_NOT_SAMPLED;
    atomicAdd(&h1[t2.e1], 1);
    if (sampled) atomicAdd(&h2[t2.e2], 1);
  }
  // gate sums over the 32 tokens of the wavefront (butterfly over the lanes with the same half:
  // a fixed order), then over the two wavefronts of a chunk
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    float v = z[k];
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 4, 64);
    v += __shfl_xor(v, 8, 64);
    v += __shfl_xor(v, 32, 64);
    z[k] = v;
  }
  if ((lane & 47) == 0) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) msw[wave * Epad + ebase + k] = z[k];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * Epad; i += 256) {
    const int c = i / Epad, e = i - c * Epad, ch = 2 * pr + c;
    if (ch < nch && e < E) {
      const size_t base = ((size_t)g * nch + ch) * E;
      msum[base + e] = msw[2 * c * Epad + e] + msw[(2 * c + 1) * Epad + e];
      hist1[base + e] = hh[c * 2 * Epad + e];
      hist2[base + e] = hh[c * 2 * Epad + Epad + e];
    }
  }
}

// Wide gates (64 < E <= 512): the NW wavefronts of a block share 128 tokens (staged
// through LDS, double buffered) and each owns ETW column tiles of 32 experts.  The
// packed weights go from L2 straight into the B operand, PB MFMA steps ahead of their use.
template <int ETW, int NW, int PB>
__global__ __launch_bounds__(64 * NW) void gate_mfma_cols_kernel(
    const bf16_t* __restrict__ x, const uint4* __restrict__ wgP, const float* __restrict__ u,
    int S, int M, int E, int nch,
    int32_t* __restrict__ expert_idx, int32_t* __restrict__ slot, float* __restrict__ weight,
    float* __restrict__ gates_opt,
    int32_t* __restrict__ hist1, int32_t* __restrict__ hist2, float* __restrict__ msum) {
  constexpr int NT = 64 * NW, T = ETW * NW, Epad = 32 * T, pitch = Epad + 8;   // 8 mod 64: see the epilogue
  constexpr int AV = 1024 / NT;                        // 16-byte vectors of x per thread and block
  constexpr int kAPitch = 72;                          // 64 + 8 bf16: 16-byte pad
  constexpr int kABytes = 2 * 128 * kAPitch * 2;       // two stages
  constexpr int kZBytes = 64 * pitch * 4;              // logits of one chunk
  constexpr int kUnion = kABytes > kZBytes ? kABytes : kZBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kUnion];
  __shared__ int hh[2 * Epad];
  bf16_t* As = reinterpret_cast<bf16_t*>(smem);
  float* zs = reinterpret_cast<float*>(smem);
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

  const int npair = (nch + 1) / 2;
  const int g = blockIdx.x / npair, pr = blockIdx.x % npair;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 31, h = lane >> 5;
  const int KB = (M + 63) / 64;

  // cooperative x loads: 128 rows x 64 features = 1024 16-byte vectors per block of features;
  // rows past S are clamped (never used), features past M read the row start (zero weights)
  const int lrow = tid >> 3, lvec = tid & 7;           // rows lrow + (NT/8) i
  const bf16_t* xrow[AV];
#pragma unroll
  for (int i = 0; i < AV; ++i) {
    int s = pr * 128 + lrow + (NT / 8) * i;
    s = s < S ? s : S - 1;
    xrow[i] = x + ((size_t)g * S + s) * M;
  }
  f32x16_t acc[4][ETW];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int t = 0; t < ETW; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[rt][t][i] = 0.f;

  // B operand of MFMA step ks (= 4 kb + j), column tile t, split sp: ring of four register
  // sets, slot ks & 3, filled PB steps ahead of its use
  const u32x4_t* bbase = reinterpret_cast<const u32x4_t*>(wgP) + (size_t)wave * ETW * 3 * 64 + lane;
  const int KS = 4 * KB;
  u32x4_t bq[4][ETW * 3];
#define MOE_GATE_LOAD_B(P, ks)                                                           \
  {                                                                                      \
    const int ksc_ = (ks) < KS ? (ks) : KS - 1;                                          \
    _Pragma("unroll") for (int q = 0; q < ETW * 3; ++q)                                  \
      bq[P][q] = bbase[((size_t)ksc_ * T * 3 + q) * 64];                                 \
  }
  // x: stage kb & 1 of LDS is multiplied while blocks kb+1 .. kb+3 sit in (or fly to)
  // register sets (kb+1)&3 .. (kb+3)&3 and block kb+4 is requested into set kb & 3:
  // a load has three iterations to land before it is written to LDS
  u32x4_t areg[4][AV];
#define MOE_GATE_LOAD_A(P, kb)                                                           \
  _Pragma("unroll") for (int i = 0; i < AV; ++i) {                                       \
    const int kbc_ = (kb) < KB ? (kb) : KB - 1;                                          \
    const int col_ = kbc_ * 64 + lvec * 8;                                               \
    areg[P][i] = *reinterpret_cast<const u32x4_t*>(xrow[i] + (col_ < M ? col_ : 0));     \
  }
#define MOE_GATE_STORE_A(P, buf)                                                         \
  _Pragma("unroll") for (int i = 0; i < AV; ++i)                                         \
    *reinterpret_cast<u32x4_t*>(As + (buf) * 128 * kAPitch +                             \
                                (lrow + (NT / 8) * i) * kAPitch + lvec * 8) = areg[P][i];
#define MOE_GATE_KBLOCK(kb, Q) /* Q = kb & 3 */                                          \
  {                                                                                      \
    MOE_GATE_LOAD_A(Q, (kb) + 4)                                                         \
    const bf16_t* as = As + ((Q) & 1) * 128 * kAPitch + r * kAPitch + 32 * h;            \
    _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                      \
      MOE_GATE_LOAD_B((j + PB) & 3, (kb) * 4 + j + PB)                                   \
      u32x4_t af[4];                                                                     \
      _Pragma("unroll") for (int rt = 0; rt < 4; ++rt)                                   \
        af[rt] = *reinterpret_cast<const u32x4_t*>(as + rt * 32 * kAPitch + 8 * j);      \
      _Pragma("unroll") for (int t = 0; t < ETW; ++t)                                    \
        _Pragma("unroll") for (int rt = 0; rt < 4; ++rt) {                               \
          acc[rt][t] = MOE_GATE_MFMA(af[rt], bq[j][t * 3 + 2], acc[rt][t]);              \
          acc[rt][t] = MOE_GATE_MFMA(af[rt], bq[j][t * 3 + 1], acc[rt][t]);              \
          acc[rt][t] = MOE_GATE_MFMA(af[rt], bq[j][t * 3 + 0], acc[rt][t]);              \
        }                                                                                \
    }                                                                                    \
    MOE_GATE_STORE_A(((Q) + 1) & 3, ((Q) + 1) & 1) /* block kb+1 (a clamped copy at the end) */ \
    __syncthreads();                                                                     \
  }

  MOE_GATE_LOAD_A(0, 0)
  MOE_GATE_STORE_A(0, 0)
  MOE_GATE_LOAD_A(1, 1)
  MOE_GATE_LOAD_A(2, 2)
  MOE_GATE_LOAD_A(3, 3)
#pragma unroll
  for (int p = 0; p < PB; ++p) MOE_GATE_LOAD_B(p, p)
  __syncthreads();
  for (int kb = 0; kb < KB; kb += 4) {
    MOE_GATE_KBLOCK(kb, 0)
    if (kb + 1 < KB) MOE_GATE_KBLOCK(kb + 1, 1)
    if (kb + 2 < KB) MOE_GATE_KBLOCK(kb + 2, 2)
    if (kb + 3 < KB) MOE_GATE_KBLOCK(kb + 3, 3)
  }
#undef MOE_GATE_KBLOCK
#undef MOE_GATE_LOAD_A
#undef MOE_GATE_STORE_A
#undef MOE_GATE_LOAD_B
  // the A stages are dead from here on; the same LDS holds one chunk of logits at a time
#pragma unroll 1
  for (int c = 0; c < 2; ++c) {
    const int ch = pr * 2 + c;
    if (ch >= nch) break;                              // block-uniform
#pragma unroll
    for (int rr = 0; rr < 2; ++rr)
#pragma unroll
      for (int t = 0; t < ETW; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          zs[(rr * 32 + 8 * (i >> 2) + 4 * h + (i & 3)) * pitch + (wave * ETW + t) * 32 + r] =
              c == 0 ? acc[rr][t][i] : acc[2 + rr][t][i];
    __syncthreads();
    gate_chunk_epilogue<NT, Epad>(zs, pitch, g, ch, S, E, nch, u, expert_idx, slot, weight, gates_opt,
                            hist1, hist2, msum, hh, hh + Epad);
  }
}
// Wide gates, 64 < E <= 256: as gate_mfma_cols_kernel, but the x rows are fetched by four
// extra wavefronts that do nothing else.  Vector loads of one wavefront return in issue order,
// so in a wavefront that fetches both, every L2-resident weight fragment requested after an x
// block waits for that block's HBM latency; split by role, the multiplying wavefronts only wait
// for L2.  The loader wavefronts keep a ring of RD feature blocks in flight (global -> registers
// -> LDS stage); both roles pass the same barriers, one per 64-feature block.
// RT 32-token row tiles per block (4 or 8): with 256 tokens a weight fragment from L2 feeds 8 MFMA
// groups instead of 4, i.e. half the L2 traffic per token (one column tile per wavefront only:
// the accumulators of 8 x 2 tiles would fill the register file).
template <int ETW, int PB, int RB, int RT = 4>   // RB: ring of B register sets (power of two), PB < RB steps ahead
__global__ __launch_bounds__(512) void gate_mfma_cols_split_kernel(
    const bf16_t* __restrict__ x, const uint4* __restrict__ wgP, const float* __restrict__ u,
    int S, int M, int E, int nch,
    int32_t* __restrict__ expert_idx, int32_t* __restrict__ slot, float* __restrict__ weight,
    float* __restrict__ gates_opt,
    int32_t* __restrict__ hist1, int32_t* __restrict__ hist2, float* __restrict__ msum) {
  constexpr int NW = 4, NT = 512, T = ETW * NW, Epad = 32 * T, pitch = Epad + 8;   // 8 mod 64: see the epilogue
  constexpr int ROWS = 32 * RT, CPB = RT / 2;          // tokens and chunks per block
  constexpr int AV = RT, RD = 32 / RT;                 // loader: 16-byte vectors per thread and block, ring depth
  constexpr int kAPitch = 72;                          // 64 + 8 bf16: 16-byte pad
  constexpr int kABytes = 2 * ROWS * kAPitch * 2;      // two stages
  constexpr int kZBytes = 64 * pitch * 4;              // logits of one chunk
  constexpr int kUnion = kABytes > kZBytes ? kABytes : kZBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kUnion];
  __shared__ int hh[2 * Epad];
  bf16_t* As = reinterpret_cast<bf16_t*>(smem);
  float* zs = reinterpret_cast<float*>(smem);
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

  const int npair = (nch + CPB - 1) / CPB;
  const int g = blockIdx.x / npair, pr = blockIdx.x % npair;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int KB = (M + 63) / 64;

  f32x16_t acc[RT][ETW];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int t = 0; t < ETW; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[rt][t][i] = 0.f;

  if (wave >= NW) {
    // ---- loader wavefronts: ROWS rows x 64 features = 8 ROWS 16-byte vectors per feature block;
    // rows past S are clamped (never used), features past M read the row start (zero weights)
    const int lt = tid - 64 * NW, lrow = lt >> 3, lvec = lt & 7;   // rows lrow + 32 i
    const bf16_t* xrow[AV];
#pragma unroll
    for (int i = 0; i < AV; ++i) {
      int s = pr * ROWS + lrow + 32 * i;
      s = s < S ? s : S - 1;
      xrow[i] = x + ((size_t)g * S + s) * M;
    }
    u32x4_t areg[RD][AV];
#define MOE_GATE_LOAD_A(P, kb)                                                           \
  _Pragma("unroll") for (int i = 0; i < AV; ++i) {                                       \
    const int kbc_ = (kb) < KB ? (kb) : KB - 1;                                          \
    const int col_ = kbc_ * 64 + lvec * 8;                                               \
    areg[P][i] = *reinterpret_cast<const u32x4_t*>(xrow[i] + (col_ < M ? col_ : 0));     \
  }
#define MOE_GATE_STORE_A(P, buf)                                                         \
  _Pragma("unroll") for (int i = 0; i < AV; ++i)                                         \
    *reinterpret_cast<u32x4_t*>(As + (buf) * ROWS * kAPitch + (lrow + 32 * i) * kAPitch + lvec * 8) = areg[P][i];
    MOE_GATE_LOAD_A(0, 0)
#pragma unroll
    for (int p = 1; p < RD; ++p) MOE_GATE_LOAD_A(p, p)
    MOE_GATE_STORE_A(0, 0)
    __syncthreads();
    for (int kb0 = 0; kb0 < KB; kb0 += RD) {
#pragma unroll
      for (int q = 0; q < RD; ++q) {
        if (kb0 + q < KB) {                            // block-uniform
          // block kb0+q is being multiplied from stage q&1: its ring slot is free again, and
          // block kb0+q+1 (a clamped copy at the end) goes into the other stage
          MOE_GATE_LOAD_A(q, kb0 + q + RD)
          MOE_GATE_STORE_A((q + 1) % RD, (q + 1) & 1)
          __syncthreads();
        }
      }
    }
#undef MOE_GATE_LOAD_A
#undef MOE_GATE_STORE_A
  } else {
    // ---- multiplying wavefronts: B operand of MFMA step ks (= 4 kb + j), column tile t, split
    // sp: ring of RB register sets, slot ks % RB, filled PB steps ahead of its use
    const u32x4_t* bbase = reinterpret_cast<const u32x4_t*>(wgP) + (size_t)wave * ETW * 3 * 64 + lane;
    const int KS = 4 * KB;
    u32x4_t bq[RB][ETW * 3];
#define MOE_GATE_LOAD_B(P, ks)                                                           \
  {                                                                                      \
    const int ksc_ = (ks) < KS ? (ks) : KS - 1;                                          \
    _Pragma("unroll") for (int q = 0; q < ETW * 3; ++q)                                  \
      bq[P][q] = bbase[((size_t)ksc_ * T * 3 + q) * 64];                                 \
  }
#pragma unroll
    for (int p = 0; p < PB; ++p) MOE_GATE_LOAD_B(p, p)
    __syncthreads();
    constexpr int KU = RB / 4;                          // feature blocks per trip: slots stay static
    for (int kb0 = 0; kb0 < KB; kb0 += KU) {
#pragma unroll
      for (int ku = 0; ku < KU; ++ku) {
        const int kb = kb0 + ku;
        if (kb < KB) {                                  // block-uniform
          const bf16_t* as = As + (kb & 1) * ROWS * kAPitch + r * kAPitch + 32 * h;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            MOE_GATE_LOAD_B((4 * ku + j + PB) % RB, kb * 4 + j + PB)
            u32x4_t af[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
              af[rt] = *reinterpret_cast<const u32x4_t*>(as + rt * 32 * kAPitch + 8 * j);
#pragma unroll
            for (int t = 0; t < ETW; ++t)
#pragma unroll
              for (int sp = 2; sp >= 0; --sp)           // smallest term first; RT independent MFMAs in a row
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                  acc[rt][t] = MOE_GATE_MFMA(af[rt], bq[(4 * ku + j) % RB][t * 3 + sp], acc[rt][t]);
          }
          __syncthreads();
        }
      }
    }
#undef MOE_GATE_LOAD_B
  }
  // the A stages are dead from here on; the same LDS holds one chunk of logits at a time
#pragma unroll
  for (int c = 0; c < CPB; ++c) {
    const int ch = pr * CPB + c;
    if (ch < nch) {                                    // block-uniform
      if (wave < NW) {
#pragma unroll
        for (int rr = 0; rr < 2; ++rr)
#pragma unroll
          for (int t = 0; t < ETW; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i)
              zs[(rr * 32 + 8 * (i >> 2) + 4 * h + (i & 3)) * pitch + (wave * ETW + t) * 32 + r] =
                  acc[2 * c + rr][t][i];
      }
      __syncthreads();
      gate_chunk_epilogue<NT, Epad>(zs, pitch, g, ch, S, E, nch, u, expert_idx, slot, weight, gates_opt,
                              hist1, hist2, msum, hh, hh + Epad);
    }
  }
}
// What gate_scan_kernel and gate_slots_kernel do, for a single chunk in all (G == 1, S <= 64): the block
// that routed the chunk has every count in LDS.  h1 / h2: its histograms (LDS), ms: its gate sums;
// the routing record is the one the block has just written (a barrier in between).  NT threads.
template <int NT>
__device__ __forceinline__ void gate_single_chunk_finish(
    int S, int E, int C, const int* h1, const int* h2, const float* __restrict__ ms,
    int32_t* expert_idx, int32_t* slot, float* weight, int32_t* __restrict__ src_token,
    int32_t* __restrict__ c1, float* __restrict__ mean_gate, int32_t* __restrict__ fill,
    float* __restrict__ aux, uint32_t* __restrict__ zero_fill, int zero_words, const RowPacking& pk) {
  const int tid = threadIdx.x, lane = tid & 63;
  const bool packing = pk.packed_src != nullptr;
  for (int i = tid; i < zero_words; i += NT) zero_fill[i] = 0u;
  for (int e = tid; e < E; e += NT) {
    const int tot = h1[e] + h2[e], f = tot < C ? tot : C;
    c1[e] = h1[e];
    mean_gate[e] = ms[e] / (float)S;
    fill[e] = f;
    if (packing) {
      pk.row_base[e] = 0;
      pk.kept[e] = f;
    }
  }
  for (long long i = tid; i < (long long)E * C; i += NT) {
    const int e = (int)(i / C), c = (int)(i - (long long)e * C);
    if (c >= h1[e] + h2[e]) src_token[i] = -1;
  }
  if (tid >= 64) return;                               // one wavefront = the chunk's tokens
  float part = 0.f;
  for (int e = lane; e < E; e += 64) part += ((float)h1[e] / (float)S) * (ms[e] / (float)S);
  part = wave_sum(part);
  if (lane == 0) aux[0] = part / (float)E;
  const bool valid = lane < S;
  int e1 = -1, e2 = -1;
  bool sampled = false;
  if (valid) {
    e1 = expert_idx[2 * lane];
    sampled = slot[2 * lane + 1] != MOE_SLOT_NOT_SAMPLED;
    if (sampled) e2 = expert_idx[2 * lane + 1];
  }
  unsigned long long peers1 = __ballot(e1 >= 0), peers2 = __ballot(e2 >= 0);
  for (int bit = 0; (E - 1) >> bit; ++bit) {           // ranks as in gate_slots_kernel
    const bool b1 = (e1 >> bit) & 1, b2 = (e2 >> bit) & 1;
    const unsigned long long m1 = __ballot(b1), m2 = __ballot(b2);
    peers1 &= b1 ? m1 : ~m1;
    peers2 &= b2 ? m2 : ~m2;
  }
  if (!valid) return;
  const unsigned long long earlier = (1ull << lane) - 1;
  const int p1 = __popcll(peers1 & earlier);
  const int s1 = p1 < C ? p1 : MOE_SLOT_OVERFLOW;
  int s2 = MOE_SLOT_NOT_SAMPLED;
  if (sampled) {
    const int p2 = h1[e2] + __popcll(peers2 & earlier);
    s2 = p2 < C ? p2 : MOE_SLOT_OVERFLOW;
  }
  slot[2 * lane] = s1;
  slot[2 * lane + 1] = s2;
  if (s1 < 0) weight[2 * lane] = 0.f;
  if (s2 < 0) weight[2 * lane + 1] = 0.f;
  if (s1 >= 0) {
    src_token[(size_t)e1 * C + s1] = lane;
    if (packing) pk.packed_src[(size_t)e1 * C + s1] = lane;
  }
  if (s2 >= 0) {
    src_token[(size_t)e2 * C + s2] = lane;
    if (packing) pk.packed_src[(size_t)e2 * C + s2] = lane;
  }
}

// One 64-token chunk per block, eight wavefronts: KW of them share the features, 8 / KW the column
// tiles of 32 experts (ETW each).  Takes the gates that would leave compute units idle or have no
// matrix form otherwise:
//   bf16, E <= 64, at most one chunk per compute unit: the 128-token blocks of gate_mfma_rows_kernel
//     (their weight traffic pays once the chip is full) would use half the units and walk a quarter
//     of the features serially.  Whole gate, launches included: 3500 tokens, M 768, E 24: 19.9 ->
//     14.8 us; 16384 tokens, M 1024, E 32 (a chunk on every unit): 22.7 -> 18.5 us; 8192 tokens,
//     E 64: 27.6 -> 22.2 us.
//   fp32, E <= 128: full fp32 products on v_mfma_f32_32x32x2_f32, wg read as it is.  64 tokens, M 32,
//     E 4: 68.6 us with the FMA kernel (a wavefront walks the features for one token at a time) ->
//     6.9 us; 3000 tokens, M 1024, E 100: 3378 -> 56 us; 32 768 tokens, M 1024, E 32: 250 us with x
//     split into bf16 terms, a logit GEMM and a softmax pass -> 45 us.
// A call with a single chunk in all (a server's step) finishes here, no scan and no slots kernel: 64
// tokens, M 1024, E 32: 16.9 -> 10.6 us.
// TAIL: fp32 and M % 32 != 0.  RAW: bf16 and wg as it is, split into its three terms on the way to the products: a
// chunk's wavefronts together read each weight once, so packing them first (a launch of 4 to 5 us) does not
// pay for one call (gate_splits_wg says where it does).  Training step of 4 x 1024 tokens, M 512, H 2048, E 16
// 211.0 -> 203.3 us.
template <typename T, int ETW, int KW, bool TAIL, bool RAW>
__global__ __launch_bounds__(512) void gate_chunk_kernel(
    const T* __restrict__ x, const uint4* __restrict__ wgP, const float* __restrict__ wg,
    const float* __restrict__ u, int S, int M, int E, int C, int nch, int32_t* expert_idx, int32_t* slot,
    float* weight, float* __restrict__ gates_opt, int32_t* __restrict__ hist1,
    int32_t* __restrict__ hist2, float* msum, int32_t* __restrict__ src_token,
    int32_t* __restrict__ c1, float* __restrict__ mean_gate, int32_t* __restrict__ fill,
    float* __restrict__ aux, uint32_t* __restrict__ zero_fill, int zero_words, RowPacking pk, int single) {
  constexpr int NT = 512, CW = 8 / KW, T32 = ETW * CW, Epad = 32 * T32, pitch = Epad + 8;  // 8 mod 32
  constexpr bool F32 = sizeof(T) == 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char gate_smem[];
  float* part = reinterpret_cast<float*>(gate_smem);             // [KW][64 * pitch]
  int* hh = reinterpret_cast<int*>(part + (size_t)KW * 64 * pitch);
  const int g = blockIdx.x / nch, ch = blockIdx.x % nch;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int kw = wave % KW, cw = wave / KW;

  const T* xrow[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    int s = ch * kChunk + 32 * rt + r;
    s = s < S ? s : S - 1;                              // clamp: surplus rows are ignored later
    xrow[rt] = x + ((size_t)g * S + s) * M;
  }
  f32x16_t acc[2][ETW];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int t = 0; t < ETW; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[rt][t][i] = 0.f;

  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  // feature blocks: 64 bf16 (lane half h owns 32, in the packed operand's order) or 32 fp32 (half h
  // owns 16), 64 bytes of the token row per lane; features past M read the row start and meet zeros (TAIL:
  // are made zeros themselves, so that an infinity at the row start stays one)
  constexpr int FB = F32 ? 32 : 64, PV = 16 / sizeof(T);
  const int KB = (M + FB - 1) / FB, per = (KB + KW - 1) / KW;
  const int kb0 = kw * per, kb1 = kb0 + per < KB ? kb0 + per : KB;
  // the loads of NB feature blocks go out together, behind a fence that keeps the compiler from moving
  // them to their uses (a block past the range is read again and not multiplied)
  constexpr int NB = !F32 && ETW == 2 ? 1 : 2;
  for (int kb = kb0; kb < kb1; kb += NB) {
    u32x4_t a[NB][2][4];
    float bf[NB][F32 ? 16 : 32][ETW];
    u32x4_t bp[NB][4][ETW * 3];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int cur = kb + n < kb1 ? kb + n : kb;
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int col = cur * FB + FB / 2 * h + PV * j;
          a[n][rt][j] = *reinterpret_cast<const u32x4_t*>(xrow[rt] + (col < M ? col : 0));
        }
      if constexpr (F32) {
#pragma unroll
        for (int q = 0; q < 16; ++q)
#pragma unroll
          for (int t = 0; t < ETW; ++t) {
            const int m = cur * FB + 16 * h + q, e = 32 * (cw * ETW + t) + r;
            bf[n][q][t] = wg[m < M && e < E ? (size_t)m * E + e : 0];
          }
      } else if constexpr (RAW) {
#pragma unroll
        for (int q = 0; q < 32; ++q)
#pragma unroll
          for (int t = 0; t < ETW; ++t) {
            const int m = cur * FB + 32 * h + q, e = 32 * (cw * ETW + t) + r;
            bf[n][q][t] = wg[m < M && e < E ? (size_t)m * E + e : 0];
          }
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const u32x4_t* p = reinterpret_cast<const u32x4_t*>(wgP) +
                             ((size_t)(cur * 4 + j) * T32 + cw * ETW) * 3 * 64 + lane;
#pragma unroll
          for (int t = 0; t < ETW * 3; ++t) bp[n][j][t] = p[t * 64];
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      if (kb + n >= kb1) break;                         // wave-uniform
      if constexpr (F32) {
        if (TAIL)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if ((kb + n) * FB + FB / 2 * h + PV * j >= M) a[n][0][j] = a[n][1][j] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
        for (int q = 0; q < 16; ++q)
#pragma unroll
          for (int t = 0; t < ETW; ++t) {
            const float b = (kb + n) * FB + 16 * h + q < M && 32 * (cw * ETW + t) + r < E ? bf[n][q][t] : 0.f;
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
              acc[rt][t] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[n][rt][q >> 2][q & 3]), b,
                                                                acc[rt][t], 0, 0, 0);
          }
      } else {
        if constexpr (RAW) {                            // the terms of gate_pack_wg_kernel
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < ETW; ++t)
#pragma unroll
              for (int i = 0; i < 8; i += 2) {
                const bool col = 32 * (cw * ETW + t) + r < E;
                const int m = (kb + n) * FB + 32 * h + 8 * j + i;
                float v0 = col && m < M ? bf[n][8 * j + i][t] : 0.f, v1 = col && m + 1 < M ? bf[n][8 * j + i + 1][t] : 0.f;
#pragma unroll
                for (int sp = 0; sp < 3; ++sp) {
                  const uint32_t w = pack_bf16x2(v0, v1);
                  bp[n][j][t * 3 + sp][i / 2] = w;
                  v0 -= __uint_as_float(w << 16);       // exact
                  v1 -= __uint_as_float(w & 0xffff0000u);
                }
              }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int t = 0; t < ETW; ++t)
#pragma unroll
            for (int sp = 2; sp >= 0; --sp)             // smallest term first
#pragma unroll
              for (int rt = 0; rt < 2; ++rt)
                acc[rt][t] = MOE_GATE_MFMA(a[n][rt][j], bp[n][j][t * 3 + sp], acc[rt][t]);
      }
    }
  }
  // acc[rt][t][i]: token row 32 rt + 8 (i/4) + 4 h + i%4, expert 32 (cw ETW + t) + r
  float* dst = part + (size_t)kw * 64 * pitch;
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int t = 0; t < ETW; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        dst[(32 * rt + 8 * (i >> 2) + 4 * h + (i & 3)) * pitch + 32 * (cw * ETW + t) + r] = acc[rt][t][i];
  __syncthreads();
  // the KW partial sums in a fixed order, into the first
  for (int i = threadIdx.x; i < 64 * (Epad / 4); i += NT) {
    float* p = part + (i / (Epad / 4)) * pitch + 4 * (i % (Epad / 4));
    f32x4_t v = *reinterpret_cast<const f32x4_t*>(p);
#pragma unroll
    for (int k = 1; k < KW; ++k) v += *reinterpret_cast<const f32x4_t*>(p + (size_t)k * 64 * pitch);
    *reinterpret_cast<f32x4_t*>(p) = v;
  }
  __syncthreads();
  gate_chunk_epilogue<NT, Epad, F32>(part, pitch, g, ch, S, E, nch, u, expert_idx, slot, weight, gates_opt,
                                     hist1, hist2, msum, hh, hh + Epad);
  if (single)
    gate_single_chunk_finish<NT>(S, E, C, hh, hh + Epad, msum, expert_idx, slot, weight, src_token, c1,
                                 mean_gate, fill, aux, zero_fill, zero_words, pk);
}
#undef MOE_GATE_MFMA

// One block per (group, 32 experts); thread (e, k) owns expert e and the k-th of 8
// contiguous segments of the chunk axis.  hist1/hist2 are replaced by their exclusive
// prefix over chunks; hist2's prefix starts at c1 (second choices queue behind all first
// choices).  Two passes over the segment (sum, then prefix) with a tiny LDS scan between.
__global__ __launch_bounds__(256) void gate_scan_kernel(
    int S, int E, int C, int G, int nch,
    int32_t* __restrict__ hist1, int32_t* __restrict__ hist2, const float* __restrict__ msum,
    int32_t* __restrict__ c1, float* __restrict__ mean_gate, int32_t* __restrict__ fill,
    int32_t* __restrict__ src_token) {
  __shared__ int t1[8][32], t2[8][32];
  __shared__ float tm[8][32];
  const int etiles = (E + 31) / 32;
  const int g = blockIdx.x / etiles, e = (blockIdx.x % etiles) * 32 + (threadIdx.x & 31);
  const int k = threadIdx.x >> 5;
  const int seg = (nch + 7) / 8;
  const int ch0 = k * seg, ch1 = (ch0 + seg < nch) ? ch0 + seg : nch;
  const bool live = e < E;
  // the loads of a batch of UN chunks are independent (one memory latency per batch); a segment
  // that fits one batch stays in registers for the second pass
  constexpr int UN = 8;
  const bool single = seg <= UN;
  int a1[UN], a2[UN];
  int s1 = 0, s2 = 0;
  float ms = 0.f;
  if (live)
    for (int c0 = ch0; c0 < ch1; c0 += UN) {
      float am[UN];
#pragma unroll
      for (int j = 0; j < UN; ++j) {
        const bool in = c0 + j < ch1;
        const size_t i = ((size_t)g * nch + (in ? c0 + j : ch0)) * E + e;
        a1[j] = in ? hist1[i] : 0;
        a2[j] = in ? hist2[i] : 0;
        am[j] = in ? msum[i] : 0.f;
      }
#pragma unroll
      for (int j = 0; j < UN; ++j) {
        s1 += a1[j];
        s2 += a2[j];
        if (c0 + j < ch1) ms += am[j];                // chunk order, as a plain loop would add
      }
    }
  t1[k][threadIdx.x & 31] = s1;
  t2[k][threadIdx.x & 31] = s2;
  tm[k][threadIdx.x & 31] = ms;
  __syncthreads();
  if (!live) return;
  int base1 = 0, base2 = 0, tot1 = 0, tot2 = 0;
  float mtot = 0.f;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    const int a = t1[kk][threadIdx.x & 31], b = t2[kk][threadIdx.x & 31];
    if (kk < k) { base1 += a; base2 += b; }
    tot1 += a;
    tot2 += b;
    mtot += tm[kk][threadIdx.x & 31];
  }
  int run1 = base1, run2 = base2 + tot1;
  for (int c0 = ch0; c0 < ch1; c0 += UN) {
    if (!single) {
#pragma unroll
      for (int j = 0; j < UN; ++j) {
        const bool in = c0 + j < ch1;
        const size_t i = ((size_t)g * nch + (in ? c0 + j : ch0)) * E + e;
        a1[j] = in ? hist1[i] : 0;
        a2[j] = in ? hist2[i] : 0;
      }
    }
#pragma unroll
    for (int j = 0; j < UN; ++j)
      if (c0 + j < ch1) {
        const size_t i = ((size_t)g * nch + c0 + j) * E + e;
        hist1[i] = run1; run1 += a1[j];
        hist2[i] = run2; run2 += a2[j];
      }
  }
  const long long tot = (long long)tot1 + tot2;
  const int f = tot < C ? (int)tot : C;
  if (k == 0) {
    c1[(size_t)g * E + e] = tot1;
    mean_gate[(size_t)g * E + e] = mtot / (float)S;
    fill[(size_t)g * E + e] = f;
  }
  int32_t* st = src_token + ((size_t)e * G + g) * C;
  for (int c = f + k; c < C; c += 8) st[c] = -1;
}

// row_base[g,e] = sum of fill over the groups before g, kept[e] = over all, for layers of many groups: block = 32
// experts, thread (e, k) walks the k-th of 32 segments of the groups, twice (sum, then prefix), loads in
// batches of eight.
__global__ __launch_bounds__(1024) void gate_row_base_kernel(int G, int E, const int32_t* __restrict__ fill,
                                                             int32_t* __restrict__ row_base,
                                                             int32_t* __restrict__ kept) {
  __shared__ int part[32][33];
  constexpr int UN = 8;
  const int c = threadIdx.x & 31, k = threadIdx.x >> 5, e = 32 * blockIdx.x + c;
  const int seg = (G + 31) / 32, g0 = k * seg < G ? k * seg : G, g1 = g0 + seg < G ? g0 + seg : G;
  const bool live = e < E;
  int sum = 0;
  if (live)
    for (int gg = g0; gg < g1; gg += UN) {
      int f[UN];
#pragma unroll
      for (int j = 0; j < UN; ++j) f[j] = gg + j < g1 ? fill[(size_t)(gg + j) * E + e] : 0;
#pragma unroll
      for (int j = 0; j < UN; ++j) sum += f[j];
    }
  part[k][c] = sum;
  __syncthreads();
  if (!live) return;
  int run = 0;
  for (int i = 0; i < k; ++i) run += part[i][c];
  for (int gg = g0; gg < g1; gg += UN) {
    int f[UN];
#pragma unroll
    for (int j = 0; j < UN; ++j) f[j] = gg + j < g1 ? fill[(size_t)(gg + j) * E + e] : 0;
#pragma unroll
    for (int j = 0; j < UN; ++j)
      if (gg + j < g1) {
        row_base[(size_t)(gg + j) * E + e] = run;
        run += f[j];
      }
  }
  if (k == 31) kept[e] = run;
}

// One wavefront per chunk.  pk.packed_src != NULL: also builds the packed row layout of the
// expert GEMMs (row of a kept choice = kept rows of the same expert in earlier groups + slot);
// BASED: gate_row_base_kernel has summed the groups, else every block does so for itself.
template <bool BASED>
__global__ __launch_bounds__(64) void gate_slots_kernel(
    int S, int E, int C, int G, int nch,
    const int32_t* __restrict__ base1, const int32_t* __restrict__ base2,
    const int32_t* __restrict__ expert_idx, int32_t* __restrict__ slot,
    float* __restrict__ weight, int32_t* __restrict__ src_token,
    const int32_t* __restrict__ c1, const float* __restrict__ mean_gate, float* __restrict__ aux,
    uint32_t* __restrict__ zero_fill, int zero_words, const int32_t* __restrict__ fill, RowPacking pk) {
  const int g = blockIdx.x / nch, ch = blockIdx.x % nch;
  const int lane = threadIdx.x;
  const bool packing = pk.packed_src != nullptr, summing = packing && !BASED;
  // optional: clear the all-zero activation row that stands in for empty expert slots when
  // the first expert GEMM gathers its rows from x
  if (blockIdx.x == 0)
    for (int i = lane; i < zero_words; i += 64) zero_fill[i] = 0u;
  if (ch == 0) {
    // l_aux[g] = (1/E) sum_e (c1/S) m_e, summed in a fixed order (lane-strided, then a tree)
    float part = 0.f;
    for (int e = lane; e < E; e += 64)
      part += ((float)c1[(size_t)g * E + e] / (float)S) * mean_gate[(size_t)g * E + e];
    part = wave_sum(part);
    if (lane == 0) aux[g] = part / (float)E;
  }
  // packed layout: row_base[:, e] = running sum of fill[:, e] over the groups, 64 experts per
  // block (coalesced rows of fill, G loads per lane)
  if (summing)
    for (int e = 64 * blockIdx.x + lane; e < E; e += 64 * gridDim.x) {   // no wave-level ops inside
      int run = 0;
      for (int gg = 0; gg < G; ++gg) {
        pk.row_base[(size_t)gg * E + e] = run;
        run += fill[(size_t)gg * E + e];
      }
      pk.kept[e] = run;
    }
  const int s = ch * kChunk + lane;
  const bool valid = s < S;
  const size_t n = (size_t)g * S + (valid ? s : 0);
  int e1 = -1, e2 = -1;      // -1: takes part in no ranking
  bool sampled = false;
  if (valid) {
    e1 = expert_idx[2 * n];
    sampled = slot[2 * n + 1] != MOE_SLOT_NOT_SAMPLED;
    if (sampled) e2 = expert_idx[2 * n + 1];
  }
  // packed layout: kept rows of the two experts in the groups before this one (loads that the
  // rank loop below hides)
  // Up to 128 experts: lane l sums the columns l and l + 64 of fill (coalesced) and the sums
  // meet in LDS after the rank loop; wider gates: every lane sums the columns of its own two
  // experts.
  __shared__ int rb_s[128];
  const bool rb_shared = E <= 128;
  int rb1 = 0, rb2 = 0;
  if (packing && BASED) {
    if (e1 >= 0) rb1 = pk.row_base[(size_t)g * E + e1];
    if (e2 >= 0) rb2 = pk.row_base[(size_t)g * E + e2];
  }
  if (summing) {
    const int ca = rb_shared ? (lane < E ? lane : -1) : e1;
    const int cb = rb_shared ? (lane + 64 < E ? lane + 64 : -1) : e2;
    for (int gg = 0; gg < g; ++gg) {
      if (ca >= 0) rb1 += fill[(size_t)gg * E + ca];
      if (cb >= 0) rb2 += fill[(size_t)gg * E + cb];
    }
  }
  // stable rank among the earlier tokens of the chunk with the same expert: the lanes that agree
  // with this one in every bit of the expert index, one ballot per bit
  unsigned long long peers1 = __ballot(e1 >= 0), peers2 = __ballot(e2 >= 0);
  for (int bit = 0; (E - 1) >> bit; ++bit) {
    const bool b1 = (e1 >> bit) & 1, b2 = (e2 >> bit) & 1;
    const unsigned long long m1 = __ballot(b1), m2 = __ballot(b2);
    peers1 &= b1 ? m1 : ~m1;
    peers2 &= b2 ? m2 : ~m2;
  }
  const unsigned long long earlier = (1ull << lane) - 1;
  const int r1 = __popcll(peers1 & earlier), r2 = __popcll(peers2 & earlier);
  if (summing && rb_shared) {
    rb_s[lane] = rb1;
    rb_s[lane + 64] = rb2;
    __syncthreads();                                  // the block is this one wavefront
    rb1 = e1 >= 0 ? rb_s[e1] : 0;
    rb2 = e2 >= 0 ? rb_s[e2] : 0;
  }
  if (!valid) return;
  const size_t cb = ((size_t)g * nch + ch) * E;
  const int p1 = base1[cb + e1] + r1;
  const int s1 = p1 < C ? p1 : MOE_SLOT_OVERFLOW;
  int s2 = MOE_SLOT_NOT_SAMPLED;
  if (sampled) {
    const int p2 = base2[cb + e2] + r2;
    s2 = p2 < C ? p2 : MOE_SLOT_OVERFLOW;
  }
  slot[2 * n] = s1;
  slot[2 * n + 1] = s2;
  if (s1 < 0) weight[2 * n] = 0.f;
  if (s2 < 0) weight[2 * n + 1] = 0.f;
  if (s1 >= 0) src_token[((size_t)e1 * G + g) * C + s1] = s;
  if (s2 >= 0) src_token[((size_t)e2 * G + g) * C + s2] = s;
  if (packing) {
    const size_t R = (size_t)G * C;
    if (s1 >= 0) pk.packed_src[(size_t)e1 * R + rb1 + s1] = (int32_t)n;
    if (s2 >= 0) pk.packed_src[(size_t)e2 * R + rb2 + s2] = (int32_t)n;
  }
}

// Kept rows of expert e in the groups k, k + stride, ... before g, from the chunk histograms.  The loads of GB
// groups x CB chunks go out together; past the last group or chunk the last one is read again, not added.
template <int GB, int CB>
__device__ __forceinline__ int kept_before(const int32_t* __restrict__ hist1, const int32_t* __restrict__ hist2,
                                           int e, int k, int g, int stride, int nch, int E, int C) {
  int rb = 0;
  for (int g0 = k; g0 < g; g0 += GB * stride) {
    long long tot[GB];
#pragma unroll
    for (int i = 0; i < GB; ++i) tot[i] = 0;
    for (int c0 = 0; c0 < nch; c0 += CB) {
      int a[GB][CB], b[GB][CB];
#pragma unroll
      for (int i = 0; i < GB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) {
          const int gg = g0 + i * stride < g ? g0 + i * stride : g0;
          const size_t at = ((size_t)gg * nch + (c0 + j < nch ? c0 + j : nch - 1)) * E + e;
          a[i][j] = hist1[at];
          b[i][j] = hist2[at];
        }
#pragma unroll
      for (int i = 0; i < GB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j)
          if (c0 + j < nch) tot[i] += a[i][j] + b[i][j];
    }
#pragma unroll
    for (int i = 0; i < GB; ++i)
      if (g0 + i * stride < g) rb += tot[i] < C ? (int)tot[i] : C;
  }
  return rb;
}

// gate_scan_kernel and gate_slots_kernel in one launch, for calls of few chunks and up to 128 experts:
// one block per chunk, which sums for itself the histograms of its group and, for the packed layout, of
// the groups before it, instead of reading a prefix that another launch has written.  hist1 / hist2 stay
// as the chunks wrote them.  The sums are integers; the gate sums (block of a group's first chunk) are
// added in gate_scan_kernel's order, so every result has the same bits.
//
// Bound: launch and L2 latency, not bytes; both sides are measured at gate_route_form.
//
// Thread (e, k): expert e of EP = 16, 32, 64 or 128, slice k of 512 / EP.  Slice k sums every 512/EP-th chunk
// of the block's own group and all chunks of every 512/EP-th earlier group.
template <int GB, int CB>
__global__ __launch_bounds__(512) void gate_route_kernel(
    int S, int E, int C, int G, int nch, int ep_log2,
    const int32_t* __restrict__ hist1, const int32_t* __restrict__ hist2, const float* __restrict__ msum,
    const int32_t* __restrict__ expert_idx, int32_t* __restrict__ slot, float* __restrict__ weight,
    int32_t* __restrict__ src_token, int32_t* __restrict__ c1, float* __restrict__ mean_gate,
    int32_t* __restrict__ fill, float* __restrict__ aux, uint32_t* __restrict__ zero_fill, int zero_words,
    RowPacking pk) {
  constexpr int NT = 512, UN = 8;
  __shared__ int sb1[NT], st1[NT], sb2[NT], st2[NT], srb[NT];   // [slices][EP]
  __shared__ float tm[8 * 128];                                 // [8][EP]
  __shared__ int base1[128], base2[128], row0[128], filled[128];
  __shared__ float aux_term[128];
  const int g = blockIdx.x / nch, ch = blockIdx.x % nch;
  const int tid = threadIdx.x, EP = 1 << ep_log2, NS = NT >> ep_log2;
  const int e = tid & (EP - 1), k = tid >> ep_log2;
  const bool packing = pk.packed_src != nullptr, live = e < E;
  if (blockIdx.x == 0)
    for (int i = tid; i < zero_words; i += NT) zero_fill[i] = 0u;

  // the token's record, requested before the counters
  const int s = ch * kChunk + tid;
  const bool token = tid < kChunk && s < S;
  const size_t n = (size_t)g * S + (token ? s : 0);
  int e1 = -1, e2 = -1;
  if (token) {
    e1 = expert_idx[2 * n];
    if (slot[2 * n + 1] != MOE_SLOT_NOT_SAMPLED) e2 = expert_idx[2 * n + 1];
  }

  int b1 = 0, t1 = 0, b2 = 0, t2 = 0, rb = 0;
  if (live) {
    const size_t own = (size_t)g * nch * E + e;
    for (int c0 = k; c0 < nch; c0 += UN * NS) {                 // loads of a batch are independent
      int a1[UN], a2[UN];
#pragma unroll
      for (int j = 0; j < UN; ++j) {
        const size_t i = own + (size_t)(c0 + j * NS < nch ? c0 + j * NS : k) * E;
        a1[j] = hist1[i];
        a2[j] = hist2[i];
      }
#pragma unroll
      for (int j = 0; j < UN; ++j) {
        const int c = c0 + j * NS;
        b1 += c < ch ? a1[j] : 0;
        b2 += c < ch ? a2[j] : 0;
        t1 += c < nch ? a1[j] : 0;
        t2 += c < nch ? a2[j] : 0;
      }
    }
    if (packing) rb = kept_before<GB, CB>(hist1, hist2, e, k, g, NS, nch, E, C);
  }
  sb1[tid] = b1;
  st1[tid] = t1;
  sb2[tid] = b2;
  st2[tid] = t2;
  srb[tid] = rb;
  if (ch == 0 && live) {
    const int seg = (nch + 7) / 8;
    for (int kk = k; kk < 8; kk += NS) {
      float ms = 0.f;
      const int end = (kk + 1) * seg < nch ? (kk + 1) * seg : nch;
      for (int c0 = kk * seg; c0 < end; c0 += UN) {
        float a[UN];
#pragma unroll
        for (int j = 0; j < UN; ++j) a[j] = c0 + j < end ? msum[((size_t)g * nch + c0 + j) * E + e] : 0.f;
#pragma unroll
        for (int j = 0; j < UN; ++j)
          if (c0 + j < end) ms += a[j];
      }
      tm[kk * EP + e] = ms;
    }
  }
  __syncthreads();
  if (tid < E) {
    b1 = t1 = b2 = t2 = rb = 0;
    for (int i = tid; i < NT; i += EP) {
      b1 += sb1[i];
      t1 += st1[i];
      b2 += sb2[i];
      t2 += st2[i];
      rb += srb[i];
    }
    const long long tot = (long long)t1 + t2;
    const int f = tot < C ? (int)tot : C;
    base1[tid] = b1;
    base2[tid] = t1 + b2;                                       // second choices queue behind all first ones
    row0[tid] = rb;
    filled[tid] = f;
    if (ch == 0) {
      float mtot = 0.f;
      for (int kk = 0; kk < 8; ++kk) mtot += tm[kk * EP + tid];
      const float mean = mtot / (float)S;
      c1[(size_t)g * E + tid] = t1;
      mean_gate[(size_t)g * E + tid] = mean;
      fill[(size_t)g * E + tid] = f;
      aux_term[tid] = ((float)t1 / (float)S) * mean;
      if (packing) {
        pk.row_base[(size_t)g * E + tid] = rb;
        if (g == G - 1) pk.kept[tid] = rb + f;
      }
    }
  }
  __syncthreads();
  if (tid >= kChunk) {
    if (ch == 0 && tid < 2 * kChunk) {                          // l_aux[g], summed as in gate_slots_kernel
      const int lane = tid & 63;
      float part = 0.f;
      for (int i = lane; i < E; i += 64) part += aux_term[i];
      part = wave_sum(part);
      if (lane == 0) aux[g] = part / (float)E;
    }
    // empty positions of every nch-th expert: one expert after another where each has work for all threads,
    // else one per wavefront at a time (one chunk, M 1024, E 128, whole gate: C 1 39.3 -> 31.7 us, C 64
    // 42.0 -> 32.1; by wavefronts the empty positions of 16 384 cost up to 5 us more)
    constexpr int T = NT - kChunk;
    const int t0 = tid - kChunk;
    const bool all = C >= T;
    const int first = all ? 0 : t0 >> 6, experts = all ? 1 : T / 64, lane = all ? t0 : t0 & 63, step = all ? T : 64;
    for (int i = ch + nch * first; i < E; i += nch * experts) {
      int32_t* st = src_token + ((size_t)i * G + g) * C;
      for (int c = filled[i] + lane; c < C; c += step) st[c] = -1;
    }
    return;
  }
  // ranks as in gate_slots_kernel
  unsigned long long peers1 = __ballot(e1 >= 0), peers2 = __ballot(e2 >= 0);
  for (int bit = 0; (E - 1) >> bit; ++bit) {
    const bool x1 = (e1 >> bit) & 1, x2 = (e2 >> bit) & 1;
    const unsigned long long m1 = __ballot(x1), m2 = __ballot(x2);
    peers1 &= x1 ? m1 : ~m1;
    peers2 &= x2 ? m2 : ~m2;
  }
  if (!token) return;
  const unsigned long long earlier = (1ull << tid) - 1;
  const int p1 = base1[e1] + __popcll(peers1 & earlier);
  const int s1 = p1 < C ? p1 : MOE_SLOT_OVERFLOW;
  int s2 = MOE_SLOT_NOT_SAMPLED;
  if (e2 >= 0) {
    const int p2 = base2[e2] + __popcll(peers2 & earlier);
    s2 = p2 < C ? p2 : MOE_SLOT_OVERFLOW;
  }
  slot[2 * n] = s1;
  slot[2 * n + 1] = s2;
  if (s1 < 0) weight[2 * n] = 0.f;
  if (s2 < 0) weight[2 * n + 1] = 0.f;
  if (s1 >= 0) src_token[((size_t)e1 * G + g) * C + s1] = s;
  if (s2 >= 0) src_token[((size_t)e2 * G + g) * C + s2] = s;
  if (packing) {
    const size_t R = (size_t)G * C;
    if (s1 >= 0) pk.packed_src[(size_t)e1 * R + row0[e1] + s1] = (int32_t)n;
    if (s2 >= 0) pk.packed_src[(size_t)e2 * R + row0[e2] + s2] = (int32_t)n;
  }
}

// The packed row layout from fill alone, for expert buffers in the [E,G,C,M] order of the staged
// entry points: row p of expert e comes from (and goes back to) row (e G + g) C + c of the buffer.
__global__ __launch_bounds__(64) void row_maps_from_fill_kernel(
    int E, int G, int C, const int32_t* __restrict__ fill, RowPacking pk,
    uint32_t* __restrict__ zero_fill, int zero_words) {
  const int lane = threadIdx.x;
  if (blockIdx.x == 0)
    for (int i = lane; i < zero_words; i += 64) zero_fill[i] = 0u;
  const size_t R = (size_t)G * C;
  const long long idx = (long long)blockIdx.x * 64 + lane;
  if (idx >= (long long)E * G * C) return;
  const int c = (int)(idx % C), g = (int)((idx / C) % G), e = (int)(idx / ((long long)C * G));
  int rb = 0;
  for (int gg = 0; gg < g; ++gg) rb += fill[(size_t)gg * E + e];
  if (c == 0) {
    pk.row_base[(size_t)g * E + e] = rb;
    if (g == G - 1) pk.kept[e] = rb + fill[(size_t)g * E + e];
  }
  if (c < fill[(size_t)g * E + e]) pk.packed_src[(size_t)e * R + rb + c] = (int32_t)idx;
}

template <typename T, bool PRE = false>
int launch_topk(const moe_config& c, int nch, const T* x, const float* wg, const float* u,
                int32_t* expert_idx, int32_t* slot, float* weight, float* gates_opt,
                int32_t* hist1, int32_t* hist2, float* msum, hipStream_t st,
                const float* zpre = nullptr, int cols = 0) {
  const size_t shm = ((PRE ? 0 : (size_t)4 * c.M) + (size_t)4 * c.E) * sizeof(float) +
                     (size_t)2 * c.E * sizeof(int);
  if (shm > 64 * 1024) return MOE_EUNSUPPORTED;   // the default dynamic LDS limit of a kernel
  const dim3 grid((unsigned)(c.G * nch)), block(256);
  const int epl = (c.E + 63) / 64;
#define MOE_GATE_CASE(N)                                                                        \
  hipLaunchKernelGGL((gate_topk_kernel<T, N, PRE>), grid, block, shm, st, x, wg, u, zpre, cols, \
                     c.S, c.M, c.E, nch, expert_idx, slot, weight, gates_opt, hist1, hist2, msum)
  if (epl <= 1) MOE_GATE_CASE(1);
  else if (epl <= 2) MOE_GATE_CASE(2);
  else if (epl <= 4) MOE_GATE_CASE(4);
  else if (epl <= 8) MOE_GATE_CASE(8);
  else if (epl <= 16) MOE_GATE_CASE(16);
  else if (epl <= 32) MOE_GATE_CASE(32);
  else return MOE_EUNSUPPORTED;  // more than 2048 experts
#undef MOE_GATE_CASE
  return check_launch();
}

}  // namespace

// Very wide gates (E > 512): wgk[3e+p, m] = term p of wg[m,e] (hi, mid, lo bf16 terms), rows
// past 3E zero: the K-contiguous B operand of a plain GEMM x . wgk^T whose fp32 result holds the
// three partial logits of every expert side by side.
namespace {
// K = reps * M: the row is repeated `reps` times along K (fp32 activations enter the product as
// three bf16 terms side by side, each of which meets every term of wg).
__global__ __launch_bounds__(256) void gate_pack_wide_kernel(
    const float* __restrict__ wg, bf16_t* __restrict__ wgk, int M, int E, int cols, int reps) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  const int K = reps * M;
  if (i >= (long long)cols * K) return;
  const int c = (int)(i / K), m = (int)(i % K) % M;
  bf16_t out = 0;
  if (c < 3 * E) {
    const float v = wg[(size_t)m * E + c / 3];
    const bf16_t hi = f32_to_bf16(v);
    const float r1 = v - bf16_to_f32(hi);
    const bf16_t mid = f32_to_bf16(r1);
    const bf16_t lo = f32_to_bf16(r1 - bf16_to_f32(mid));
    out = c % 3 == 0 ? hi : (c % 3 == 1 ? mid : lo);
  }
  wgk[i] = out;
}

// xk[n, a*M + m] = term a (hi, mid, lo) of the fp32 activation x[n,m]: x = hi + mid + lo exactly
__global__ __launch_bounds__(256) void gate_split_x_kernel(
    const float* __restrict__ x, bf16_t* __restrict__ xk, int M, long long tokens) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= tokens * M) return;
  const long long n = i / M;
  const int m = (int)(i % M);
  const float v = x[i];
  const bf16_t hi = f32_to_bf16(v);
  const float r1 = v - bf16_to_f32(hi);
  const bf16_t mid = f32_to_bf16(r1);
  bf16_t* d = xk + n * 3 * M + m;
  d[0] = hi;
  d[M] = mid;
  d[2 * (size_t)M] = f32_to_bf16(r1 - bf16_to_f32(mid));
}
}  // namespace

// fp32 gates of up to 128 experts: gate_chunk_kernel, nothing to pack
static bool gate_f32_chunks(const moe_config& c) { return c.act_dtype == MOE_F32 && c.E <= 128; }

// Logits as one GEMM on the matrix cores, for bf16 gates wider than 512 experts and for wider fp32
// gates (x split into three bf16 terms, K = 3 M): needs the persistent GEMM's shapes (token
// count a multiple of 256, K of 32) and at most 2048 experts (registers of the epilogue kernel).
struct WideGeom { int cols, k; size_t z_bytes, w_bytes, x_bytes; };
static WideGeom wide_geom(const moe_config& c) {
  WideGeom w{};
  const long long tokens = (long long)c.G * c.S;
  const long long cols = ((long long)3 * c.E + 255) / 256 * 256;
  const long long k = c.act_dtype == MOE_F32 ? (long long)3 * c.M : c.M;
  if (gate_f32_chunks(c) || (c.act_dtype == MOE_BF16 && c.E <= 512) || c.E > 2048 || tokens > 0x7fffffffLL ||
      k > 0x7fffffffLL || !gemm_bf16_f32out_ok((int)tokens, (int)cols, (int)k))
    return w;
  w.cols = (int)cols;
  w.k = (int)k;
  w.z_bytes = (size_t)tokens * cols * 4;
  w.w_bytes = (size_t)cols * k * 2;
  w.x_bytes = c.act_dtype == MOE_F32 ? (size_t)tokens * k * 2 : 0;
  return w;
}

// Geometry of the packed gate weights (bf16 MFMA path).
struct PackGeom { int T, KS; size_t bytes; };
static PackGeom pack_geom(const moe_config& c) {
  PackGeom p{};
  if (c.act_dtype != MOE_BF16 || c.E > 512) return p;   // bytes == 0: plain kernel
  const int epad = c.E <= 64 ? (c.E + 31) / 32 * 32 : c.E <= 128 ? 128 : c.E <= 256 ? 256 : 512;
  p.T = epad / 32;
  p.KS = (c.M + 63) / 64 * 4;
  p.bytes = (size_t)p.KS * p.T * 3 * 64 * 16;
  return p;
}

size_t gate_workspace_bytes(const moe_config& c) {
  const size_t nch = (size_t)(c.S + kChunk - 1) / kChunk;
  const WideGeom w = wide_geom(c);
  return 3 * align_up((size_t)c.G * nch * c.E * 4, 256) + align_up(pack_geom(c).bytes, 256) +
         align_up(w.w_bytes, 256) + align_up(w.z_bytes, 256) + align_up(w.x_bytes, 256);
}

// The gate weights in the form the logit kernels multiply: three bf16 terms per weight in the
// MFMA operand order (E <= 512, bf16 activations) or as the K-contiguous operand of the logit
// GEMM (wider gates, fp32 activations with GEMM-friendly shapes); 0 bytes when the gate reads
// wg as it is.
size_t gate_pack_bytes(const moe_config& c) {
  const PackGeom pg = pack_geom(c);
  return pg.bytes != 0 ? pg.bytes : wide_geom(c).w_bytes;
}

int launch_gate_pack(const moe_config& c, const float* wg, void* packed, hipStream_t st) {
  const WideGeom w = wide_geom(c);
  if (w.cols != 0) {
    const long long n = (long long)w.cols * w.k;
    hipLaunchKernelGGL(gate_pack_wide_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, wg,
                       static_cast<bf16_t*>(packed), c.M, c.E, w.cols, w.k / c.M);
    return check_launch();
  }
  const PackGeom pg = pack_geom(c);
  if (pg.bytes == 0) return MOE_OK;
  const int total = pg.KS * pg.T * 64;
  hipLaunchKernelGGL(gate_pack_wg_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, wg,
                     static_cast<uint4*>(packed), c.M, c.E, pg.T, total);
  return check_launch();
}

// partial logits [4][128][Epad + 4], per-wavefront gate sums [4][Epad], histograms [4][Epad]
constexpr size_t kGateRowsLds1 = (4 * 128 * 36 + 8 * 32) * 4, kGateRowsLds2 = (4 * 128 * 68 + 8 * 64) * 4;

// partial logits [KW][64][Epad + 8] and two histograms [Epad]
template <int ETW, int KW> constexpr int kGateChunkLds = (KW * 64 * (32 * ETW * 8 / KW + 8) + 2 * 32 * ETW * 8 / KW) * 4;

template <typename T, int ETW, int KW, bool TAIL, bool RAW = false>
static int prepare_gate_chunk() {
  static LdsLimitOnce once;
  return ensure_lds_limit(once, reinterpret_cast<const void*>(gate_chunk_kernel<T, ETW, KW, TAIL, RAW>),
                          kGateChunkLds<ETW, KW>);
}

template <int ET>
static int prepare_gate_rows() {
  static LdsLimitOnce once;
  return ensure_lds_limit(once, reinterpret_cast<const void*>(gate_mfma_rows_kernel<ET>),
                          (int)(ET == 1 ? kGateRowsLds1 : kGateRowsLds2));
}

int prepare_gate() {
  const int rcs[] = {prepare_gate_rows<1>(), prepare_gate_rows<2>(),
                     prepare_gate_chunk<bf16_t, 1, 8, false>(), prepare_gate_chunk<bf16_t, 2, 8, false>(),
                     prepare_gate_chunk<bf16_t, 1, 8, false, true>(), prepare_gate_chunk<bf16_t, 2, 8, false, true>(),
                     prepare_gate_chunk<float, 1, 8, false>(), prepare_gate_chunk<float, 1, 8, true>(),
                     prepare_gate_chunk<float, 2, 8, false>(), prepare_gate_chunk<float, 2, 8, true>(),
                     prepare_gate_chunk<float, 2, 4, false>(), prepare_gate_chunk<float, 2, 4, true>()};
  for (int rc : rcs)
    if (rc != MOE_OK) return rc;
  return MOE_OK;
}

// One launch for positions and row maps (gate_route_kernel), or the scan and the slots kernel.  Every block
// of the first reads up to all counters of the call, so its work grows with the square of the chunks; the
// other two pay a launch, and slots a serial loop over the earlier groups.  Whole layer of M 128, H 8 (us,
// two launches -> one; G x tokens, E): 5 x 700, 24: 28.8 -> 26.0; 4 x 1024, 16: 28.6 -> 26.2; 16 x 1024, 2:
// 33.7 -> 30.6; 128 x 64, 16: 49.0 -> 28.4; 1 x 16 384, 32: 39.2 -> 31.7; 1 x 32 768, 16: 62.6 -> 47.5;
// 8 x 1024, 128: 36.0 -> 32.5; at the line 8 x 4096, 32 (512 chunks, 16 384 counters): 47.5 -> 46.7; past
// it 4 x 4096, 128: 40.0 -> 41.0.
static bool gate_route_form(const moe_config& c, long long chunks) {
  return c.E <= 128 && chunks <= 512 && chunks * c.E <= 16384;
}

// Packed layers of more groups than this sum them in a launch of their own (gate_row_base_kernel) before
// gate_slots_kernel, whose blocks otherwise each walk the groups before theirs, up to 0.4 us a group.  Whole
// layer of M 256, H 64 (us, walked / summed; G x tokens, E): 12 x 2816, 4 74.5 / 76.3, 512 137.7 / 138.9;
// 16 x 2112, 4 74.6 / 75.7, 130 103.5 / 100.7; 24 x 1408, 4 75.1 / 75.9, 32 80.3 / 76.2; 48 x 704, 32 86.9 /
// 75.6; 1000 x 20, 32 318 / 76.
constexpr int kSumGroups = 16;

// Whether a bf16 gate of few chunks without packed weights splits wg itself.  A block's chain of loads, splits and products
// grows with M, and with two tiles of columns per wavefront it has half the loads in flight: then the launch that
// packs is the shorter way from 2560 on.  Layer of H 64, us, packed first / split here (tokens, M, E): 64, 4096, 32 67.7 / 59.9;
// 64, 1024, 33 33.0 / 32.0; 700, 1536, 64 48.3 / 47.1; 4 x 1024, 2048, 64 65.7 / 64.7; 64, 2048, 33 46.8 / 47.4; 700, 2560, 33
// 63.1 / 65.3; 64, 3072, 64 65.2 / 69.3; 64, 4096, 33 78.3 / 84.2.
bool gate_splits_wg(int E, int M) { return E <= 32 || M <= 2048; }

int launch_gate(const moe_config& c, const void* x, const float* wg, const float* u,
                int32_t* expert_idx, int32_t* slot, float* weight, int32_t* fill,
                int32_t* src_token, int32_t* c1, float* mean_gate, float* aux,
                float* gates_opt, void* ws, void* zero_row, const RowPacking* packing,
                const void* wg_prepacked, hipStream_t st) {
  const int nch = (c.S + kChunk - 1) / kChunk;
  const size_t seg = align_up((size_t)c.G * nch * c.E * 4, 256);
  int32_t* hist1 = reinterpret_cast<int32_t*>(ws);
  int32_t* hist2 = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + seg);
  float* msum = reinterpret_cast<float*>(static_cast<char*>(ws) + 2 * seg);
  // the packed weights: the caller's (packed once with launch_gate_pack) or this call's own
  char* const own = static_cast<char*>(ws) + 3 * seg;
  uint4* wgP = wg_prepacked != nullptr ? static_cast<uint4*>(const_cast<void*>(wg_prepacked))
                                        : reinterpret_cast<uint4*>(own);
  const PackGeom pg = pack_geom(c);
  int rc, cus = 0;
  if (compute_units(&cus) != MOE_OK) return MOE_EHIP;
  const long long chunks = (long long)c.G * nch;
  const bool chunk_form = gate_f32_chunks(c) || (c.act_dtype == MOE_BF16 && c.E <= 64 && chunks <= cus);
  const bool single = chunk_form && chunks == 1;
  const int zero_words = zero_row != nullptr ? c.M / 2 : 0;
  const RowPacking pk = packing != nullptr ? *packing : RowPacking{nullptr, nullptr, nullptr};
  const bool raw = chunk_form && c.act_dtype == MOE_BF16 && wg_prepacked == nullptr && gate_splits_wg(c.E, c.M);
  if (wg_prepacked == nullptr && !raw && (rc = launch_gate_pack(c, wg, own, st)) != MOE_OK) return rc;
  if (chunk_form) {
#define MOE_GATE_CHUNK(T, ETW, KW, TAIL, RAW)                                                           \
  {                                                                                                     \
    if (prepare_gate_chunk<T, ETW, KW, TAIL, RAW>() != MOE_OK) return MOE_EHIP;                         \
    hipLaunchKernelGGL((gate_chunk_kernel<T, ETW, KW, TAIL, RAW>), dim3((unsigned)chunks), dim3(512),   \
                       (kGateChunkLds<ETW, KW>), st, static_cast<const T*>(x), wgP, wg, u, c.S, c.M, c.E, c.C, \
                       nch, expert_idx, slot, weight, gates_opt, hist1, hist2, msum, src_token, c1,     \
                       mean_gate, fill, aux, static_cast<uint32_t*>(zero_row), zero_words, pk, single); \
  }
#define MOE_GATE_CHUNK_F32(ETW, KW)                                                                     \
  if (c.M % 32 != 0) MOE_GATE_CHUNK(float, ETW, KW, true, false) else MOE_GATE_CHUNK(float, ETW, KW, false, false)
    if (c.act_dtype == MOE_BF16) {
      if (c.E <= 32) {
        if (raw) MOE_GATE_CHUNK(bf16_t, 1, 8, false, true) else MOE_GATE_CHUNK(bf16_t, 1, 8, false, false)
      } else if (raw) {
        MOE_GATE_CHUNK(bf16_t, 2, 8, false, true)
      } else {
        MOE_GATE_CHUNK(bf16_t, 2, 8, false, false)
      }
    } else if (c.E <= 32) {
      MOE_GATE_CHUNK_F32(1, 8)
    } else if (c.E <= 64) {
      MOE_GATE_CHUNK_F32(2, 8)
    } else {
      MOE_GATE_CHUNK_F32(2, 4)
    }
#undef MOE_GATE_CHUNK_F32
#undef MOE_GATE_CHUNK
    if ((rc = check_launch()) != MOE_OK || single) return rc;
  } else if (wide_geom(c).cols != 0) {
    // pg.bytes == 0 here: the packed-operand region is empty; wgk, the logits and (fp32) the
    // split activations follow it
    const WideGeom w = wide_geom(c);
    const long long tokens = (long long)c.G * c.S;
    const bf16_t* wgk = reinterpret_cast<const bf16_t*>(wgP);
    char* after = own + align_up(w.w_bytes, 256);
    float* zpre = reinterpret_cast<float*>(after);
    bf16_t* xk = reinterpret_cast<bf16_t*>(after + align_up(w.z_bytes, 256));
    const void* a = x;
    if (c.act_dtype == MOE_F32) {
      hipLaunchKernelGGL(gate_split_x_kernel, dim3((unsigned)((tokens * c.M + 255) / 256)), dim3(256),
                         0, st, static_cast<const float*>(x), xk, c.M, tokens);
      if ((rc = check_launch()) != MOE_OK) return rc;
      a = xk;
    }
    rc = launch_gemm_bf16_f32out(false, a, wgk, zpre, 1, (int)tokens, w.cols, w.k, st);
    if (rc != MOE_OK) return rc;
    rc = c.act_dtype == MOE_F32
             ? launch_topk<float, true>(c, nch, static_cast<const float*>(x), wg, u, expert_idx, slot,
                                        weight, gates_opt, hist1, hist2, msum, st, zpre, w.cols)
             : launch_topk<bf16_t, true>(c, nch, static_cast<const bf16_t*>(x), wg, u, expert_idx,
                                         slot, weight, gates_opt, hist1, hist2, msum, st, zpre, w.cols);
  } else if (c.act_dtype == MOE_F32) {
    rc = launch_topk<float>(c, nch, static_cast<const float*>(x), wg, u, expert_idx, slot, weight,
                            gates_opt, hist1, hist2, msum, st);
  } else if (pg.bytes == 0) {
    rc = launch_topk<bf16_t>(c, nch, static_cast<const bf16_t*>(x), wg, u, expert_idx, slot,
                             weight, gates_opt, hist1, hist2, msum, st);
  } else {
    const dim3 grid((unsigned)(c.G * ((nch + 1) / 2))), block(256);
    const bf16_t* xb = static_cast<const bf16_t*>(x);
#define MOE_GATE_ARGS xb, wgP, u, c.S, c.M, c.E, nch, expert_idx, slot, weight, gates_opt, hist1, hist2, msum
    if (c.E <= 64) {
      const size_t lds1 = kGateRowsLds1, lds2 = kGateRowsLds2;
      if ((c.E <= 32 ? prepare_gate_rows<1>() : prepare_gate_rows<2>()) != MOE_OK) return MOE_EHIP;
      if (c.E <= 32) hipLaunchKernelGGL(gate_mfma_rows_kernel<1>, grid, block, lds1, st, MOE_GATE_ARGS);
      else hipLaunchKernelGGL(gate_mfma_rows_kernel<2>, grid, block, lds2, st, MOE_GATE_ARGS);
    }
    else if (c.E <= 128) {
      // 256-token blocks once they give every compute unit a block
      const long long blocks256 = (long long)c.G * ((nch + 3) / 4);
      if (blocks256 >= cus)
        hipLaunchKernelGGL((gate_mfma_cols_split_kernel<1, 6, 8, 8>), dim3((unsigned)blocks256), dim3(512), 0, st, MOE_GATE_ARGS);
      else
        hipLaunchKernelGGL((gate_mfma_cols_split_kernel<1, 6, 8>), grid, dim3(512), 0, st, MOE_GATE_ARGS);
    }
    else if (c.E <= 256) hipLaunchKernelGGL((gate_mfma_cols_split_kernel<2, 2, 4>), grid, dim3(512), 0, st, MOE_GATE_ARGS);
    else hipLaunchKernelGGL((gate_mfma_cols_kernel<2, 8, 2>), grid, dim3(512), 0, st, MOE_GATE_ARGS);
#undef MOE_GATE_ARGS
    rc = check_launch();
  }
  if (rc != MOE_OK) return rc;
  if (gate_route_form(c, chunks)) {
    // groups of one or two chunks are added up eight at a time
    auto route = pk.packed_src != nullptr && nch <= 2 ? gate_route_kernel<8, 2> : gate_route_kernel<1, 16>;
    hipLaunchKernelGGL(route, dim3((unsigned)chunks), dim3(512), 0, st, c.S, c.E, c.C, c.G, nch,
                       c.E <= 16 ? 4 : c.E <= 32 ? 5 : c.E <= 64 ? 6 : 7, hist1, hist2, msum, expert_idx, slot, weight,
                       src_token, c1, mean_gate, fill, aux, static_cast<uint32_t*>(zero_row), zero_words, pk);
    return check_launch();
  }
  hipLaunchKernelGGL(gate_scan_kernel, dim3((unsigned)(c.G * ((c.E + 31) / 32))), dim3(256), 0, st,
                     c.S, c.E, c.C, c.G, nch, hist1, hist2, msum, c1, mean_gate, fill, src_token);
  if ((rc = check_launch()) != MOE_OK) return rc;
  const bool based = pk.packed_src != nullptr && c.G > kSumGroups;
  if (based) {
    hipLaunchKernelGGL(gate_row_base_kernel, dim3((unsigned)((c.E + 31) / 32)), dim3(1024), 0, st, c.G, c.E,
                       fill, pk.row_base, pk.kept);
    if ((rc = check_launch()) != MOE_OK) return rc;
  }
  hipLaunchKernelGGL(based ? gate_slots_kernel<true> : gate_slots_kernel<false>, dim3((unsigned)(c.G * nch)),
                     dim3(64), 0, st, c.S, c.E, c.C, c.G, nch, hist1, hist2, expert_idx, slot, weight,
                     src_token, c1, mean_gate, aux, static_cast<uint32_t*>(zero_row), zero_words, fill, pk);
  return check_launch();
}

int launch_row_maps_from_fill(const moe_config& c, const int32_t* fill, const RowPacking& pk,
                              void* zero_row, hipStream_t st) {
  const long long slots = (long long)c.E * c.G * c.C;
  hipLaunchKernelGGL(row_maps_from_fill_kernel, dim3((unsigned)((slots + 63) / 64)), dim3(64), 0, st,
                     c.E, c.G, c.C, fill, pk, static_cast<uint32_t*>(zero_row),
                     zero_row != nullptr ? c.M / 2 : 0);
  return check_launch();
}

}  // namespace moe
