// Backward pass of the top-2 MoE layer: everything except the large expert GEMMs.
//
// The paper differentiates Algorithm 2 automatically and states only that the counts
// c_e of the auxiliary loss carry no gradient while the mean gates m_e do (Section 2.2,
// "Auxiliary loss").  Written out by the chain rule, with all discrete routing decisions
// of Algorithm 1 as constants:
//
//   combine_bwd   dout[e,g,c,:] = weight[g,s,k] * dy[g,s,:]          (Eq. 3 transposed)
//                 dweight[g,s,k] = <dy[g,s,:], out[e,g,c,:]>
//                 and, in the same kernel: weight_1 = g1/(g1+g2), weight_2 = g2/(g1+g2)  (Algorithm 1) =>
//                 dgate[e1] = (dw1 - dw2) g2 / (g1+g2)^2,  dgate[e2] = (dw2 - dw1) g1 / (g1+g2)^2
//                 l_aux = (1/E) sum_e (c_e/S) m_e  =>  dgate[e] += daux[g] c_e / (E S^2)
//                 softmax: dz[e] = g[e] (dgate[e] - sum_e' g[e'] dgate[e'])
//   dwg           dwg[m,e] = sum_tokens x[t,m] dz[t,e]
//   dx            dx[g,s,:] = sum_k dbuf[e_k,g,c_k,:] + sum_e dz[g,s,e] wg[:,e]
//                 (dispatch transposed + the gate projection)
#include "common.h"

namespace moe {
namespace {

constexpr int kRowsPerBlock = 4;  // one wavefront per row / token
constexpr int kZeroRows = 64;     // rows that a block of combine_bwd_kernel checks and clears

// One wavefront per token: the gradient rows dout of its kept choices, their rows of the dispatched activations
// (buf, the first weight gradient's operand; the forward pass of packed layers never writes one), and the gradient of
// its gate logits, for which the choices' dweight stay in registers.  The blocks behind those of the tokens clear the
// rows that no token fills: of packed rows (kept != NULL) the ones from kept[e] to the end of that 256-row tile, which enter
// the weight gradients' sums.
// dz: NULL, or [tokens, ez] fp32 with zeros behind the E columns; dzp: NULL, or the three bf16 terms side by side
// in `cols` columns.
// Bound: HBM, x and dy rows once, out rows in, buf and dout rows out; for few tokens the chain routing -> rows -> sum -> gates.
// One wavefront per expert row read x and dy once per choice, and the gates were a launch of their own behind it:
// us of both, before / now: 4 x 1024 tokens, M 512, E 16 14.6 / 8.5; 3 x 1333 tokens, M 520, E 12 14.9 / 9.8; fp32,
// 4 x 1024 tokens, M 1024, E 16 31.7 / 27.9.
struct GateGrad {
  const float* gates;
  const int32_t* c1;
  const float* daux;
  float* dz;
  bf16_t* dzp;
  int ez, cols;
};
template <typename T>
__global__ __launch_bounds__(256) void combine_bwd_kernel(
    const uint4* __restrict__ dy, const uint4* __restrict__ out, const uint4* __restrict__ x,
    const int32_t* __restrict__ expert_idx, const int32_t* __restrict__ slot, const float* __restrict__ weight,
    uint4* __restrict__ dout, uint4* __restrict__ buf, int S, int G, int C, int E, int vec_per_row, long long tokens,
    unsigned token_blocks, const int32_t* __restrict__ src_token, const int32_t* __restrict__ kept,
    const int32_t* __restrict__ row_base, GateGrad gate) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (blockIdx.x >= token_blocks) {
    const long long per_expert = (long long)G * C;
    const unsigned zb = blockIdx.x - token_blocks;
    constexpr int kPerWave = kZeroRows / 4;
    long long r0;
    bool empty = false;
    if (kept != nullptr) {
      constexpr int kBlocks = 256 / kZeroRows;                   // per expert
      const int e = zb / kBlocks, ke = kept[e];
      const long long p0 = ke + (long long)(zb % kBlocks) * kZeroRows + wave * kPerWave;
      const long long end = (ke + 255) & ~255;
      r0 = e * per_expert + p0;
      empty = lane < kPerWave && p0 + lane < end && p0 + lane < per_expert;
    } else {
      r0 = (long long)zb * kZeroRows + wave * kPerWave;
      if (lane < kPerWave && r0 + lane < E * per_expert) empty = src_token[r0 + lane] < 0;
    }
    const uint4 zero = {0u, 0u, 0u, 0u};
    for (unsigned long long left = __ballot(empty); left != 0; left &= left - 1) {
      const long long o = (r0 + __builtin_ctzll(left)) * vec_per_row;
      for (int v = lane; v < vec_per_row; v += 64) dout[o + v] = buf[o + v] = zero;
    }
    return;
  }
  const long long n = (long long)blockIdx.x * kRowsPerBlock + wave;
  if (n >= tokens) return;
  const int g = (int)(n / S);
  const float* const p = gate.gates + n * E;
  const int32_t* const cg = gate.c1 + (long long)g * E;
  const int e1 = expert_idx[2 * n], e2 = expert_idx[2 * n + 1];
  const int s1 = slot[2 * n], s2 = slot[2 * n + 1];
  const float w1 = weight[2 * n], w2 = weight[2 * n + 1];
  const float g1 = p[e1], g2 = p[e2];
  // row of a kept choice: (e G + g) C + slot, or e G C + row_base[g,e] + slot when packed
  auto row_of = [&](int e, int s) {
    return row_base != nullptr ? (long long)e * G * C + row_base[(size_t)g * E + e] + s : ((long long)e * G + g) * C + s;
  };
  const uint4 *const dyr = dy + n * vec_per_row, *const xr = x + n * vec_per_row;
  const long long o1 = s1 >= 0 ? row_of(e1, s1) * vec_per_row : 0, o2 = s2 >= 0 ? row_of(e2, s2) * vec_per_row : 0;
  float d1 = 0.f, d2 = 0.f;
  if (s1 >= 0 || s2 >= 0) {
    // (two rounds of an fp32 row at a time, or few tokens of wide rows wait for each in turn: 64 tokens, M 4096 13.9 us by
    // expert row, 15.9 without, 13.8 now; bf16 rows of one to two rounds lose by it: 2048 tokens, M 768 8.2 / 9.3)
    constexpr int K = Vec16<T>::kElts, kRounds = sizeof(T) == 4 ? 2 : 1;
#pragma unroll kRounds
    for (int v = lane; v < vec_per_row; v += 64) {
      const uint4 dv = dyr[v], xv = xr[v];
      uint4 ov1 = {0u, 0u, 0u, 0u}, ov2 = ov1;
      if (s1 >= 0) ov1 = out[o1 + v];
      if (s2 >= 0) ov2 = out[o2 + v];
      float f[K], o[K];
      Vec16<T>::unpack(dv, f);
      auto choice = [&](const uint4& ov, float w, float* d, long long at) {
        float h[K];
        Vec16<T>::unpack(ov, o);
#pragma unroll
        for (int i = 0; i < K; ++i) {
          *d = fmaf(f[i], o[i], *d);
          h[i] = f[i] * w;
        }
        buf[at + v] = xv;
        dout[at + v] = Vec16<T>::pack(h);
      };
      if (s1 >= 0) choice(ov1, w1, &d1, o1);
      if (s2 >= 0) choice(ov2, w2, &d2, o2);
    }
    d1 = wave_sum(d1);
    d2 = wave_sum(d2);
  }
  const float inv = 1.f / ((g1 + g2) * (g1 + g2));
  const float t1 = (d1 - d2) * g2 * inv, t2 = (d2 - d1) * g1 * inv;
  const float scale = gate.daux[g] / ((float)E * (float)S * (float)S);
  float dot = 0.f;
  for (int e = lane; e < E; e += 64) {
    const float dp = scale * (float)cg[e] + (e == e1 ? t1 : 0.f) + (e == e2 ? t2 : 0.f);
    dot = fmaf(p[e], dp, dot);
  }
  dot = wave_sum(dot);
  for (int e = lane; e < E; e += 64) {
    const float dp = scale * (float)cg[e] + (e == e1 ? t1 : 0.f) + (e == e2 ? t2 : 0.f);
    const float v = p[e] * (dp - dot);
    if (gate.dz != nullptr) gate.dz[n * gate.ez + e] = v;
    if (gate.dzp != nullptr) {
      // v = hi + mid + lo exactly (three bf16 terms cover the 24 mantissa bits), stored side
      // by side so that a bf16 matrix product over these columns is an fp32-faithful one
      const bf16_t hi = f32_to_bf16(v);
      const float r1 = v - bf16_to_f32(hi);
      const bf16_t mid = f32_to_bf16(r1);
      const bf16_t lo = f32_to_bf16(r1 - bf16_to_f32(mid));
      bf16_t* d = gate.dzp + n * gate.cols + 3 * e;
      d[0] = hi; d[1] = mid; d[2] = lo;
    }
  }
  if (gate.dz != nullptr)
    for (int e = E + lane; e < gate.ez; e += 64) gate.dz[n * gate.ez + e] = 0.f;
  if (gate.dzp != nullptr)
    for (int cidx = 3 * E + lane; cidx < gate.cols; cidx += 64) gate.dzp[n * gate.cols + cidx] = 0;
}

// wgp[m, 3e+p] = bf16(wg[m,e]) for the three terms p of dz, zero in the padding columns
__global__ __launch_bounds__(256) void wg_pack_bwd_kernel(
    const float* __restrict__ wg, bf16_t* __restrict__ wgp, int M, int E, int cols) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long long)M * cols) return;
  const int m = (int)(i / cols), cidx = (int)(i % cols);
  wgp[i] = cidx < 3 * E ? f32_to_bf16(wg[(size_t)m * E + cidx / 3]) : (bf16_t)0;
}

// dx[n,:] = round( dxg[n,:] + dbuf row of the first kept choice + of the second ), bf16
__global__ __launch_bounds__(256) void dx_rows_kernel(
    const float4* __restrict__ dxg, const uint4* __restrict__ dbuf,
    const int32_t* __restrict__ expert_idx, const int32_t* __restrict__ slot,
    uint4* __restrict__ dx, int S, int G, int C, int E, int vec_per_row, long long tokens,
    const int32_t* __restrict__ row_base) {
  const long long n = (long long)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
  if (n >= tokens) return;
  const int lane = threadIdx.x & 63;
  const int g = (int)(n / S);
  const int s0 = slot[2 * n], s1 = slot[2 * n + 1];
  // row of a kept choice: (e G + g) C + slot, or e G C + row_base[g,e] + slot when packed
  const uint4 *r0 = nullptr, *r1 = nullptr;
  if (s0 >= 0) {
    const long long e = expert_idx[2 * n];
    r0 = dbuf + (row_base != nullptr ? e * G * C + row_base[(long long)g * E + e] + s0
                                     : (e * G + g) * C + s0) * vec_per_row;
  }
  if (s1 >= 0) {
    const long long e = expert_idx[2 * n + 1];
    r1 = dbuf + (row_base != nullptr ? e * G * C + row_base[(long long)g * E + e] + s1
                                     : (e * G + g) * C + s1) * vec_per_row;
  }
  for (int v = lane; v < vec_per_row; v += 64) {
    const float4 a = dxg[(n * vec_per_row + v) * 2], b = dxg[(n * vec_per_row + v) * 2 + 1];
    float acc[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    if (r0 != nullptr) {
      float f[8];
      Vec16<bf16_t>::unpack(r0[v], f);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += f[i];
    }
    if (r1 != nullptr) {
      float f[8];
      Vec16<bf16_t>::unpack(r1[v], f);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += f[i];
    }
    dx[n * vec_per_row + v] = Vec16<bf16_t>::pack(acc);
  }
}

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
static __device__ const f32x4_t bwd_zero_line = {0.f, 0.f, 0.f, 0.f};

// dwg[m,e] = sum_t x[t,m] dz[t,e]: partial sums over a range of tokens per block, then a reduction
// over the ranges in a fixed order (no atomics: the result is reproducible).
//
// Block = 128 features x 32 ET experts x one range; wavefront = 32 features; v_mfma_f32_32x32x2_f32 with
// k = tokens (x widened to fp32, so products are exact and the sums fp32).  Both operands are row-of-k:
// stages of 32 tokens of x and dz travel global -> LDS directly, rows past the range or M read a zero
// line.  (64 banks: chunk c of an odd row sits at c ^ 4 for 256-byte rows of bf16 x, c ^ 8 for longer
// ones, so the two tokens of a step fall into different banks.)
// Bound: one read of x.  32 768 tokens, M 1024, E 32: 56 us as a padded bf16 GEMM (three terms of dz in
// 256 columns, 67 MB of partial sums) and its reduction -> 33 us; 3999 tokens, M 520, E 12: 59 us on
// FMA -> 11 us.
template <typename T, int ET>
__global__ __launch_bounds__(256) void dwg_partial_kernel(
    const T* __restrict__ x, const float* __restrict__ dz, float* __restrict__ partial, int M, int ez,
    long long tokens, int tokens_per_split) {
  constexpr int TK = 32, ST = 3;
  constexpr int XP = 128 * sizeof(T), ZP = 128 * ET;             // row pitches in bytes
  constexpr int kX = TK * XP, kStage = kX + TK * ZP;
  constexpr int XC = XP / 16, ZC = ZP / 16;                      // 16-byte chunks per row
  constexpr int XQ = kX / 4096, ZQ = ET;                         // copies per wavefront and stage
  constexpr int XSW = sizeof(T) == 2 ? 4 : 8, ZSW = ET > 1 ? 8 : 0;
  extern __shared__ __attribute__((aligned(16))) unsigned char dwg_smem[];
  typedef unsigned char __attribute__((address_space(3))) * lds_ptr;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_ptr)dwg_smem);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, hf = lane >> 5;
  const int m0 = blockIdx.x * 128, e0 = blockIdx.y * 32 * ET;
  const long long t0 = (long long)blockIdx.z * tokens_per_split;
  const long long left = tokens - t0;
  const int cnt = left < 0 ? 0 : (left < tokens_per_split ? (int)left : tokens_per_split);
  const int KT = (cnt + TK - 1) / TK;
  const uint64_t zline = (uint64_t)(uintptr_t)&bwd_zero_line;
  uint64_t xa[XQ], za[ZQ];
  int xk[XQ], zk[ZQ];
  bool xok[XQ];
#pragma unroll
  for (int q = 0; q < XQ; ++q) {
    xk[q] = (64 / XC) * (wave * XQ + q) + lane / XC;
    const int col = m0 + (16 / (int)sizeof(T)) * ((lane % XC) ^ (XSW * (xk[q] & 1)));
    xok[q] = col < M;
    xa[q] = (uint64_t)(uintptr_t)(x + (t0 + xk[q]) * M + (xok[q] ? col : 0));
  }
#pragma unroll
  for (int q = 0; q < ZQ; ++q) {
    zk[q] = (64 / ZC) * (wave * ZQ + q) + lane / ZC;
    // columns past ez (a multiple of 32): only in the last of several expert tiles
    const int col = e0 + 4 * ((lane % ZC) ^ (ZSW * (zk[q] & 1)));
    za[q] = col < ez ? (uint64_t)(uintptr_t)(dz + (t0 + zk[q]) * ez + col) : 0;
  }
#define MOE_DWG_COPY(LDS_U32, ADDR_U64)                                                      \
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"            \
               :: "s"(LDS_U32), "v"(ADDR_U64) : "memory")
  auto start_step = [&](int p, int stage) {
    const uint32_t lx = lds0 + stage * kStage + wave * (XQ * 1024);
    const uint32_t lz = lds0 + stage * kStage + kX + wave * (ZQ * 1024);
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
      const uint64_t s = xok[q] && p * TK + xk[q] < cnt ? xa[q] + (uint64_t)p * TK * M * sizeof(T) : zline;
      MOE_DWG_COPY(lx + q * 1024, s);
    }
#pragma unroll
    for (int q = 0; q < ZQ; ++q) {
      const uint64_t s = za[q] != 0 && p * TK + zk[q] < cnt ? za[q] + (uint64_t)p * TK * ez * 4 : zline;
      MOE_DWG_COPY(lz + q * 1024, s);
    }
  };
  f32x16_t acc[ET];
#pragma unroll
  for (int j = 0; j < ET; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
  typedef const T __attribute__((address_space(3))) * lds_t_ptr;
  typedef const float __attribute__((address_space(3))) * lds_f_ptr;
  const int m = 32 * wave + l32;                                 // feature inside the tile
  constexpr int XE = 16 / sizeof(T);
  const uint32_t x_rd = hf * XP + (((m / XE) ^ (XSW * hf)) * 16) + (m % XE) * sizeof(T);
  uint32_t z_rd[ET];
#pragma unroll
  for (int j = 0; j < ET; ++j) z_rd[j] = kX + hf * ZP + (((8 * j + l32 / 4) ^ (ZSW * hf)) * 16) + (l32 % 4) * 4;
  int p = 0, pstage = 0, stage = 0;
  for (; p < ST - 1 && p < KT; ++p) start_step(p, pstage++);
  for (int s = 0; s < KT; ++s) {
    if (s + 1 < KT) {
      if (XQ + ZQ == 3) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
      else if (XQ + ZQ == 4) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      else if (XQ + ZQ == 5) asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
      else if (XQ + ZQ == 6) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    if (p < KT) {
      start_step(p, pstage);
      pstage = pstage + 1 == ST ? 0 : pstage + 1;
      ++p;
    }
    const uint32_t sb = lds0 + stage * kStage;
    stage = stage + 1 == ST ? 0 : stage + 1;
#pragma unroll
    for (int k = 0; k < TK / 2; ++k) {                           // tokens 2 k + hf
      float a;
      const T xv = *(lds_t_ptr)(uintptr_t)(sb + x_rd + k * 2 * XP);
      if constexpr (sizeof(T) == 2) a = bf16_to_f32(xv);
      else a = xv;
#pragma unroll
      for (int j = 0; j < ET; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, *(lds_f_ptr)(uintptr_t)(sb + z_rd[j] + k * 2 * ZP), acc[j], 0, 0, 0);
    }
  }
#undef MOE_DWG_COPY
  // acc[j][v]: feature 8 (v/4) + 4 hf + v%4 of the wavefront, expert 32 j + lane%32
  float* dst = partial + (size_t)blockIdx.z * M * ez;
#pragma unroll
  for (int j = 0; j < ET; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = m0 + 32 * wave + 8 * (v >> 2) + 4 * hf + (v & 3), e = e0 + 32 * j + l32;
      if (row < M && e < ez) dst[(size_t)row * ez + e] = acc[j][v];
    }
}

// dwg[m,e] = sum over the token ranges, 64 elements of [M, ez] per block: four threads per element add
// every fourth range, then their four sums (a fixed order)
__device__ __forceinline__ void dwg_sum(float* red, const float* __restrict__ partial, float* __restrict__ dwg,
                                        int block, int M, int E, int ez, int splits) {
  const int c = threadIdx.x & 63, k = threadIdx.x >> 6;
  const long long i = (long long)block * 64 + c;
  const long long size = (long long)M * ez;
  float acc = 0.f;
  if (i < size) {
#pragma unroll 8
    for (int s = k; s < splits; s += 4) acc += partial[s * size + i];
  }
  red[64 * k + c] = acc;
  __syncthreads();
  const int m = (int)(i / ez), e = (int)(i % ez);
  if (k == 0 && i < size && e < E)
    dwg[(size_t)m * E + e] = (red[c] + red[64 + c]) + (red[128 + c] + red[192 + c]);
}

// dwg[m,e] = sum over token ranges (in order) of the `terms` adjacent columns of e
__global__ __launch_bounds__(256) void dwg_reduce_kernel(
    const float* __restrict__ partial, float* __restrict__ dwg, int M, int E, int cols, int terms,
    int splits) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long long)M * E) return;
  const int m = (int)(i / E), e = (int)(i % E);
  float acc = 0.f;
  for (int s = 0; s < splits; ++s) {
    const float* p = partial + ((size_t)s * M + m) * cols + (size_t)terms * e;
    float t = p[0];
    for (int k = 1; k < terms; ++k) t += p[k];
    acc += t;
  }
  dwg[i] = acc;
}

// dx tile of 64 tokens x 128 features: the gate projection dz . wg^T in fp32 on the matrix cores, then
// the gradient rows of the token's kept choices are added (first, then second choice) and the sum is
// rounded once.  Wavefront = 32 tokens x 64 features; 32 experts of both operands at a time in LDS; the
// product (wg rows first, so a lane owns four consecutive features of a token) turns through LDS so that
// the rows of dbuf and dx move in 16-byte pieces.
// The first blocks add up dwg instead (dwg_sum): the same launch, since neither needs the other.
// Bound: the two dbuf rows read and the dx row written per token.  32 768 tokens, M 1024, E 32: 102 us as
// a bf16 GEMM with an fp32 result in memory and a pass that adds the rows -> 64 us; 3999 tokens, M 520,
// E 12: 21.5 us on FMA -> 9.1 us.
template <typename T>
__global__ __launch_bounds__(256) void dx_kernel(
    const float* __restrict__ dz, const float* __restrict__ wg, const T* __restrict__ dbuf,
    const int32_t* __restrict__ expert_idx, const int32_t* __restrict__ slot,
    T* __restrict__ dx, int S, int G, int C, int M, int E, int ez, int mtiles, long long tokens,
    const int32_t* __restrict__ row_base, const float* __restrict__ partial, float* __restrict__ dwg,
    int splits, int sum_blocks) {
  constexpr int P = 36, OP = 68;                                 // pitches: 4 mod 32 floats
  static_assert((128 + 64) * P <= 4 * 32 * OP, "the operands fit the space of the results");
  __shared__ __attribute__((aligned(16))) float ops[4 * 32 * OP];      // wg rows, dz rows; then the results
  __shared__ int rows_s[64][2];                                  // dbuf rows of the tokens' kept choices
  if ((int)blockIdx.x < sum_blocks) {
    dwg_sum(ops, partial, dwg, blockIdx.x, M, E, ez, splits);
    return;
  }
  const int block = blockIdx.x - sum_blocks;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, hf = lane >> 5;
  const long long n0 = (long long)(block / mtiles) * 64;
  const int m0 = block % mtiles * 128;
  const int wt = (wave >> 1) * 32, wm = (wave & 1) * 64;         // the wavefront's tokens, features
  if (tid < 128) {
    const long long n = n0 + (tid >> 1);
    const int k = tid & 1;
    int row = -1;
    if (n < tokens) {
      const int s = slot[2 * n + k];
      if (s >= 0) {
        // row of a kept choice: (e G + g) C + slot, or e G C + row_base[g,e] + slot when packed
        const int e = expert_idx[2 * n + k], g = (int)(n / S);
        row = row_base != nullptr ? e * G * C + row_base[(size_t)g * E + e] + s : (e * G + g) * C + s;
      }
    }
    rows_s[tid >> 1][k] = row;
  }
  // the dbuf pieces this lane adds at the end, requested first: they come from HBM behind the product
  constexpr int K = Vec16<T>::kElts, LPR = 64 / K, RPP = 64 / LPR;   // lanes per row, rows per pass
  const int m = m0 + wm + K * (lane % LPR);                      // M is a multiple of K
  uint4 drow[32 / RPP][2];
  __syncthreads();
#pragma unroll
  for (int ps = 0; ps < 32 / RPP; ++ps)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int row = rows_s[wt + RPP * ps + lane / LPR][k];
      drow[ps][k] = uint4{0u, 0u, 0u, 0u};
      if (row >= 0 && m < M) drow[ps][k] = *reinterpret_cast<const uint4*>(dbuf + (size_t)row * M + m);
    }
  f32x16_t acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
  float* zs = ops + 128 * P;
  const bool quads = (E & 3) == 0;                               // rows of wg are whole 16-byte pieces
  for (int e0 = 0; e0 < E; e0 += 32) {
    if (e0 > 0) __syncthreads();                                 // the previous experts are multiplied
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = (tid >> 3) + 32 * i, c = 4 * (tid & 7), m = m0 + r;
      f32x4_t v = {0.f, 0.f, 0.f, 0.f};
      if (m < M) {
        const float* src = wg + (size_t)m * E + e0 + c;
        if (quads) {
          if (e0 + c < E) v = *reinterpret_cast<const f32x4_t*>(src);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (e0 + c + q < E) v[q] = src[q];
        }
      }
      *reinterpret_cast<f32x4_t*>(&ops[r * P + c]) = v;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (tid >> 3) + 32 * i, c = 4 * (tid & 7);
      const long long n = n0 + r;
      f32x4_t v = {0.f, 0.f, 0.f, 0.f};
      if (n < tokens) v = *reinterpret_cast<const f32x4_t*>(dz + n * ez + e0 + c);
      *reinterpret_cast<f32x4_t*>(&zs[r * P + c]) = v;
    }
    __syncthreads();
#pragma unroll
    for (int kg = 0; kg < 4; ++kg) {                             // experts 8 kg + 4 hf + q
      const f32x4_t b = *reinterpret_cast<const f32x4_t*>(&zs[(wt + l32) * P + 8 * kg + 4 * hf]);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f32x4_t a = *reinterpret_cast<const f32x4_t*>(&ops[(wm + 32 * j + l32) * P + 8 * kg + 4 * hf]);
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], acc[j], 0, 0, 0);
      }
    }
  }
  // acc[j][v]: token lane%32, feature 32 j + 8 (v/4) + 4 hf + v%4 of the wavefront
  __syncthreads();
  float* o = ops + wave * 32 * OP;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<f32x4_t*>(&o[l32 * OP + 32 * j + 8 * q + 4 * hf]) =
          f32x4_t{acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
  __builtin_amdgcn_wave_barrier();
  if (m >= M) return;
#pragma unroll
  for (int ps = 0; ps < 32 / RPP; ++ps) {
    const int r = RPP * ps + lane / LPR;
    const long long n = n0 + wt + r;
    if (n >= tokens) continue;
    float f[K];
#pragma unroll
    for (int i = 0; i < K; ++i) f[i] = o[r * OP + K * (lane % LPR) + i];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      float d[K];
      Vec16<T>::unpack(drow[ps][k], d);
#pragma unroll
      for (int i = 0; i < K; ++i) f[i] += d[i];
    }
    *reinterpret_cast<uint4*>(dx + n * M + m) = Vec16<T>::pack(f);
  }
}

}  // namespace

int launch_combine_bwd(const moe_config& c, const void* dy, const void* out, const void* x, const int32_t* src_token,
                       const int32_t* expert_idx, const int32_t* slot, const float* weight, void* dout, void* buf,
                       const int32_t* kept, const int32_t* row_base, const float* gates, const int32_t* c1,
                       const float* daux, const GateBwdWs& w, hipStream_t st) {
  const GateBwdPlan p = gate_bwd_plan(c);
  const int elt = c.act_dtype == MOE_F32 ? 4 : 2;
  const int vec_per_row = c.M * elt / 16;
  const long long tokens = (long long)c.G * c.S, rows = (long long)c.E * c.G * c.C;
  const long long tblocks = (tokens + kRowsPerBlock - 1) / kRowsPerBlock;
  const long long zblocks = kept != nullptr ? (long long)c.E * (256 / kZeroRows) : (rows + kZeroRows - 1) / kZeroRows;
  const GateGrad gate{gates, c1, daux, p.mfma ? nullptr : w.dz, p.mfma ? w.dzp : nullptr, p.ez, p.cols};
#define MOE_COMBINE_BWD(T)                                                                                              \
  hipLaunchKernelGGL(combine_bwd_kernel<T>, dim3((unsigned)(tblocks + zblocks)), dim3(256), 0, st,                      \
                     static_cast<const uint4*>(dy), static_cast<const uint4*>(out), static_cast<const uint4*>(x),       \
                     expert_idx, slot, weight, static_cast<uint4*>(dout), static_cast<uint4*>(buf), c.S, c.G, c.C, c.E, \
                     vec_per_row, tokens, (unsigned)tblocks, src_token, kept, row_base, gate)
  if (c.act_dtype == MOE_F32) MOE_COMBINE_BWD(float);
  else MOE_COMBINE_BWD(bf16_t);
#undef MOE_COMBINE_BWD
  return check_launch();
}

// three stages of 32 tokens: 128 features of x, 32 ET experts of dz
template <typename T, int ET> constexpr int kDwgLds = 3 * 32 * 128 * ((int)sizeof(T) + ET);

template <typename T, int ET>
static int prepare_dwg() {
  static LdsLimitOnce once;
  return ensure_lds_limit(once, reinterpret_cast<const void*>(dwg_partial_kernel<T, ET>), kDwgLds<T, ET>);
}

int prepare_backward() {
  const int rcs[] = {prepare_dwg<bf16_t, 1>(), prepare_dwg<bf16_t, 2>(), prepare_dwg<bf16_t, 4>(),
                     prepare_dwg<float, 1>(), prepare_dwg<float, 2>(), prepare_dwg<float, 4>()};
  for (int rc : rcs)
    if (rc != MOE_OK) return rc;
  return MOE_OK;
}

GateBwdPlan gate_bwd_plan(const moe_config& c) {
  GateBwdPlan p{};
  const long long tokens = (long long)c.G * c.S;
  const long long cols = ((long long)3 * c.E + 255) / 256 * 256;
  // up to 128 experts the products are small enough for full fp32 (dwg_partial_kernel, dx_kernel)
  p.mfma = c.act_dtype == MOE_BF16 && c.E > 128 && tokens % 256 == 0 && tokens <= 0x7fffffffLL &&
           cols <= 0x7fffffffLL && gemm_bf16_f32out_ok((int)tokens, c.M, (int)cols) &&
           gemm_bf16_f32out_ok(c.M, (int)cols, 128);
  if (p.mfma) {
    p.cols = (int)cols;
    // token ranges (a power of two of them, each a multiple of 32 tokens and at least 128)
    // so that there is about one 256x256 tile per compute unit
    const long long tiles = (long long)(c.M / 256) * (cols / 256);
    int s = 1;
    while ((long long)s * 2 * tiles <= 256 && (tokens / 32) % (s * 2) == 0 && tokens / (s * 2) >= 128)
      s *= 2;
    p.splits = s;
    p.dzp_bytes = (size_t)tokens * cols * 2;
    p.wgp_bytes = (size_t)c.M * cols * 2;
    p.dxg_bytes = (size_t)tokens * c.M * 4;
    p.partial_bytes = (size_t)s * c.M * cols * 4;
  } else {
    // token ranges of at least 128 tokens, about two blocks per compute unit
    p.ez = (c.E + 31) / 32 * 32;
    const long long tiles = (long long)((c.M + 127) / 128) * ((p.ez + 127) / 128);
    long long s = (512 + tiles - 1) / tiles;
    if (s > (tokens + 127) / 128) s = (tokens + 127) / 128;
    p.splits = (int)s;
    p.dz_bytes = (size_t)tokens * p.ez * 4;
    p.partial_bytes = (size_t)p.splits * c.M * p.ez * 4;
  }
  return p;
}

int launch_dwg(const moe_config& c, const void* x, const GateBwdWs& w, float* dwg, hipStream_t st) {
  const GateBwdPlan p = gate_bwd_plan(c);
  const long long tokens = (long long)c.G * c.S;
  const long long size = (long long)c.M * c.E;
  if (p.mfma) {
    // dwg = x^T . dz as one batched MFMA GEMM over the token ranges, the three bf16 terms of
    // dz side by side in the columns; the reduction adds ranges and terms in a fixed order
    const int rc = launch_gemm_bf16_f32out(true, x, w.dzp, w.partial, p.splits, c.M, p.cols,
                                           (int)(tokens / p.splits), st);
    if (rc != MOE_OK) return rc;
    hipLaunchKernelGGL(dwg_reduce_kernel, dim3((unsigned)((size + 255) / 256)), dim3(256), 0, st,
                       w.partial, dwg, c.M, c.E, p.cols, 3, p.splits);
    return check_launch();
  }
  const long long tps = ((tokens + p.splits - 1) / p.splits + 31) / 32 * 32;
  const int et = p.ez <= 32 ? 1 : p.ez <= 64 ? 2 : 4;
  const dim3 pgrid((unsigned)((c.M + 127) / 128), (unsigned)((p.ez + 32 * et - 1) / (32 * et)), (unsigned)p.splits);
#define MOE_DWG(T, ET)                                                                                 \
  {                                                                                                    \
    if (prepare_dwg<T, ET>() != MOE_OK) return MOE_EHIP;                                               \
    hipLaunchKernelGGL((dwg_partial_kernel<T, ET>), pgrid, dim3(256), (kDwgLds<T, ET>), st,            \
                       static_cast<const T*>(x), w.dz, w.partial, c.M, p.ez, tokens, (int)tps);        \
  }
  if (c.act_dtype == MOE_F32) {
    if (et == 1) MOE_DWG(float, 1) else if (et == 2) MOE_DWG(float, 2) else MOE_DWG(float, 4)
  } else {
    if (et == 1) MOE_DWG(bf16_t, 1) else if (et == 2) MOE_DWG(bf16_t, 2) else MOE_DWG(bf16_t, 4)
  }
#undef MOE_DWG
  return check_launch();                                         // the dx launch adds the ranges up
}

int launch_dx(const moe_config& c, const float* wg, const void* dbuf, const int32_t* expert_idx,
              const int32_t* slot, const GateBwdWs& w, void* dx, float* dwg, const int32_t* row_base,
              hipStream_t st) {
  const GateBwdPlan p = gate_bwd_plan(c);
  const long long tokens = (long long)c.G * c.S;
  if (p.mfma) {
    // gate projection dz . wg^T on the matrix cores (fp32 result), then one pass that adds
    // the gradient rows of the kept choices and rounds once
    const long long n = (long long)c.M * p.cols;
    hipLaunchKernelGGL(wg_pack_bwd_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, wg,
                       w.wgp, c.M, c.E, p.cols);
    if (check_launch() != MOE_OK) return MOE_EHIP;
    const int rc = launch_gemm_bf16_f32out(false, w.dzp, w.wgp, w.dxg, 1, (int)tokens, c.M, p.cols, st);
    if (rc != MOE_OK) return rc;
    const unsigned grid = (unsigned)((tokens + kRowsPerBlock - 1) / kRowsPerBlock);
    hipLaunchKernelGGL(dx_rows_kernel, dim3(grid), dim3(256), 0, st,
                       reinterpret_cast<const float4*>(w.dxg), static_cast<const uint4*>(dbuf),
                       expert_idx, slot, static_cast<uint4*>(dx), c.S, c.G, c.C, c.E, c.M / 8, tokens,
                       row_base);
    return check_launch();
  }
  const int mtiles = (c.M + 127) / 128;
  const long long blocks = (tokens + 63) / 64 * mtiles;
  const long long sum_blocks = ((long long)c.M * p.ez + 63) / 64;
  if (blocks + sum_blocks > 0x7fffffffLL) return MOE_EUNSUPPORTED;
#define MOE_DX(T)                                                                                      \
  hipLaunchKernelGGL(dx_kernel<T>, dim3((unsigned)(blocks + sum_blocks)), dim3(256), 0, st, w.dz, wg,  \
                     static_cast<const T*>(dbuf), expert_idx, slot, static_cast<T*>(dx), c.S, c.G, c.C, \
                     c.M, c.E, p.ez, mtiles, tokens, row_base, w.partial, dwg, p.splits, (int)sum_blocks)
  if (c.act_dtype == MOE_F32) MOE_DX(float); else MOE_DX(bf16_t);
#undef MOE_DX
  return check_launch();
}

}  // namespace moe
