// Scaled dot-product attention on the matrix cores, forward and backward (bf16, d = 64 or 128, any L).  Section 2.1 of
// the paper names the self-attention sub-layer; the derivative is the chain rule of ctx = softmax(q k^T / sqrt(d)) v, with
// the probabilities recomputed from q, k and the stored row statistic lse = log sum_k exp(score):
//
//   p = exp(score - lse),  D = rowsum(dctx * ctx),  dv = p^T dctx,
//   ds = p * (dctx v^T - D) / sqrt(d),  dq = ds k,  dk = ds^T q
//
// Everything is transposed so that a lane owns one column of a score tile:
//
//   forward   a wavefront owns 32 queries: S^T = K Q^T, online softmax, O^T += V^T P^T
//   dq        32 queries: S^T = K Q^T, dP^T = V dO^T, dQ^T += K^T dS^T; also writes D
//   dk, dv    32 CT keys: S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS
//
// MFMA register layout (v_mfma_f32_32x32x16_bf16): lane (r = lane % 32, hf = lane / 32) supplies row r of the first
// operand and column r of the second, k = 8 hf .. 8 hf + 7 of the step; it receives C[8 (i/4) + 4 hf + i%4][r] in value
// i.  Values 8 s .. 8 s + 7 of a score tile are therefore exactly what the lane owes step s of the next product, for the
// rows 16 s + 8 (j/4) + 4 hf + j%4, which the transposing LDS read fetches in that order.
//
// Four wavefronts per block share blocks of 64 rows of the other side.  These are staged by register-bypassing copies, one
// step ahead, and once: chunk c of row r sits at c ^ att_swizzle(r), which puts the same chunk of 16 consecutive rows
// (16-byte row reads) and four chunks of four rows (transposing reads) into different banks.  Products, exponentials and
// LDS reads take turns unless something interleaves them, and the compiler does not (its scheduler gives up on loops of
// this size), so a step is a list of units, each one fragment read, its products and the vector work that
// runs under them, in program order (run_units).  dk, dv: one tile of 32 keys per wavefront, or for d 128 and many
// blocks two, each fragment then feeding two products (512 registers).
//
// Before, 32-column kernels staged through registers, K (dq) or Q and dO (dk, dv) twice, and left the interleaving to
// scheduling hints; they were busy multiplying a quarter of the time.  us before / now: forward, dq, dk and dv of 16 x 1024
// tokens, 16 heads of 128 180 / 155, 307 / 198, 487 / 268 (0.89, 1.04 and 1.03 PFLOP/s now); of 2 x 1024, 4 heads of 128
// 28.6 / 23.2, 49.4 / 26.4, 47.6 / 31.5; of 62 x 1024, 4 heads of 64 57.4 / 47.2, 69.1 / 59.3, 145 / 75; of 42 x 700, 4 heads
// of 128 98 / 88, 118 / 113, 263 / 187.  What bounds them now (32 x 1024 tokens, 16 heads): the matrix
// pipes are busy 47, 62 and 53 % of forward, dq, dk and dv, at the 1.6 to 1.9 of 2.4 GHz that power leaves, the vector ALU
// 66, 55 and 39 %; for dk and dv also the first rows of a block, which nothing overlaps.
//
// Short ragged sequences have kernels of their own with less on the way to the first product: attention_short_kernel,
// attention_bwd_dq_short_kernel.  Without one: dk and dv of up to 33 tokens, d 64, in up to 192 blocks took 0.2 us of 6 less in
// the kernels before these (1.4 to 2.1 times as long in more blocks), forward of 65 to 80 tokens 0.3 of 7.
//
// RAGGED: L is no multiple of 128.  Rows past the end are staged as zeros; their scores become -inf (forward), their part
// of P and dS 0; columns past the end are computed from row L - 1 and not stored, and a wavefront without
// others only stages.  P and dS stay fp32, as in the plain kernels that served these lengths first: they enter
// the products as three bf16 terms (split_bf16x8), so ctx, dq, dk and dv differ from float64 by their own rounding and 2e-7 of
// the sum's magnitude.  L % 128 == 0 keeps the form without these tests, whose P and dS are rounded to bf16 (2e-3 of it).
#include <math.h>
#include <float.h>
#include <type_traits>
#include <utility>
#include "common.h"

namespace moe {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef s16x4_t __attribute__((address_space(3))) * lds_s16x4_ptr;
typedef u32x4_t __attribute__((address_space(3))) * lds_u4_ptr;
typedef f32x4_t __attribute__((address_space(3))) * lds_f4_ptr;
typedef unsigned char __attribute__((address_space(3))) * lds_ptr;

static __device__ const u32x4_t att_zero_line = {0u, 0u, 0u, 0u};

template <int D> struct AttGeom {
  static constexpr int kRow = 2 * D, kChunks = D / 8, kBlock = 64 * kRow;      // bytes, 16-byte chunks, bytes
  static constexpr int kRowsPerCopy = 1024 / kRow, kCopies = kBlock / 4096;    // 1 KB copies per wavefront
};
template <int D>
__device__ __forceinline__ constexpr int att_swizzle(int row) {
  return D == 128 ? ((row & 3) << 2) | ((row >> 2) & 3) : (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}

#define MOE_MFMA(a, b, c)                                                                      \
  __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),                      \
                                          __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0)
// acc += a . b with acc in accumulation registers (gradients, whose tiles no vector instruction touches).  Score tiles, which
// vector instructions read, stay in vector registers (builtin above, and see the build's flag for this file): left to
// itself the compiler puts all results of a kernel into one kind and copies.  It does not see what this instruction asks
// for: 2 wait states after a vector instruction that wrote a or b (fresh_operand) and 11 before anything but the next product
// into it touches acc (settle_all; 19 for longer products).  Both stand where the source needs them; that the compiler
// puts no copy or spill in between is read from the compiled code by tests/test_attention_wait_states.py.
__device__ __forceinline__ void mfma_acc(f32x16_t& acc, const u32x4_t& a, const u32x4_t& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void fresh_operand() { asm volatile("s_nop 1"); }
// zeros in accumulation registers
__device__ __forceinline__ void clear_acc(f32x16_t& acc) {
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  asm volatile("" : "+a"(acc));
}

// f(0), f(1), .. f(N - 1), the argument a constant
template <typename F, int... I>
__device__ __forceinline__ void unroll_list(std::integer_sequence<int, I...>, F&& f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void unroll(F&& f) { unroll_list(std::make_integer_sequence<int, N>{}, f); }
// A step as units FIRST .. N - 1.  Unit u's fragment is fetched AHEAD units early by read(u); count(u) products use it, and after
// product p comes a share of the vector work, side(u, p, n): one wavefront issues in order, so what is to run under
// a product stands right behind it, and a second product right behind the first would only wait for the pipe.  Fences
// keep it that way.
template <int FIRST, int N, int AHEAD, typename Count, typename Read, typename Multiply, typename Side>
__device__ __forceinline__ void run_units(Count&& count, Read&& read, Multiply&& multiply, Side&& side) {
  u32x4_t f[AHEAD + 1];
  unroll<AHEAD>([&](auto I) __attribute__((always_inline)) {
    constexpr int u = FIRST + decltype(I)::value;
    f[u % (AHEAD + 1)] = read(std::integral_constant<int, u>{});
  });
  unroll<N - FIRST>([&](auto I) __attribute__((always_inline)) {
    constexpr std::integral_constant<int, FIRST + decltype(I)::value> U{};
    constexpr int u = FIRST + decltype(I)::value;
    constexpr int n = decltype(count(U))::value;
    if constexpr (u + AHEAD < N) f[(u + AHEAD) % (AHEAD + 1)] = read(std::integral_constant<int, u + AHEAD>{});
    unroll<n>([&](auto P) __attribute__((always_inline)) {
      multiply(U, P, f[u % (AHEAD + 1)]);
      __builtin_amdgcn_sched_barrier(0);
      side(U, P, std::integral_constant<int, n>{});
      __builtin_amdgcn_sched_barrier(0);
    });
  });
}

// wait states between the last products into the tiles and reads of them
template <int CT, int DT>
__device__ __forceinline__ void settle_all(f32x16_t (&a)[CT][DT]) {
  asm volatile("s_nop 15\n\ts_nop 3" : "+a"(a[0][0]));
#pragma unroll
  for (int i = 1; i < CT * DT; ++i) asm volatile("" : "+a"(a[i / DT][i % DT]));
}

template <typename V>
__device__ __forceinline__ u32x4_t pack8(const V& v, int first) {
  return u32x4_t{pack_bf16x2(v[first], v[first + 1]), pack_bf16x2(v[first + 2], v[first + 3]),
                 pack_bf16x2(v[first + 4], v[first + 5]), pack_bf16x2(v[first + 6], v[first + 7])};
}
// the terms of a fragment of P or dS: three bf16 terms that hold all 24 bits, or one rounded to bf16
template <int TERMS, typename V>
__device__ __forceinline__ void fragment_terms(const V& v, int first, bf16x8_bits_t (&t)[TERMS]) {
  if constexpr (TERMS == 3) split_bf16x8(v, first, t);
  else t[0] = pack8(v, first);
}
// dS = p (dp - D), rounded.  The compiler fused it with the subtractions of split_bf16x8 in some kernels and not in others: the
// terms were then those of the unrounded product, and a sequence's dq would depend on the kernel that forms it.
__device__ __forceinline__ float dscore(float p, float dp, float D) {
#pragma clang fp contract(off)
  return p * (dp - D);
}
// Every XCD (own L2) takes a contiguous range of work items: the blocks of one (sequence, head) read the same rows.
__device__ __forceinline__ unsigned xcd_contiguous(unsigned block, unsigned blocks) {
  const unsigned per_xcd = blocks / 8;
  return block < per_xcd * 8 ? (block % 8) * per_xcd + block / 8 : block;
}

// Per-lane byte offsets of this wavefront's copies of a block of 64 rows, `ld` elements apart.
template <int D>
__device__ __forceinline__ void copy_offsets(uint32_t (&off)[AttGeom<D>::kCopies], size_t ld, int wave, int lane) {
  using GM = AttGeom<D>;
#pragma unroll
  for (int q = 0; q < GM::kCopies; ++q) {
    const int row = GM::kRowsPerCopy * (GM::kCopies * wave + q) + lane / GM::kChunks;
    off[q] = (uint32_t)(row * ld * 2) + 16 * ((lane % GM::kChunks) ^ att_swizzle<D>(row));
  }
}
// Start copy q of this wavefront of the rows first .. first + 63 (RAGGED: zeros from row L on) to the LDS block at `lds`.
template <int D, bool RAGGED>
__device__ __forceinline__ void stage_copy(uint32_t lds, const bf16_t* rows, size_t ld, int first, int L,
                                           const uint32_t (&off)[AttGeom<D>::kCopies], int q, int wave, int lane) {
  using GM = AttGeom<D>;
  const bf16_t* const src = rows + (size_t)first * ld;
  lds += (wave * GM::kCopies + q) * 1024;
  if (RAGGED && first + 64 > L) {
    const int row = first + GM::kRowsPerCopy * (GM::kCopies * wave + q) + lane / GM::kChunks;
    const uint64_t at = row < L ? (uint64_t)(uintptr_t)src + off[q] : (uint64_t)(uintptr_t)&att_zero_line;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(at) : "memory");
  } else {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off[q]), "s"(src) : "memory");
  }
}
// Start the copies of the wavefront's own 32 CT rows (row L - 1 in place of those past it) to its own LDS block.
template <int D, int CT>
__device__ __forceinline__ void stage_own(uint32_t lds, const bf16_t* rows, size_t ld, int first, int L, int lane) {
  using GM = AttGeom<D>;
#pragma unroll
  for (int q = 0; q < 32 * CT * GM::kRow / 1024; ++q) {
    const int row = GM::kRowsPerCopy * q + lane / GM::kChunks, at = first + row < L ? first + row : L - 1;
    const uint64_t src = (uint64_t)(uintptr_t)(rows + (size_t)at * ld + 8 * ((lane % GM::kChunks) ^ att_swizzle<D>(row)));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds + q * 1024), "v"(src) : "memory");
  }
}
__device__ __forceinline__ void wait_all_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// LDS addresses, relative to a staged block, of a lane's fragments.
//   rows:       lane (r, hf) reads d = 16 s + 8 hf .. + 7 of row 32 t + r
//   transposed: lane needs d = 32 dt + lane%32 of the rows 16 s + 4 hf .. + 3 (x = 0) and 16 s + 8 + 4 hf .. + 3
//               (x = 1), the k order in which a result tile's registers already hold the other operand
template <int D>
struct AttReads {
  using GM = AttGeom<D>;
  uint32_t row0, tr0;
  __device__ __forceinline__ AttReads(uint32_t lds0, int lane) {
    const int r = lane & 31, hf = lane >> 5, p16 = lane & 15, b1 = (lane >> 4) & 1, rr = p16 >> 2;
    row0 = lds0 + r * GM::kRow + ((hf ^ att_swizzle<D>(r)) << 4);
    const int sw = D == 128 ? rr << 2 : (rr >> 1) << 2;
    tr0 = lds0 + (4 * hf + rr) * GM::kRow + ((((2 * b1 + ((p16 >> 1) & 1)) ^ hf) ^ sw) << 4) + 8 * (p16 & 1);
  }
  __device__ __forceinline__ u32x4_t row(uint32_t block, int t, int s) const {
    return *(lds_u4_ptr)(uintptr_t)((row0 ^ (s << 5)) + block + t * 32 * GM::kRow);
  }
  __device__ __forceinline__ u32x4_t transposed(uint32_t block, int row16, int dt) const {
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)((tr0 ^ (dt << 6)) + block + row16 * GM::kRow));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4_ptr)(uintptr_t)((tr0 ^ (dt << 6) ^ 32) + block + (row16 + 8) * GM::kRow));
    return __builtin_bit_cast(u32x4_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// the block's (sequence, head), its first column, and the wavefront's
template <int CT> struct AttWork {
  long long bh, b;
  int h, col0;
  __device__ __forceinline__ AttWork(int L, int heads, int wave) {
    const int blocks = (L + 128 * CT - 1) / (128 * CT);
    const unsigned work = xcd_contiguous(blockIdx.x, gridDim.x);
    bh = work / blocks;
    h = (int)(bh % heads);
    b = bh / heads;
    col0 = (int)(work % blocks) * (128 * CT) + wave * (32 * CT);
  }
};

// The wavefront's result tiles, element (d = 32 dt + 8 (i/4) + 4 hf + i%4, column 32 c + r) times factor, as whole
// rows of the columns first .. (not from L on), turned through the wavefront's own LDS block at `lds`.
template <int D, int CT>
__device__ __forceinline__ void store_own(const f32x16_t (&acc)[CT][D / 32], float factor, uint32_t lds, bf16_t* rows,
                                          size_t ld, int first, int L, int lane) {
  using GM = AttGeom<D>;
  typedef u32x2_t __attribute__((address_space(3))) * lds_u2_ptr;
  const int r = lane & 31, hf = lane >> 5;
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(lds_u2_ptr)(uintptr_t)(lds + (32 * c + r) * GM::kRow + (((4 * dt + g) ^ att_swizzle<D>(r)) << 4) + 8 * hf) =
            u32x2_t{pack_bf16x2(acc[c][dt][4 * g] * factor, acc[c][dt][4 * g + 1] * factor),
                    pack_bf16x2(acc[c][dt][4 * g + 2] * factor, acc[c][dt][4 * g + 3] * factor)};
#pragma unroll
  for (int q = 0; q < 32 * CT * GM::kRow / 1024; ++q) {
    const int row = GM::kRowsPerCopy * q + lane / GM::kChunks, chunk = lane % GM::kChunks;
    const u32x4_t v = *(lds_u4_ptr)(uintptr_t)(lds + row * GM::kRow + ((chunk ^ att_swizzle<D>(row)) << 4));
    if (first + row < L) *reinterpret_cast<u32x4_t*>(rows + (size_t)(first + row) * ld + 8 * chunk) = v;
  }
}

// ---------------------------------------------------------------- staging of the short ragged kernels
// Blocks of 64 rows through registers into LDS, the rows of a transposing read in an order of their own.
template <int D> struct ShortGeom {          // row pitches: 16-byte row reads 4 banks apart, transposing reads 16
  static constexpr int kRowPitch = D * 2 + 16, kTrPitch = D * 2 + 64;
  static constexpr int kRowBlock = 64 * kRowPitch, kTrBlock = 64 * kTrPitch;
};
__device__ __forceinline__ int swap_bits_2_3(int row) {
  return (row & ~12) | ((row & 4) << 1) | ((row & 8) >> 1);
}
// first operand fragment [32 d-rows x 16 staged rows] of a block staged [rows][d] with the
// transposing pitch: lane needs (d = 32 dt + lane%32, 8 consecutive staged rows of its half)
template <int PITCH>
__device__ __forceinline__ bf16x8_t read_transposed(uint32_t block, int row16, int dt, int lane) {
  const int p16 = lane & 15, bb = lane >> 4;
  const int krow0 = 8 * (bb >> 1) + (p16 >> 2);
  const int col = 32 * dt + 16 * (bb & 1) + 4 * (p16 & 3);
  const uint32_t pv = block + (row16 + krow0) * PITCH + 2 * col;
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)pv);
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(pv + 4 * PITCH));
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// ---------------------------------------------------------------- forward
template <int D, bool RAGGED>
__global__ __launch_bounds__(256, 2) void attention_mfma_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ ctx,
                                                                float* __restrict__ lse, int L, int heads) {
  using GM = AttGeom<D>;
  constexpr int CT = 1, KS = D / 16, DT = D / 32, TERMS = RAGGED ? 3 : 1, kOwnBlock = 32 * CT * GM::kRow;
  constexpr int kV = 2 * GM::kBlock;                           // LDS: two K blocks, two V blocks
  extern __shared__ __attribute__((aligned(256))) unsigned char att_lds[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_ptr)att_lds);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, hf = lane >> 5;
  const AttWork<CT> w(L, heads, wave);
  const int A = heads * D;
  const size_t ld = (size_t)3 * A;
  const bf16_t* const base = qkv + (size_t)w.b * L * ld + (size_t)w.h * D;
  const bool live = w.col0 < L;

  uint32_t off[GM::kCopies];
  copy_offsets<D>(off, ld, wave, lane);
  const int nkb = (L + 63) / 64;
  // copy x of step j's: K block j + 1 (after the last one, that once more), V block j
  auto start = [&](int j, int x) __attribute__((always_inline)) {
    const int k = j + 1 < nkb ? j + 1 : nkb - 1, v = j;
    if (x < GM::kCopies) stage_copy<D, RAGGED>(lds0 + ((j + 1) & 1) * GM::kBlock, base + A, ld, 64 * k, L, off, x, wave, lane);
    else stage_copy<D, RAGGED>(lds0 + kV + (j & 1) * GM::kBlock, base + 2 * A, ld, 64 * v, L, off, x - GM::kCopies, wave, lane);
  };
  constexpr int COPIES = 2 * GM::kCopies;
  // the wavefront's own rows come (and its results go) through the second places of K and V
  const uint32_t own = GM::kBlock + (wave & 1) * kOwnBlock + (wave >> 1) * kV;
#pragma unroll
  for (int x = 0; x < GM::kCopies; ++x) { start(-1, x); start(0, GM::kCopies + x); }     // K and V block 0
  if (live) stage_own<D, CT>(lds0 + own, base, ld, w.col0, L, lane);
  wait_all_copies();

  const float sl2 = 1.4426950408889634f / sqrtf((float)D);
  const AttReads<D> rd(lds0, lane);
  u32x4_t qf[KS];                                              // Q^T fragments: lane (r, hf) holds d = 16 s + 8 hf .. + 7
  f32x16_t o[DT];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    qf[s] = rd.row(own, 0, s);
    asm volatile("" : "+v"(qf[s]) :: "memory");
  }
  __syncthreads();
  if (nkb > 1) {
#pragma unroll
    for (int x = 0; x < GM::kCopies; ++x) start(0, x);         // K block 1
  }
  if (!live) {                                                 // a wavefront without columns only stages
    for (int kb = 0; kb + 1 < nkb; ++kb) {
      wait_all_copies();
      __syncthreads();
#pragma unroll
      for (int x = 0; x < COPIES; ++x) start(kb + 1, x);
    }
    wait_all_copies();
    __syncthreads();
    __syncthreads();
    return;
  }
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[t][i] = 0.f;
  // running maximum (in log2 units) and sum; the maximum starts finite, so that a block of keys whose scores
  // are all -inf adds nothing
  float m_run = -FLT_MAX, l_run = 0.f, m_new;
  f32x16_t sacc[2];                                            // scores of block kb [32-key tile], and the maximum with them
  auto mask_end = [&](f32x16_t (&acc)[2], int kb) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (kb * 64 + 32 * t + 8 * (i >> 2) + 4 * hf + (i & 3) >= L) acc[t][i] = -INFINITY;
  };
  auto block_max = [&](const f32x16_t (&acc)[2]) __attribute__((always_inline)) {
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc[t][i]);
    return mx;
  };
  auto new_max = [&](float mx) __attribute__((always_inline)) {
    m_new = fmaxf(m_run, fmaxf(mx, __shfl_xor(mx, 32, 64)) * sl2);        // sl2 > 0: scaling commutes with max
  };
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int s = 0; s < KS; ++s) sacc[t] = MOE_MFMA(rd.row(0, t, s), qf[s], s == 0 ? f32x16_t{} : sacc[t]);
  if (RAGGED && 64 > L) mask_end(sacc, 0);
  new_max(block_max(sacc));

  // One block of keys; after the LAST there are no scores to multiply ahead.
  auto step = [&](int kb, auto last) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last)::value;
    constexpr int FIRST = LAST ? 2 * KS : 0;                   // (units 0 .. 2 KS - 1 are those scores)
    wait_all_copies();                                         // K block kb + 1 and V block kb are there;
    __syncthreads();                                           // K block kb and V block kb - 1 are read, their places free
    const uint32_t kst = ((kb + 1) & 1) * GM::kBlock, vst = kV + (kb & 1) * GM::kBlock;
    // rescale only when some query of the wavefront needs it (alpha == 1 exactly otherwise)
    if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on the first block
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[t][i] *= alpha;
    }
    m_run = m_new;
    float psum = 0.f, mx = -INFINITY;
    f32x16_t snext[2];
    bf16x8_bits_t pf[2][TERMS];                                // P^T, k step % 2
    auto exponentials = [&](int t, int first, int last) __attribute__((always_inline)) {
#pragma unroll
      for (int i = first; i < last; ++i) {
        const float v = __builtin_amdgcn_exp2f(fmaf(sacc[t][i], sl2, -m_run));
        sacc[t][i] = v;
        psum += v;
      }
    };
    if constexpr (LAST) {
      exponentials(0, 0, 16);
      fragment_terms(sacc[0], 0, pf[0]);
      fragment_terms(sacc[0], 8, pf[1]);
    }
    // units 0 .. 2 KS - 1: scores of block kb + 1, under them the first tile's exponentials; then 4 DT units of O^T, under
    // them the second tile's and the next block's maximum
    run_units<FIRST, 2 * KS + 4 * DT, 4>(
        [&](auto U) __attribute__((always_inline)) { return std::integral_constant<int, decltype(U)::value < 2 * KS ? 1 : TERMS>{}; },
        [&](auto U) __attribute__((always_inline)) {
          constexpr int u = decltype(U)::value, v = u - 2 * KS;
          if constexpr (u < 2 * KS) return rd.row(kst, u / KS, u % KS);
          else return rd.transposed(vst, 16 * (v / DT), v % DT);
        },
        [&](auto U, auto P, const u32x4_t& f) __attribute__((always_inline)) {
          constexpr int u = decltype(U)::value, v = u - 2 * KS, k = TERMS - 1 - decltype(P)::value;
          if constexpr (u < 2 * KS) snext[u / KS] = MOE_MFMA(f, qf[u % KS], u % KS == 0 ? f32x16_t{} : snext[u / KS]);
          else o[v % DT] = MOE_MFMA(f, pf[(v / DT) % 2][k], o[v % DT]);          // smallest term first
        },
        [&](auto U, auto P, auto NP) __attribute__((always_inline)) {
          constexpr int u = decltype(U)::value, v = u - 2 * KS, p = decltype(P)::value, n = decltype(NP)::value;
          if constexpr (!LAST && u < COPIES && p == 0) start(kb + 1, u);
          if constexpr (u < 2 * KS) {
            exponentials(0, u * 8 / KS, (u + 1) * 8 / KS);
            if constexpr (u == KS + 1) fragment_terms(sacc[0], 0, pf[0]);
            if constexpr (u == 2 * KS - 1) fragment_terms(sacc[0], 8, pf[1]);
          } else if constexpr (v < 2 * DT) {
            constexpr int x = n * v + p, all = 2 * DT * n;
            exponentials(1, x * 16 / all, (x + 1) * 16 / all);
            // the terms of k step 0 are free after DT units, the second tile's first 8 values done by then
            if constexpr (v == DT && p == 0) fragment_terms(sacc[1], 0, pf[0]);
          } else {
            if constexpr (v == 2 * DT && p == 0) fragment_terms(sacc[1], 8, pf[1]);
            constexpr int x = n * (v - 2 * DT - 1) + p, all = (2 * DT - 1) * n;
            if constexpr (!LAST && x >= 0) {
#pragma unroll
              for (int j = x * 32 / all; j < (x + 1) * 32 / all; ++j) mx = fmaxf(mx, snext[j >> 4][j & 15]);
            }
          }
        });
    l_run += psum + __shfl_xor(psum, 32, 64);
    if constexpr (LAST) return;
    if (RAGGED && kb + 2 == nkb) {                             // the last block comes next: without its keys past the end
      mask_end(snext, kb + 1);
      mx = block_max(snext);
    }
    new_max(mx);
    sacc[0] = snext[0];
    sacc[1] = snext[1];
  };
  for (int kb = 0; kb + 1 < nkb; ++kb) step(kb, std::false_type{});
  step(nkb - 1, std::true_type{});
  __syncthreads();                                             // the other wavefronts have read the last blocks
  const int q = w.col0 + r;
  // row statistic for the backward pass: log sum_k exp(score) in natural-log units
  if (lse != nullptr && hf == 0 && q < L) lse[(size_t)w.bh * L + q] = (m_run + log2f(l_run)) * 0.6931471805599453f;
  const f32x16_t (&tiles)[1][DT] = reinterpret_cast<const f32x16_t (&)[1][DT]>(o);
  store_own<D, CT>(tiles, 1.0f / l_run, lds0 + own, ctx + (size_t)w.b * L * A + (size_t)w.h * D, A, w.col0, L, lane);
}

// ---------------------------------------------------------------- forward of one block of keys (L <= 64)
// The sums of the kernel above without its loop: K and V through registers, the queries' rows straight from memory and
// the results straight to it.  What counts here is the way to the first product, and room for more blocks on a unit (91 or
// 127 registers instead of 182 or 250).  us, the kernel above / this one: d 64, 8 sequence-heads of 16 tokens 4.9 / 4.3, 520 of 48
// 9.2 / 5.8, 2200 of 64 21.2 / 17.7; d 128, 64 of 48 6.9 / 6.4, 1000 of 48 16.7 / 13.9, but 4000 of 48 51.7 / 50.9, 400 of 64
// 9.6 / 10.1 and 4000 of 64 55.6 / 65.8: rows of 256 bytes read and written piece by piece are what it waits for then.
template <int D>
__global__ __launch_bounds__(256, 2) void attention_short_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ ctx,
                                                                 float* __restrict__ lse, int L, int heads) {
  using GM = ShortGeom<D>;
  constexpr int KS = D / 16, DT = D / 32, VV = 64 * D / 8 / 256, VPR = D / 8;
  __shared__ __attribute__((aligned(256))) unsigned char kv[GM::kRowBlock + GM::kTrBlock];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, hf = lane >> 5;
  const unsigned bh = xcd_contiguous(blockIdx.x, gridDim.x);
  const int h = (int)(bh % heads);
  const long long b = bh / heads;
  const int A = heads * D;
  const size_t ld = (size_t)3 * A;
  const bf16_t* const base = qkv + (size_t)b * L * ld + (size_t)h * D;
  const int q = wave * 32 + r;

  u32x4_t qf[KS], kreg[VV], vreg[VV];
#pragma unroll
  for (int s = 0; s < KS; ++s) qf[s] = *reinterpret_cast<const u32x4_t*>(base + (size_t)(q < L ? q : L - 1) * ld + 16 * s + 8 * hf);
#pragma unroll
  for (int i = 0; i < VV; ++i) {
    const int f = tid + 256 * i, key = f / VPR;
    const bf16_t* const row = base + (size_t)(key < L ? key : L - 1) * ld + 8 * (f % VPR);
    kreg[i] = *reinterpret_cast<const u32x4_t*>(row + A);
    vreg[i] = *reinterpret_cast<const u32x4_t*>(row + 2 * A);
  }
#pragma unroll
  for (int i = 0; i < VV; ++i) {
    const int f = tid + 256 * i, key = f / VPR, c = f % VPR;
    *reinterpret_cast<u32x4_t*>(kv + key * GM::kRowPitch + 16 * c) = kreg[i];
    *reinterpret_cast<u32x4_t*>(kv + GM::kRowBlock + swap_bits_2_3(key) * GM::kTrPitch + 16 * c) = key < L ? vreg[i] : u32x4_t{0u, 0u, 0u, 0u};
  }
  __syncthreads();
  if (wave * 32 >= L) return;
  const uint32_t kst = (uint32_t)(uintptr_t)((lds_ptr)kv), vst = kst + GM::kRowBlock;
  const float sl2 = 1.4426950408889634f / sqrtf((float)D);
  f32x16_t sacc[2], o[DT];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const u32x4_t kf = *(lds_u4_ptr)(uintptr_t)(kst + (32 * t + r) * GM::kRowPitch + 32 * s + 16 * hf);
      sacc[t] = MOE_MFMA(kf, qf[s], s == 0 ? f32x16_t{} : sacc[t]);
    }
  float mx = -INFINITY, psum = 0.f;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (32 * t + 8 * (i >> 2) + 4 * hf + (i & 3) >= L) sacc[t][i] = -INFINITY;
      mx = fmaxf(mx, sacc[t][i]);
    }
  const float m = fmaxf(-FLT_MAX, fmaxf(mx, __shfl_xor(mx, 32, 64)) * sl2);
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      sacc[t][i] = __builtin_amdgcn_exp2f(fmaf(sacc[t][i], sl2, -m));
      psum += sacc[t][i];
    }
  psum += __shfl_xor(psum, 32, 64);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x16_t{};
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    bf16x8_bits_t pf[3];
    split_bf16x8(sacc[s / 2], 8 * (s % 2), pf);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const bf16x8_t vt = read_transposed<GM::kTrPitch>(vst, 16 * s, dt, lane);
#pragma unroll
      for (int k = 2; k >= 0; --k) o[dt] = MOE_MFMA(vt, pf[k], o[dt]);
    }
  }
  if (q >= L) return;
  const float inv = 1.0f / psum;
  if (lse != nullptr && hf == 0) lse[(size_t)bh * L + q] = (m + log2f(psum)) * 0.6931471805599453f;
  // o[dt][i]: d = 32 dt + 8 (i/4) + 4 hf + i%4 of query r
  bf16_t* const row = ctx + ((size_t)b * L + q) * A + (size_t)h * D;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<u32x2_t*>(row + 32 * dt + 8 * g + 4 * hf) =
          u32x2_t{pack_bf16x2(o[dt][4 * g] * inv, o[dt][4 * g + 1] * inv), pack_bf16x2(o[dt][4 * g + 2] * inv, o[dt][4 * g + 3] * inv)};
}

// ---------------------------------------------------------------- dq (and D)
template <int D, bool RAGGED>
__global__ __launch_bounds__(256, 2) void attention_bwd_dq_mfma_kernel(
    const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ ctx, const bf16_t* __restrict__ dctx,
    const float* __restrict__ lse, bf16_t* __restrict__ dqkv, float* __restrict__ dvec, int L, int heads) {
  using GM = AttGeom<D>;
  constexpr int CT = 1, KS = D / 16, DT = D / 32, TERMS = RAGGED ? 3 : 1, kOwnBlock = 32 * CT * GM::kRow;
  // LDS: three K blocks, two V blocks; the wavefronts' own rows go through all of their places but the first, so that
  // two blocks share a compute unit
  constexpr bool PEEL = !RAGGED;
  constexpr int kV = 3 * GM::kBlock, kQ = GM::kBlock, kGrad = kQ + 4 * kOwnBlock;
  extern __shared__ __attribute__((aligned(256))) unsigned char att_lds[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_ptr)att_lds);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, hf = lane >> 5;
  const AttWork<CT> w(L, heads, wave);
  const int A = heads * D;
  const size_t ld = (size_t)3 * A;
  const bf16_t* const base = qkv + (size_t)w.b * L * ld + (size_t)w.h * D;
  const bool live = w.col0 < L;

  uint32_t off[GM::kCopies];
  copy_offsets<D>(off, ld, wave, lane);
  const int nkb = (L + 63) / 64;
  // copy x of step j's: K block j + 1 to place `slot`, V block j (after the last ones, those once more)
  auto start = [&](int j, int slot, int x) __attribute__((always_inline)) {
    const int k = j + 1 < nkb ? j + 1 : nkb - 1, v = j < nkb ? j : nkb - 1;
    if (x < GM::kCopies) stage_copy<D, RAGGED>(lds0 + slot * GM::kBlock, base + A, ld, 64 * k, L, off, x, wave, lane);
    else stage_copy<D, RAGGED>(lds0 + kV + (j & 1) * GM::kBlock, base + 2 * A, ld, 64 * v, L, off, x - GM::kCopies, wave, lane);
  };
  constexpr int COPIES = 2 * GM::kCopies;

  // Q^T and dO^T fragments of this wavefront's queries, D and lse of the lane's.  The rows come through LDS: read as
  // fragments from memory, 16 bytes of 32 rows at a time, they take longer (O, one of three, hides behind the others).
  const uint32_t own = kQ + wave * kOwnBlock;
  const size_t head = (size_t)w.b * L * A + (size_t)w.h * D;
  const float scale = 1.0f / sqrtf((float)D), sl2 = 1.4426950408889634f * scale;
  const AttReads<D> rd(lds0, lane);
  u32x4_t qf[CT][KS], dof[CT][KS], of[CT][KS];
#pragma unroll
  for (int x = 0; x < GM::kCopies; ++x) start(-1, 0, x);       // K block 0
  if (live) {
    stage_own<D, CT>(lds0 + own, base, ld, w.col0, L, lane);
    stage_own<D, CT>(lds0 + kGrad + wave * kOwnBlock, dctx + head, A, w.col0, L, lane);
    const int q = w.col0 + r;
#pragma unroll
    for (int s = 0; s < KS; ++s)
      of[0][s] = *reinterpret_cast<const u32x4_t*>(ctx + head + (size_t)(q < L ? q : L - 1) * A + 16 * s + 8 * hf);
    wait_all_copies();
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        qf[c][s] = rd.row(own, c, s);
        dof[c][s] = rd.row(kGrad + wave * kOwnBlock, c, s);
        asm volatile("" : "+a"(qf[c][s]), "+a"(dof[c][s]) :: "memory");
        asm volatile("" : "+v"(of[c][s]));
      }
  }
  wait_all_copies();
  __syncthreads();
#pragma unroll
  for (int x = 0; x < COPIES; ++x) start(0, 1, x);             // K block 1 and V block 0

  if (!live) {                                                 // a wavefront without columns only stages
    for (int kb = 0, k2 = 2; kb < nkb; ++kb) {
      wait_all_copies();
      __syncthreads();
      if (!PEEL || kb + 1 < nkb) {
#pragma unroll
        for (int x = 0; x < COPIES; ++x) start(kb + 1, k2, x);
      }
      k2 = k2 == 2 ? 0 : k2 + 1;
    }
    wait_all_copies();
    __syncthreads();
    return;
  }
  f32x16_t dq[CT][DT];
  float dd[CT], lse2[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int q = w.col0 + 32 * c + r, qc = q < L ? q : L - 1;
    dd[c] = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      float g[8], ov[8];
      Vec16<bf16_t>::unpack(uint4{dof[c][s][0], dof[c][s][1], dof[c][s][2], dof[c][s][3]}, g);
      Vec16<bf16_t>::unpack(uint4{of[c][s][0], of[c][s][1], of[c][s][2], of[c][s][3]}, ov);
#pragma unroll
      for (int i = 0; i < 8; ++i) dd[c] = fmaf(g[i], ov[i], dd[c]);
    }
    dd[c] += __shfl_xor(dd[c], 32, 64);
    if (hf == 0 && q < L) dvec[(size_t)w.bh * L + q] = dd[c];
    lse2[c] = lse[(size_t)w.bh * L + qc] * 1.4426950408889634f;
#pragma unroll
    for (int t = 0; t < DT; ++t) clear_acc(dq[c][t]);
  }
#pragma unroll
  for (int c = 0; c < CT; ++c) asm volatile("" : "+v"(lse2[c]));         // loaded here, not waited for in the loop
  f32x16_t sacc[CT];                                            // scores of 32 keys
  {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const u32x4_t f = rd.row(0, 0, s);
#pragma unroll
      for (int c = 0; c < CT; ++c) sacc[c] = MOE_MFMA(f, qf[c][s], s == 0 ? f32x16_t{} : sacc[c]);
    }
  }

  int k0 = 0;                                                  // place of K block kb
  // One block of keys; LAST: nothing follows.  (RAGGED keeps one copy of its long loop: a second one, run once, costs more
  // in fetching it than the products it leaves out.)
  auto step = [&](int kb, auto last) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last)::value;
    wait_all_copies();                                         // K block kb + 1 and V block kb are there;
    __syncthreads();                                           // K and V block kb - 1 are read, their places free
    const int k1 = k0 == 2 ? 0 : k0 + 1, k2 = k1 == 2 ? 0 : k1 + 1;
    {
      const uint32_t kst = k0 * GM::kBlock, knext = k1 * GM::kBlock, vst = kV + (kb & 1) * GM::kBlock;
      f32x16_t dpacc[CT], snext[CT];
      bf16x8_bits_t dsf[2][CT][TERMS];                          // [k step][column tile]
      // per 32 keys: KS units of dP, under them P; KS of the next 32 keys' scores (unless there are none),
      // under them dS; 2 DT of dQ
      constexpr int UNITS = 2 * KS + 2 * DT;
      auto end_mask = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kb * 64 + 32 * t + 8 * (i >> 2) + 4 * hf + (i & 3) >= L) {
#pragma unroll
            for (int c = 0; c < CT; ++c) sacc[c][i] = 0.f;
          }
      };
      run_units<0, 2 * UNITS, 4>(
          [&](auto U) __attribute__((always_inline)) { constexpr int t = decltype(U)::value / UNITS, u = decltype(U)::value % UNITS;
            return std::integral_constant<int, u < 2 * KS ? CT : CT * TERMS>{};
          },
          [&](auto U) __attribute__((always_inline)) {
            constexpr int t = decltype(U)::value / UNITS, u = decltype(U)::value % UNITS, v = u - 2 * KS;
            if constexpr (u < KS) return rd.row(vst, t, u);
            else if constexpr (u < 2 * KS) return rd.row(t == 0 ? kst : knext, 1 - t, u - KS);
            else return rd.transposed(kst, 32 * t + 16 * (v / DT), v % DT);
          },
          [&](auto U, auto P, const u32x4_t& f) __attribute__((always_inline)) {
            constexpr int t = decltype(U)::value / UNITS, u = decltype(U)::value % UNITS, v = u - 2 * KS;
            constexpr int c = decltype(P)::value % CT, k = TERMS - 1 - decltype(P)::value / CT;
            if constexpr (LAST && t == 1 && u >= KS && u < 2 * KS) return;       // (no scores to multiply ahead)
            if constexpr (u < KS) dpacc[c] = MOE_MFMA(f, dof[c][u], u == 0 ? f32x16_t{} : dpacc[c]);
            else if constexpr (u < 2 * KS) snext[c] = MOE_MFMA(f, qf[c][u - KS], u == KS ? f32x16_t{} : snext[c]);
            else {
              if constexpr (v % DT == 0 && decltype(P)::value == 0) fresh_operand();
              mfma_acc(dq[c][v % DT], f, dsf[v / DT][c][k]);
            }
          },
          [&](auto U, auto P, auto) __attribute__((always_inline)) {
            constexpr int t = decltype(U)::value / UNITS, u = decltype(U)::value % UNITS, p = decltype(P)::value;
            if constexpr (!LAST && decltype(U)::value < COPIES && p == 0) start(kb + 1, k2, decltype(U)::value);
            if constexpr (u < KS) {
              constexpr int w = CT * u + p;                    // value j: row j / CT, column tile j % CT
#pragma unroll
              for (int j = w * 16 / KS; j < (w + 1) * 16 / KS; ++j)
                sacc[j % CT][j / CT] = __builtin_amdgcn_exp2f(fmaf(sacc[j % CT][j / CT], sl2, -lse2[j % CT]));
              if (RAGGED && u == KS - 1 && p == CT - 1 && kb + 1 == nkb) end_mask(t);      // (dP of a row of zeros is 0)
            } else if constexpr (u < 2 * KS) {
              constexpr int w = CT * (u - KS) + p - 1, all = CT * KS - 1;      // (not right behind dP's last product)
              if constexpr (w >= 0) {
#pragma unroll
                for (int j = w * 16 * CT / all; j < (w + 1) * 16 * CT / all; ++j) sacc[j % CT][j / CT] = dscore(sacc[j % CT][j / CT], dpacc[j % CT][j / CT], dd[j % CT]);
              }
              if constexpr (u == KS + KS / 2 + 1) fragment_terms(sacc[p], 0, dsf[0][p]);
            } else if constexpr (u == 2 * KS && p < CT) {
              fragment_terms(sacc[p], 8, dsf[1][p]);
            }
            if constexpr (u == UNITS - 1 && p == CT * TERMS - 1) {
#pragma unroll
              for (int c = 0; c < CT; ++c) sacc[c] = snext[c];
            }
          });
    }
    k0 = k1;
  };
  for (int kb = 0; kb + (PEEL ? 1 : 0) < nkb; ++kb) step(kb, std::false_type{});
  if constexpr (PEEL) step(nkb - 1, std::true_type{});
  else wait_all_copies();
  settle_all(dq);
  __syncthreads();                                             // the other wavefronts have read the last blocks
  store_own<D, CT>(dq, scale, lds0 + own, dqkv + (size_t)w.b * L * ld + (size_t)w.h * D, ld, w.col0, L, lane);
}

// ---------------------------------------------------------------- dq (and D) of short ragged sequences
// K and V blocks through registers into one LDS stage, K once more in the order of the transposing read: more traffic
// in LDS, but a shorter way to the first product, which is what counts for a few blocks of keys, and for d 64 three
// blocks on a unit instead of two (attention_dq_short below says which calls take it).
template <int D>
__global__ __launch_bounds__(256, 2) void attention_bwd_dq_short_kernel(
    const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ ctx, const bf16_t* __restrict__ dctx,
    const float* __restrict__ lse, bf16_t* __restrict__ dqkv, float* __restrict__ dvec, int L,
    int heads) {
  using GM = ShortGeom<D>;
  constexpr int KS = D / 16, DT = D / 32;
  constexpr int TERMS = 3;                                            // bf16 terms of dS
  constexpr int kVRows = GM::kRowBlock, kKPerm = 2 * GM::kRowBlock;   // stage: K rows, V rows, K permuted
  constexpr int kStage = 2 * GM::kRowBlock + GM::kTrBlock;
  extern __shared__ __attribute__((aligned(256))) unsigned char att_lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 31, hf = lane >> 5;
  const int qblocks = (L + 127) / 128;
  const unsigned work = xcd_contiguous(blockIdx.x, gridDim.x);
  const int qb = work % qblocks;
  const long long bh = work / qblocks;
  const int h = (int)(bh % heads);
  const long long b = bh / heads;
  const int A = heads * D;
  const size_t ld = (size_t)3 * A;
  const bf16_t* base = qkv + (size_t)b * L * ld + (size_t)h * D;
  const bf16_t* kbase = base + A;
  const bf16_t* vbase = base + 2 * A;
  const int q = qb * 128 + wave * 32 + r;

  // Q^T and dO^T fragments of this wavefront's queries, D of the lane's query
  const int qc = q >= L ? L - 1 : q;
  const bool live = qb * 128 + __builtin_amdgcn_readfirstlane(wave) * 32 < L;
  const bf16_t* qrow = base + (size_t)qc * ld;
  const size_t crow = ((size_t)b * L + qc) * A + (size_t)h * D;
  u32x4_t qf[KS], dof[KS];
  float dd = 0.f;
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    qf[s] = *reinterpret_cast<const u32x4_t*>(qrow + 16 * s + 8 * hf);
    dof[s] = *reinterpret_cast<const u32x4_t*>(dctx + crow + 16 * s + 8 * hf);
    const u32x4_t of = *reinterpret_cast<const u32x4_t*>(ctx + crow + 16 * s + 8 * hf);
    float g[8], o[8];
    Vec16<bf16_t>::unpack(uint4{dof[s][0], dof[s][1], dof[s][2], dof[s][3]}, g);
    Vec16<bf16_t>::unpack(uint4{of[0], of[1], of[2], of[3]}, o);
#pragma unroll
    for (int i = 0; i < 8; ++i) dd = fmaf(g[i], o[i], dd);
  }
  dd += __shfl_xor(dd, 32, 64);
  if (hf == 0 && q < L) dvec[(size_t)bh * L + q] = dd;
  const float lse2 = lse[(size_t)bh * L + qc] * 1.4426950408889634f;
  const float scale = 1.0f / sqrtf((float)D);
  const float sl2 = 1.4426950408889634f * scale;

  f32x16_t dq[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) dq[t][i] = 0.f;

  constexpr int VV = 64 * D / 8 / 256, VPR = D / 8;
  u32x4_t kreg[VV], vreg[VV];
#define MOE_ATTB_LOAD(kb)                                                                     \
  _Pragma("unroll") for (int i = 0; i < VV; ++i) {                                            \
    const int f = tid + 256 * i, c = f % VPR;                                                 \
    int key = (kb) * 64 + f / VPR;                                                            \
    key = key < L ? key : L - 1;                                                  \
    kreg[i] = *reinterpret_cast<const u32x4_t*>(kbase + (size_t)key * ld + 8 * c);            \
    vreg[i] = *reinterpret_cast<const u32x4_t*>(vbase + (size_t)key * ld + 8 * c);            \
  }
#define MOE_ATTB_STORE(stage)                                                                 \
  _Pragma("unroll") for (int i = 0; i < VV; ++i) {                                            \
    const int f = tid + 256 * i, key = f / VPR, c = f % VPR;                                  \
    unsigned char* sb = att_lds + (stage) * kStage;                                       \
    *reinterpret_cast<u32x4_t*>(sb + key * GM::kRowPitch + 16 * c) = kreg[i];                 \
    *reinterpret_cast<u32x4_t*>(sb + kVRows + key * GM::kRowPitch + 16 * c) = vreg[i];        \
    *reinterpret_cast<u32x4_t*>(sb + kKPerm + swap_bits_2_3(key) * GM::kTrPitch + 16 * c) = kreg[i]; \
  }
  const int nkb = (L + 63) / 64;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_ptr)att_lds);
  for (int kb = 0; kb < nkb; ++kb) {
    // one LDS stage, two blocks per CU: the other block multiplies while this one stages
    MOE_ATTB_LOAD(kb)
    __syncthreads();                         // the previous key block has been read by everyone
    MOE_ATTB_STORE(0)
    __syncthreads();
    if (!live) continue;                     // (both barriers of the next block are still reached)
    const uint32_t kst = lds0, vst = kst + kVRows, kpst = kst + kKPerm;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x16_t sacc, dpacc;
#pragma unroll
      for (int i = 0; i < 16; ++i) { sacc[i] = 0.f; dpacc[i] = 0.f; }
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const uint32_t off = (32 * t + r) * GM::kRowPitch + 32 * s + 16 * hf;
        const u32x4_t kf = *(lds_u4_ptr)(uintptr_t)(kst + off);
        const u32x4_t vf = *(lds_u4_ptr)(uintptr_t)(vst + off);
        sacc = MOE_MFMA(kf, qf[s], sacc);
        dpacc = MOE_MFMA(vf, dof[s], dpacc);
      }
      float ds[16];
#pragma unroll
      for (int i = 0; i < 16; ++i)
        ds[i] = dscore(__builtin_amdgcn_exp2f(fmaf(sacc[i], sl2, -lse2)), dpacc[i], dd);
      if (kb * 64 + 64 > L) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kb * 64 + 32 * t + 8 * (i >> 2) + 4 * hf + (i & 3) >= L) ds[i] = 0.f;
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        u32x4_t dsf[3];
        split_bf16x8(ds, 8 * s, dsf);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const bf16x8_t kt = read_transposed<GM::kTrPitch>(kpst, 32 * t + 16 * s, dt, lane);
#pragma unroll
          for (int k = TERMS - 1; k >= 0; --k) dq[dt] = MOE_MFMA(kt, dsf[k], dq[dt]);
        }
      }
    }
  }
#undef MOE_ATTB_LOAD
#undef MOE_ATTB_STORE
  if (q >= L) return;
  // dq[dt][i]: d = 32 dt + 8 (i/4) + 4 hf + i%4 of query r
  bf16_t* orow = dqkv + ((size_t)b * L + q) * ld + (size_t)h * D;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const u32x2_t w = {pack_bf16x2(dq[dt][4 * q4] * scale, dq[dt][4 * q4 + 1] * scale),
                         pack_bf16x2(dq[dt][4 * q4 + 2] * scale, dq[dt][4 * q4 + 3] * scale)};
      *reinterpret_cast<u32x2_t*>(orow + 32 * dt + 8 * q4 + 4 * hf) = w;
    }
}

// ---------------------------------------------------------------- dk, dv
template <int D, int CT, bool RAGGED>
__global__ __launch_bounds__(256, 1) void attention_bwd_dkv_mfma_kernel(
    const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dctx, const float* __restrict__ lse,
    const float* __restrict__ dvec, bf16_t* __restrict__ dqkv, int L, int heads) {
  using GM = AttGeom<D>;
  constexpr int KS = D / 16, DT = D / 32, TERMS = RAGGED ? 3 : 1, kOwnBlock = 32 * CT * GM::kRow;
  constexpr int kGrad = GM::kBlock, kStats = 2 * GM::kBlock, kStage = kStats + 512;   // Q rows, dO rows, 64 lse, 64 D
  constexpr bool kValuesInLds = D == 128 && CT == 2;           // there both operands' fragments and both results are
  constexpr int kOwn = 2 * kStage;                             // 384 registers, too many beside S and dP
  extern __shared__ __attribute__((aligned(256))) unsigned char att_lds[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_ptr)att_lds);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, hf = lane >> 5;
  const AttWork<CT> w(L, heads, wave);
  const int A = heads * D;
  const size_t ld = (size_t)3 * A;
  const bf16_t* const qbase = qkv + (size_t)w.b * L * ld + (size_t)w.h * D;
  const bf16_t* const gbase = dctx + (size_t)w.b * L * A + (size_t)w.h * D;
  const float* const stat = (wave & 1 ? dvec : lse) + (size_t)w.bh * L;      // (two wavefronts copy the same 64 values)
  const bool live = w.col0 < L;

  uint32_t qoff[GM::kCopies], goff[GM::kCopies];
  copy_offsets<D>(qoff, ld, wave, lane);
  copy_offsets<D>(goff, A, wave, lane);
  const int nqb = (L + 63) / 64;
  // copy x of block j: Q rows, dO rows, 64 values of lse and D
  auto start = [&](int j, int x) __attribute__((always_inline)) {
    const uint32_t st = lds0 + (j & 1) * kStage;
    const int first = 64 * j;
    if (x < GM::kCopies) stage_copy<D, RAGGED>(st, qbase, ld, first, L, qoff, x, wave, lane);
    else if (x < 2 * GM::kCopies) stage_copy<D, RAGGED>(st + kGrad, gbase, A, first, L, goff, x - GM::kCopies, wave, lane);
    else {
      const int row = first + lane;
      const uint32_t soff = 4 * (RAGGED && row >= L ? L - 1 : row);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(st + kStats + (wave & 1) * 256),
                   "v"(soff), "s"(stat) : "memory");
    }
  };
  constexpr int COPIES = 2 * GM::kCopies + 1;

  // K and V fragments of this wavefront's keys: lane (r, hf) holds d = 16 s + 8 hf .. + 7.  K comes through the places
  // of Q and dO, V through the wavefront's own block.
  const AttReads<D> rd(lds0, lane);
  const uint32_t own = kOwn + wave * kOwnBlock;
  u32x4_t kf[CT][KS], vf[CT][kValuesInLds ? 1 : KS];
  if (live) {
    stage_own<D, CT>(lds0 + wave * kOwnBlock, qbase + A, ld, w.col0, L, lane);
    stage_own<D, CT>(lds0 + own, qbase + 2 * A, ld, w.col0, L, lane);
    wait_all_copies();
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        kf[c][s] = rd.row(wave * kOwnBlock, c, s);
        asm volatile("" : "+v"(kf[c][s]) :: "memory");
        if (!kValuesInLds) vf[c][s] = rd.row(own, c, s);
      }
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < COPIES; ++x) start(0, x);
  if (!live) {                                                 // a wavefront without columns only stages
    for (int qb = 0; qb + 1 < nqb; ++qb) {
      wait_all_copies();
      __syncthreads();
#pragma unroll
      for (int x = 0; x < COPIES; ++x) start(qb + 1, x);
    }
    wait_all_copies();
    __syncthreads();
    return;
  }
  f32x16_t dk[CT][DT], dv[CT][DT];
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int t = 0; t < DT; ++t) { clear_acc(dk[c][t]); clear_acc(dv[c][t]); }
  const float scale = 1.0f / sqrtf((float)D), sl2 = 1.4426950408889634f * scale;
  // value i of a tile belongs to query 32 t + 8 (i/4) + 4 hf + i%4: four consecutive queries per i/4
  auto stat4 = [&](uint32_t block, int t, int g) __attribute__((always_inline)) {
    return *(lds_f4_ptr)(uintptr_t)(lds0 + block + 4 * (32 * t + 8 * g + 4 * hf));
  };
  auto step = [&](int qb, auto last) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last)::value;
    wait_all_copies();                                         // block qb is there;
    __syncthreads();                                           // block qb - 1 is read, its place free
    {
      const uint32_t qst = (qb & 1) * kStage, gst = qst + kGrad, sst = qst + kStats;
      f32x16_t p[CT], ds[CT];                                    // S, then P; dP, then dS: [query][key]
      bf16x8_bits_t pt[2][CT][TERMS], dst[2][CT][TERMS];         // [k step][column tile]
      f32x4_t l4[2], d4[2];
      u32x4_t vcol[3][CT];
      // per 32 queries: KS units of S; KS of dP, under them P; 2 DT of dV, under them dS; 2 DT of dK
      constexpr int UNITS = 2 * KS + 4 * DT;
      auto end_mask = [&](f32x16_t (&v)[CT], int t, int first) __attribute__((always_inline)) {
#pragma unroll
        for (int i = first; i < first + 8; ++i)
          if (qb * 64 + 32 * t + 8 * (i >> 2) + 4 * hf + (i & 3) >= L) {
#pragma unroll
            for (int c = 0; c < CT; ++c) v[c][i] = 0.f;
          }
      };
      run_units<0, 2 * UNITS, 3>(
          [&](auto U) __attribute__((always_inline)) { return std::integral_constant<int, decltype(U)::value % UNITS < 2 * KS ? CT : CT * TERMS>{}; },
          [&](auto U) __attribute__((always_inline)) {
            constexpr int t = decltype(U)::value / UNITS, u = decltype(U)::value % UNITS, v = u - 2 * KS, x = v - 2 * DT;
            if constexpr (u < KS) return rd.row(qst, t, u);
            else if constexpr (u < 2 * KS) return rd.row(gst, t, u - KS);
            else if constexpr (v < 2 * DT) return rd.transposed(gst, 32 * t + 16 * (v / DT), v % DT);
            else return rd.transposed(qst, 32 * t + 16 * (x / DT), x % DT);
          },
          [&](auto U, auto P, const u32x4_t& f) __attribute__((always_inline)) {
            constexpr int u = decltype(U)::value % UNITS, v = u - 2 * KS, x = v - 2 * DT;
            constexpr int c = decltype(P)::value % CT, k = TERMS - 1 - decltype(P)::value / CT;
            if constexpr (kValuesInLds && u >= KS - 2 && u < 2 * KS - 2) vcol[(u - KS + 2) % 3][c] = rd.row(own, c, u - KS + 2);
            if constexpr (u < KS) p[c] = MOE_MFMA(f, kf[c][u], u == 0 ? f32x16_t{} : p[c]);
            else if constexpr (u < 2 * KS) {
              u32x4_t col;                                     // (V from LDS was fetched two units ago)
              if constexpr (kValuesInLds) col = vcol[(u - KS) % 3][c];
              else col = vf[c][u - KS];
              ds[c] = MOE_MFMA(f, col, u == KS ? f32x16_t{} : ds[c]);
            } else {
              if constexpr (v % DT == 0 && decltype(P)::value == 0) fresh_operand();
              if constexpr (x < 0) mfma_acc(dv[c][v % DT], f, pt[v / DT][c][k]);
              else mfma_acc(dk[c][x % DT], f, dst[x / DT][c][k]);
            }
          },
          [&](auto U, auto P, auto NP) __attribute__((always_inline)) {
            constexpr int t = decltype(U)::value / UNITS, u = decltype(U)::value % UNITS, v = u - 2 * KS, x = v - 2 * DT;
            constexpr int pc = decltype(P)::value, n = decltype(NP)::value;
            if constexpr (!LAST && decltype(U)::value < COPIES && pc == 0) start(qb + 1, decltype(U)::value);
            if constexpr (u == KS - 1 && pc == 0) l4[0] = stat4(sst, t, 0);
            if constexpr (u >= KS && u < 2 * KS) {             // P
              constexpr int w = CT * (u - KS) + pc, first = w * 16 / KS, to = (w + 1) * 16 / KS;      // value j: row j / CT, column tile j % CT
              if constexpr (first % (4 * CT) == 0 && first + 4 * CT < 16 * CT) l4[(first / (4 * CT) + 1) % 2] = stat4(sst, t, first / (4 * CT) + 1);
#pragma unroll
              for (int j = first; j < to; ++j)
                p[j % CT][j / CT] = __builtin_amdgcn_exp2f(fmaf(p[j % CT][j / CT], sl2, -(l4[j / (4 * CT) % 2][j / CT % 4] * 1.4426950408889634f)));
              if constexpr (RAGGED && LAST && to % (8 * CT) == 0) end_mask(p, t, to / CT - 8);
              if constexpr (u == KS + KS / 2 + 1) fragment_terms(p[pc], 0, pt[0][pc]);
              if constexpr (u == 2 * KS - 1 && pc == 0) d4[0] = stat4(sst + 256, t, 0);
            }
            if constexpr (v == 0 && pc < CT) fragment_terms(p[pc], 8, pt[1][pc]);
            if constexpr (v >= 0 && x < 0) {                   // dS
              constexpr int w = n * v + pc, all = 2 * DT * n, first = w * 16 * CT / all, to = (w + 1) * 16 * CT / all;
              if constexpr (first % (4 * CT) == 0 && first != to && first + 4 * CT < 16 * CT) d4[(first / (4 * CT) + 1) % 2] = stat4(sst + 256, t, first / (4 * CT) + 1);
#pragma unroll
              for (int j = first; j < to; ++j) ds[j % CT][j / CT] = p[j % CT][j / CT] * (ds[j % CT][j / CT] - d4[j / (4 * CT) % 2][j / CT % 4]);
              if constexpr (RAGGED && LAST && first != to && to % (8 * CT) == 0) end_mask(ds, t, to / CT - 8);
              if constexpr (v == DT + 1 && pc < CT) fragment_terms(ds[pc], 0, dst[0][pc]);
            }
            if constexpr (x == 0 && pc < CT) fragment_terms(ds[pc], 8, dst[1][pc]);
          });
    }
  };
  for (int qb = 0; qb + 1 < nqb; ++qb) step(qb, std::false_type{});
  step(nqb - 1, std::true_type{});
  settle_all(dk);
  settle_all(dv);
  bf16_t* const out = dqkv + (size_t)w.b * L * ld + A + (size_t)w.h * D;
  store_own<D, CT>(dk, scale, lds0 + own, out, ld, w.col0, L, lane);
  store_own<D, CT>(dv, 1.f, lds0 + own, out + A, ld, w.col0, L, lane);
}

}  // namespace

// dk, dv of d 128, L % 128 == 0: two tiles of 32 keys per wavefront.  One block shares a compute unit with no other, and 256 keys of
// a block take 1.46 times as long as 128 (L 1024, 192 blocks of 128 35.4 us, 96 of 256 51.7; with the three terms of ragged
// lengths 1.75 times, and never worth it).
bool attention_dkv_wide(long long sequence_heads, int L, int cus) {
  const long long rounds = (sequence_heads * (L / 128) + cus - 1) / cus, rounds2 = (sequence_heads * ((L + 255) / 256) + cus - 1) / cus;
  return 1.46 * (double)rounds2 < (double)rounds;
}

// Which dq kernel a ragged length takes, from 680 calls of both (us, short kernel / the other; sequence-heads of L tokens).
// Under 256 tokens the short one: d 128, 64 of 48 7.8 / 9.9, 400 of 100 21.5 / 21.9; d 64, 64 of 48 6.0 / 6.7, 1000 of 100
// 25.5 / 26.2, 32 of 193 11.6 / 12.7 (three blocks of keys of d 64 are as often faster with either: 96 of 191 11.0 / 12.1, 96 of
// 192 11.8 / 10.9).  For d 128 and more than two blocks of keys only while units have one block each: 96 of 191 15.6 / 16.0, 200 of 200
// 29.5 / 29.0, 152 of 200 28.2 / 27.1; then 132 of 300 34.4 / 32.4, 128 of 700 95 / 90.  For d 64 three short blocks share a
// unit, or two of the others: past one round of those the short kernel has fewer rounds or, up to 896 tokens, shorter ones: 88 of 700
// 46.8 / 52.1, 248 of 700 88.8 / 91.6, 80 of 900 58 / 62, 80 of 1000 64 / 69, but with as many rounds 112 of 1000 88.9 / 86.9.
bool attention_dq_short(int d, int L, long long blocks, int cus) {
  if (d == 128) return L <= 128 || (L < 256 && blocks <= cus);
  auto rounds = [&](long long per_unit) { return (blocks + per_unit * cus - 1) / (per_unit * cus); };
  return L < 256 || (rounds(2) > 1 && (L <= 896 || rounds(3) < rounds(2)));
}

namespace {

template <int D> constexpr int kLdsForward = 4 * AttGeom<D>::kBlock;
template <int D> constexpr int kLdsQ = 5 * AttGeom<D>::kBlock;
template <int D> constexpr int kLdsQShort = 2 * ShortGeom<D>::kRowBlock + ShortGeom<D>::kTrBlock;
template <int D, int CT> constexpr int kLdsKV = 2 * (2 * AttGeom<D>::kBlock + 512) + 128 * CT * AttGeom<D>::kRow;

template <int D, bool RAGGED>
int prepare_kernels() {
  static LdsLimitOnce once, once_q, once_short, once_kv1, once_kv2;
  int rc = ensure_lds_limit(once, reinterpret_cast<const void*>(attention_mfma_kernel<D, RAGGED>), kLdsForward<D>);
  if (rc == MOE_OK) rc = ensure_lds_limit(once_q, reinterpret_cast<const void*>(attention_bwd_dq_mfma_kernel<D, RAGGED>), kLdsQ<D>);
  if constexpr (RAGGED)
    if (rc == MOE_OK) rc = ensure_lds_limit(once_short, reinterpret_cast<const void*>(attention_bwd_dq_short_kernel<D>), kLdsQShort<D>);
  if (rc == MOE_OK) rc = ensure_lds_limit(once_kv1, reinterpret_cast<const void*>(attention_bwd_dkv_mfma_kernel<D, 1, RAGGED>), (kLdsKV<D, 1>));
  if constexpr (D == 128 && !RAGGED)
    if (rc == MOE_OK) rc = ensure_lds_limit(once_kv2, reinterpret_cast<const void*>(attention_bwd_dkv_mfma_kernel<D, 2, RAGGED>), (kLdsKV<D, 2>));
  return rc;
}

template <int D, bool RAGGED>
int launch(const bf16_t* qkv, bf16_t* ctx, float* lse, long long B, int L, int heads, hipStream_t st) {
  if (prepare_kernels<D, RAGGED>() != MOE_OK) return MOE_EHIP;
  const long long blocks = B * heads * ((L + 127) / 128);
  if (blocks > 0x7fffffffLL) return MOE_EUNSUPPORTED;
  if constexpr (RAGGED)
    if (L <= (D == 64 ? 64 : 48)) {                            // (figures at the kernel)
      hipLaunchKernelGGL((attention_short_kernel<D>), dim3((unsigned)blocks), dim3(256), 0, st, qkv, ctx, lse, L, heads);
      return check_launch();
    }
  hipLaunchKernelGGL((attention_mfma_kernel<D, RAGGED>), dim3((unsigned)blocks), dim3(256), kLdsForward<D>, st, qkv, ctx, lse, L, heads);
  return check_launch();
}
template <int D, bool RAGGED>
int launch_bwd(const bf16_t* qkv, const bf16_t* ctx, const bf16_t* dctx, const float* lse, bf16_t* dqkv, float* dvec,
               long long B, int L, int heads, hipStream_t st) {
  int cus = 0;
  if (prepare_kernels<D, RAGGED>() != MOE_OK || compute_units(&cus) != MOE_OK) return MOE_EHIP;
  const long long blocks = B * heads * ((L + 127) / 128), blocks2 = B * heads * ((L + 255) / 256);
  if (blocks > 0x7fffffffLL) return MOE_EUNSUPPORTED;
  const bool dq_short = RAGGED && attention_dq_short(D, L, blocks, cus);
  if constexpr (RAGGED) {
    if (dq_short) hipLaunchKernelGGL((attention_bwd_dq_short_kernel<D>), dim3((unsigned)blocks), dim3(256), kLdsQShort<D>, st, qkv, ctx,
                                     dctx, lse, dqkv, dvec, L, heads);
  }
  if (!dq_short)
    hipLaunchKernelGGL((attention_bwd_dq_mfma_kernel<D, RAGGED>), dim3((unsigned)blocks), dim3(256), kLdsQ<D>, st, qkv, ctx, dctx,
                     lse, dqkv, dvec, L, heads);
  if constexpr (D == 128 && !RAGGED)
    if (attention_dkv_wide(B * heads, L, cus)) {
      hipLaunchKernelGGL((attention_bwd_dkv_mfma_kernel<D, 2, RAGGED>), dim3((unsigned)blocks2), dim3(256), (kLdsKV<D, 2>), st, qkv,
                         dctx, lse, dvec, dqkv, L, heads);
      return check_launch();
    }
  hipLaunchKernelGGL((attention_bwd_dkv_mfma_kernel<D, 1, RAGGED>), dim3((unsigned)blocks), dim3(256), (kLdsKV<D, 1>), st, qkv,
                     dctx, lse, dvec, dqkv, L, heads);
  return check_launch();
}

}  // namespace

int prepare_attention_mfma() {
  const int rcs[] = {prepare_kernels<64, false>(), prepare_kernels<64, true>(), prepare_kernels<128, false>(), prepare_kernels<128, true>()};
  for (int rc : rcs)
    if (rc != MOE_OK) return rc;
  return MOE_OK;
}

// Copies address the rows of a block by unsigned 32-bit byte offsets, and the row statistics of a head by signed ones.  The
// widths that the calls accept (heads . d below 2^23) stay below the first.
bool attention_mfma_ok(int act_dtype, int L, int heads, int d) {
  return act_dtype == MOE_BF16 && (d == 64 || d == 128) && (long long)64 * 3 * heads * d * 2 < 1LL << 32 && L < 1 << 29;
}

int launch_attention_mfma(const void* qkv, void* ctx, float* lse, long long B, int L, int heads, int d, hipStream_t st) {
  auto q = static_cast<const bf16_t*>(qkv);
  auto c = static_cast<bf16_t*>(ctx);
  if (L % 128 != 0) return d == 64 ? launch<64, true>(q, c, lse, B, L, heads, st) : launch<128, true>(q, c, lse, B, L, heads, st);
  return d == 64 ? launch<64, false>(q, c, lse, B, L, heads, st) : launch<128, false>(q, c, lse, B, L, heads, st);
}

int launch_attention_bwd_mfma(const void* qkv, const void* ctx, const void* dctx, const float* lse, void* dqkv, float* dvec,
                              long long B, int L, int heads, int d, hipStream_t st) {
  auto q = static_cast<const bf16_t*>(qkv);
  auto c = static_cast<const bf16_t*>(ctx);
  auto g = static_cast<const bf16_t*>(dctx);
  auto o = static_cast<bf16_t*>(dqkv);
  if (L % 128 != 0)
    return d == 64 ? launch_bwd<64, true>(q, c, g, lse, o, dvec, B, L, heads, st)
                   : launch_bwd<128, true>(q, c, g, lse, o, dvec, B, L, heads, st);
  return d == 64 ? launch_bwd<64, false>(q, c, g, lse, o, dvec, B, L, heads, st)
                 : launch_bwd<128, false>(q, c, g, lse, o, dvec, B, L, heads, st);
}

}  // namespace moe
