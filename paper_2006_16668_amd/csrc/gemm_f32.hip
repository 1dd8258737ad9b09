// fp32 expert GEMMs on the matrix cores.  The paper trained its experts in fp32 (Section 4, "Model
// Details"); bf16 is this library's fast path, this kernel is the fp32 one for all six expert GEMMs of
// the forward and backward pass and the dense layers around them.
//
// The bf16 pipes multiply sixteen times as fast as the fp32 ones, so every operand enters as the three
// bf16 terms that hold its 24 bits (a = hi + mid + lo, each what is left rounded to nearest) and a product of two
// numbers as six products of terms (hi hi, hi mid, mid hi, mid mid, hi lo, lo hi), exact in fp32 and summed in
// fp32.  What is left out (mid lo, lo mid, lo lo) is at most 2^-24 of a product, as much as one fp32 rounding of it,
// 2^-27 in the mean, and of either sign; terms cut off instead of rounded left out up to 2^-21, always with the
// product's sign.  A sum of one step (16 k), which the fp32 instruction rounds seldom too, takes mid lo and lo mid
// as well: one product's error 2.65e-8 -> 2.59e-8, a single rounding.
// The five smaller products have sums of their own, so the sum that carries the result is rounded twice per 16 k
// where v_mfma_f32_32x32x2_f32 rounds it 16 times; all six in one sum were worse than that instruction where the
// operand is half zeros.  Error against float64, relative (2-norm), v_mfma_f32 / this kernel, normal operands:
// K 4 4.1e-8 / 2.7e-8, K 16 7.3e-8 / 3.2e-8, K 64 1.4e-7 / 5.1e-8, K 1024 5.7e-7 / 1.9e-7, K 3424 with a ReLU'd
// operand 7.4e-7 / 2.9e-7; all operands 1.2345678, K 1024 6.6e-6 / 2.2e-8.
// Operands are scaled by 2^24, results by 2^-48: the smallest fp32 number's terms are normal bf16 numbers then, and
// products keep all their bits (error with operands of 2^-124: 1e-3 and 3e-2 without, 8e-8 with; a multiplication per
// element fetched, 2 % of the time of large shapes).
// Terms of an operand that is not finite make NaN where the fp32 product may be an infinity, and sums past 2^80 or
// operands past 2^104 overflow by the scale, so a wavefront whose result holds anything but finite numbers multiplies
// its tiles again with v_mfma_f32_32x32x2_f32, operands straight from memory.  16 experts of 512 rows, M 1024, H 2048, us,
// all finite / every row NaN / an infinity in every 64th row: 350 / 620 / 997 (with two k at a time and nothing in
// flight 348 / 1740 / 3230; the fp32 instruction from LDS stages 535).
//
// One block of four wavefronts (2 x 2) per tile, or KG groups of four that take the steps of 16 k in turn and
// meet at the end.  A thread fetches its pieces of a step PD steps ahead into registers, from an address of
// its own: a row, column or k past an edge, or an unoccupied packed row, reads a zero line.  Their terms go
// to one of two LDS buffers, once for all wavefronts (split by every wavefront that reads an element,
// straight from fp32 stages, the same products took 8 % longer).  Unit strides run along dimensions that
// are multiples of 4 elements.
//
// Bound: six matrix instructions of 32 cycles per product of two fragments; per 128 x 128 tile and step 768
// matrix cycles, about 560 of LDS and 450 of vector instructions on each SIMD, which overlap in part.
// Large shapes run at 195 to 205 TFLOP/s (the fp32 instruction: 130, peak 157); few tiles are bound by
// a step's chain of barrier, reads, products, split and writes, about 900 cycles, hence the groups.  Both expert
// products, start of this design (fp32 instruction) / now, us, two sets of operands in turn:
//   E 2  R 8192 M 1024 H 4096  2100 / 1326    E 16 R 512 M 1024 H 2048  535 / 350
//   E 66 R 12   M 848  H 3424   470 /  328    E 24 R 295 M 768  H 3072  664 / 437
//   E 19 R 24   M 608  H 2504    96 /   71    E 16 R 128 M 512  H 1024   50 /  39
#include "common.h"

namespace moe {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

static __device__ const f32x4_t f32_zero_line = {0.f, 0.f, 0.f, 0.f};

constexpr int kBK = 16;
constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;               // of an operand, of a sum

// LDS of a block: two buffers of the three bf16 planes of a step's operands.
//   K-contiguous operand: plane [2 halves of 8 k][rows][16 bytes], the halves 128 bytes apart beyond their
//     size (a half-wavefront's 8-byte writes then meet every bank once); a fragment is one 16-byte read
//   row-of-k operand: plane [16 k][rows], 16-byte chunk c of row k at c ^ swizzle(k), read transposing
template <int T, bool KC>
struct F32Plane {
  static constexpr int kRows = 64 * T, kHalf = kRows * 16 + 128;
  static constexpr int kBytes = KC ? 2 * kHalf : 16 * kRows * 2;
  static __device__ __forceinline__ int swizzle(int k) { return T == 1 ? 4 * ((k >> 1) & 1) : 4 * (k & 3); }
  // where 4 consecutive k (KC) or rows of operand row `row` at `k` go
  static __device__ __forceinline__ uint32_t offset(int row, int k) {
    return KC ? (k >> 3) * kHalf + row * 16 + 2 * (k & 7)
              : k * (kRows * 2) + (((row >> 3) ^ swizzle(k)) * 16) + 2 * (row & 7);
  }
};

template <int TM, int TN, int KG, bool A_KC, bool B_KC>
struct F32Smem {
  static constexpr int kBOff = 3 * F32Plane<TM, A_KC>::kBytes, kBuf = kBOff + 3 * F32Plane<TN, B_KC>::kBytes;
  static constexpr int kBytes = KG * 2 * kBuf;
  static_assert((KG - 1) * TM * TN * 64 * 64 * 4 <= kBytes, "the groups' sums meet in the planes' place");
};

// TM x TN tiles of 32 x 32 per wavefront, PD steps of 16 k on their way in registers; KG groups of four
// wavefronts share a tile, group g taking steps g, g + KG, ...  The other parameters are those of GemmArgs
// and of the bf16 kernel: EPI 0 plain, 1 relu, 2 zero where mask[e,r,n] <= 0; gathered rows of A, kept rows
// of an expert (or, K_KEPT, the length of its sum).
template <int TM, int TN, int PD, int KG, int EPI, bool A_KC, bool B_KC, bool K_KEPT>
__global__ __launch_bounds__(256 * KG, TM * TN >= 4 ? 2 : TM * TN >= 2 ? 3 : 4) void gemm_f32_mfma_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ Cout,
    const float* __restrict__ mask, int R, int N, int K, int tiles_r, int tiles_n,
    const int32_t* __restrict__ gather, const int32_t* __restrict__ kept) {
  using PA = F32Plane<TM, A_KC>;
  using PB = F32Plane<TN, B_KC>;
  static_assert(PD % 2 == 0, "a buffer per parity of the step");
  using SM = F32Smem<TM, TN, KG, A_KC, B_KC>;
  constexpr int BM = 64 * TM, BN = 64 * TN, kBOff = SM::kBOff, kBuf = SM::kBuf;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef unsigned char __attribute__((address_space(3))) * lds_ptr;
  const int tid = threadIdx.x & 255, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const uint32_t smem0 = (uint32_t)(uintptr_t)((lds_ptr)smem), lds0 = smem0 + group * 2 * kBuf;
  // Consecutive workgroups go to different XCDs (8, each with its own L2).  Give every XCD a
  // contiguous range of tiles, in bands of 8 row tiles with the row tile fastest, so that the tiles
  // that share panels run next to each other under one L2.
  unsigned blk = blockIdx.x;
  const unsigned per_xcd = gridDim.x / 8;
  if (blk < per_xcd * 8) blk = (blk % 8) * per_xcd + blk / 8;
  const int per_e = tiles_r * tiles_n;
  const int e = (int)(blk / per_e), t = (int)(blk - (unsigned)e * per_e);
  const int band = t / (8 * tiles_n), rem = t - band * 8 * tiles_n;
  const int left = tiles_r - 8 * band, brows = left < 8 ? left : 8;
  const int ct = rem / brows, rt = 8 * band + (rem - ct * brows);
  const int r0 = rt * BM, n0 = ct * BN;
  const int rows = kept != nullptr && !K_KEPT ? kept[e] : R;
  if (r0 >= rows) return;                                      // block-uniform
  const int KE = K_KEPT ? kept[e] : K;
  const int KT = (KE + KG * kBK - 1) / (KG * kBK);             // steps of a group
  const int wm0 = (wave >> 1) * 32 * TM, wn0 = (wave & 1) * 32 * TN;
  const int l32 = lane & 31, hf = lane >> 5;

  // The 16-byte pieces a thread fetches of a step: 4 k of a row (K-contiguous) or 4 rows of a k
  // (row-of-k); where they come from, how far that moves per step (0 on the zero line), where their
  // terms go
  const uint64_t zline = (uint64_t)(uintptr_t)&f32_zero_line;
  uint64_t a_addr[TM], b_addr[TN];
  uint32_t a_inc[TM], b_inc[TN], a_put[TM], b_put[TN];
  auto piece_row = [&](bool kc, int q, int T) { return kc ? 64 * q + (tid >> 2) : 4 * ((tid + 256 * q) % (16 * T)); };
  auto piece_k = [&](bool kc, int q, int T) { return kc ? 4 * (tid & 3) : (tid + 256 * q) / (16 * T); };
  const int kg = group * kBK;                                  // the group's first k
#pragma unroll
  for (int q = 0; q < TM; ++q) {
    const int row = piece_row(A_KC, q, TM), k = piece_k(A_KC, q, TM);
    bool ok;
    const float* src;
    if (A_KC) {
      ok = r0 + row < rows && kg + k < KE;
      long long arow = (long long)e * R + r0 + row;
      if (gather != nullptr) {
        const int tok = ok ? gather[arow] : -1;
        ok = tok >= 0;
        arow = tok;
      }
      src = A + arow * K + kg + k;
    } else {
      ok = r0 + row < R && kg + k < KE;
      src = A + ((size_t)e * K + kg + k) * R + r0 + row;
    }
    a_addr[q] = ok ? (uint64_t)(uintptr_t)src : zline;
    a_inc[q] = ok ? (A_KC ? 1u : (uint32_t)R) * (KG * kBK * 4) : 0u;
    a_put[q] = PA::offset(row, k);
  }
#pragma unroll
  for (int q = 0; q < TN; ++q) {
    const int row = piece_row(B_KC, q, TN), k = piece_k(B_KC, q, TN);
    const bool ok = n0 + row < N && kg + k < KE;
    const float* src = B_KC ? B + ((size_t)e * N + n0 + row) * K + kg + k : B + ((size_t)e * K + kg + k) * N + n0 + row;
    b_addr[q] = ok ? (uint64_t)(uintptr_t)src : zline;
    b_inc[q] = ok ? (B_KC ? 1u : (uint32_t)N) * (KG * kBK * 4) : 0u;
    b_put[q] = kBOff + PB::offset(row, k);
  }
  f32x4_t raw[PD][TM + TN];
  auto fetch = [&](int p, f32x4_t (&r)[TM + TN]) __attribute__((always_inline)) {      // step p, the next in order
    if (p > 0) {
#pragma unroll
      for (int q = 0; q < TM; ++q) a_addr[q] += a_inc[q];
#pragma unroll
      for (int q = 0; q < TN; ++q) b_addr[q] += b_inc[q];
      const int kl = KE - p * (KG * kBK) - kg;                             // k left, this step's included
      if (kl < kBK) {                                          // block-uniform, from the last step on
#pragma unroll
        for (int q = 0; q < TM; ++q)
          if (piece_k(A_KC, q, TM) >= kl) a_addr[q] = zline;
#pragma unroll
        for (int q = 0; q < TN; ++q)
          if (piece_k(B_KC, q, TN) >= kl) b_addr[q] = zline;
      }
    }
    typedef const f32x4_t __attribute__((address_space(1))) * glb_f4_ptr;
#pragma unroll
    for (int q = 0; q < TM; ++q) r[q] = *(glb_f4_ptr)(uintptr_t)a_addr[q];
#pragma unroll
    for (int q = 0; q < TN; ++q) r[TM + q] = *(glb_f4_ptr)(uintptr_t)b_addr[q];
  };
  // the terms of the fetched pieces into the planes of a buffer
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  typedef u32x2_t __attribute__((address_space(3))) * lds_u2_ptr;
  auto put = [&](const f32x4_t& v, uint32_t at, int plane_bytes) __attribute__((always_inline)) {
    float x[4] = {v[0] * kUp, v[1] * kUp, v[2] * kUp, v[3] * kUp};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      u32x2_t w;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        w[i] = pack_bf16x2(x[2 * i], x[2 * i + 1]);
        if (k == 2) continue;                                  // (nothing is left)
        x[2 * i] -= __uint_as_float(w[i] << 16);
        x[2 * i + 1] -= __uint_as_float(w[i] & 0xffff0000u);
      }
      *(lds_u2_ptr)(uintptr_t)(at + k * plane_bytes) = w;
    }
  };
  auto split = [&](const f32x4_t (&r)[TM + TN], int buf) __attribute__((always_inline)) {
    const uint32_t base = lds0 + buf * kBuf;
#pragma unroll
    for (int q = 0; q < TM; ++q) put(r[q], base + a_put[q], PA::kBytes);
#pragma unroll
    for (int q = 0; q < TN; ++q) put(r[TM + q], base + b_put[q], PB::kBytes);
  };

  // fragment reads: 8 k (8 hf ..) of row l32 of 32-row tile i
  typedef short s16x4_t __attribute__((ext_vector_type(4)));
  typedef s16x4_t __attribute__((address_space(3))) * lds_s16x4_ptr;
  typedef bf16x8_t __attribute__((address_space(3))) * lds_bf16x8_ptr;
  const int p16 = lane & 15, bb = lane >> 4, bk = 8 * (bb >> 1) + (p16 >> 2);
  uint32_t a_rd[TM], b_rd[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
    a_rd[i] = A_KC ? PA::offset(wm0 + 32 * i + l32, 8 * hf)
                   : PA::offset(wm0 + 32 * i + 16 * (bb & 1) + 4 * (p16 & 3), bk);
#pragma unroll
  for (int j = 0; j < TN; ++j)
    b_rd[j] = kBOff + (B_KC ? PB::offset(wn0 + 32 * j + l32, 8 * hf)
                            : PB::offset(wn0 + 32 * j + 16 * (bb & 1) + 4 * (p16 & 3), bk));
  auto read_frag = [&](bool kc, uint32_t at, int pitch) __attribute__((always_inline)) {
    if (kc) return *(lds_bf16x8_ptr)(uintptr_t)at;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)at);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(at + 4 * pitch));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  // main: the products of the leading terms; rest: all others
  f32x16_t main[TM][TN], rest[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) main[i][j][v] = rest[i][j][v] = 0.f;

#pragma unroll
  for (int u = 0; u < PD; ++u)
    fetch(u, raw[u]);
  split(raw[0], 0);
  __syncthreads();
  // step s, whose pieces were in raw[u]
  auto step = [&](int s, int u) __attribute__((always_inline)) {
    // unconditional (past the end: zeros, never multiplied): a wait for the older fetches would
    // otherwise have to be one for all.  What raw[u] held went to the planes a step ago.
    fetch(s + PD, raw[u]);
    __builtin_amdgcn_sched_barrier(0);                         // (the compiler sinks them behind the split)
    const uint32_t sb = lds0 + (u & 1) * kBuf;
    bf16x8_t a[TM][3];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k) a[i][k] = read_frag(A_KC, sb + a_rd[i] + k * PA::kBytes, BM * 2);
    // terms of A and B in a product, smallest first
    constexpr int ta[6] = {2, 0, 1, 1, 0, 0}, tb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      bf16x8_t b[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) b[k] = read_frag(B_KC, sb + b_rd[j] + k * PB::kBytes, BN * 2);
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          f32x16_t& c = q == 5 ? main[i][j] : rest[i][j];
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][ta[q]], b[tb[q]], c, 0, 0, 0);
        }
    }
    // the next step's planes: last read in step s - 1, before the previous barrier
    split(raw[(u + 1) % PD], (u + 1) & 1);
    __syncthreads();
  };
  int s = 0;
  for (; s + PD <= KT; s += PD) {
#pragma unroll
    for (int u = 0; u < PD; ++u) step(s + u, u);
  }
#pragma unroll
  for (int u = 0; u < PD - 1; ++u)
    if (s + u < KT) step(s + u, u);
  // a short sum: mid lo and lo mid too, from the planes of its only step
  if (KE <= KG * kBK) {                                        // block-uniform
    bf16x8_t a[TM][2];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int k = 0; k < 2; ++k) a[i][k] = read_frag(A_KC, lds0 + a_rd[i] + (k + 1) * PA::kBytes, BM * 2);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      bf16x8_t b[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) b[k] = read_frag(B_KC, lds0 + b_rd[j] + (k + 1) * PB::kBytes, BN * 2);
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < TM; ++i)
          rest[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][q], b[1 - q], rest[i][j], 0, 0, 0);
    }
    if (KG > 1) __syncthreads();                               // the groups' sums will overwrite the planes
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) main[i][j][v] += rest[i][j][v];
  if (KG > 1) {                                                // the groups' sums, in order
    float* const sums = reinterpret_cast<float*>(smem) + wave * (TM * TN * 1024) + lane;
    if (group > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            sums[(group - 1) * (TM * TN * 4096) + ((i * TN + j) * 16 + v) * 64] = main[i][j][v];
    }
    __syncthreads();
    if (group > 0) return;
#pragma unroll
    for (int g = 0; g < KG - 1; ++g)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) main[i][j][v] += sums[g * (TM * TN * 4096) + ((i * TN + j) * 16 + v) * 64];
  }

  // c[v] of the wavefront's 32 x 32 tile (i, j): row 32 i + 8 (v/4) + 4 hf + v%4, column 32 j + lane%32: a
  // store covers whole 128-byte pieces of two rows
  auto store_tile = [&](int i, int j, const f32x16_t& c, const f32x16_t& m) {
    const int n = n0 + wn0 + 32 * j + l32, rb = r0 + wm0 + 32 * i + 4 * hf;
    if (n >= N) return;
    const size_t o = ((size_t)e * R + rb) * N + n;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int dr = 8 * (v >> 2) + (v & 3);
      float x = c[v];
      if (EPI == 1) x = fmaxf(x, 0.f);
      if (EPI == 2) x = m[v] > 0.f ? x : 0.f;
      if (rb + dr < rows) Cout[o + (size_t)dr * N] = x;
    }
  };

  // Its mask, past an edge the last row or column.  All tiles' are asked for at once, without branches, as the sums
  // are over: a block waits for memory once instead of once per tile (128 x 128 tiles, training step of 4096 tokens,
  // M 1024, H 2048, 16 experts 1125 -> 1090 us).
  auto load_mask = [&](int i, int j) {
    f32x16_t m;
    if (EPI == 2) {
      const int n = n0 + wn0 + 32 * j + l32, rb = r0 + wm0 + 32 * i + 4 * hf;
      const float* const mc = mask + (size_t)e * R * N + (n < N ? n : N - 1);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = rb + 8 * (v >> 2) + (v & 3);
        m[v] = mc[(size_t)(row < rows ? row : rows - 1) * N];
      }
    }
    return m;
  };
  f32x16_t masks[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) masks[i][j] = load_mask(i, j);

  // The wavefront's tiles with v_mfma_f32_32x32x2_f32, operands straight from memory, eight k ahead: lane half
  // hf takes k = 4 hf + q of eight in step q.
  auto fp32_products = [&](f32x16_t (&c)[TM][TN]) __attribute__((always_inline)) {
    uint64_t ap[TM], bp[TN];                                   // where a lane's k starts, 0: a row or column past an edge
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = r0 + wm0 + 32 * i + l32;
      bool ok = row < (A_KC ? rows : R);
      long long arow = (long long)e * R + row;
      if (A_KC && gather != nullptr) {
        arow = ok ? gather[arow] : -1;
        ok = arow >= 0;
      }
      const float* src = A_KC ? A + arow * K + 4 * hf : A + ((size_t)e * K + 4 * hf) * R + row;
      ap[i] = ok ? (uint64_t)(uintptr_t)src : 0;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + wn0 + 32 * j + l32;
      const float* src = B_KC ? B + ((size_t)e * N + col) * K + 4 * hf : B + ((size_t)e * K + 4 * hf) * N + col;
      bp[j] = col < N ? (uint64_t)(uintptr_t)src : 0;
    }
    auto load = [&](bool kc, uint64_t p, int k0, int ld) __attribute__((always_inline)) {
      const int k = k0 + 4 * hf;
      if (kc) return *reinterpret_cast<const f32x4_t*>((uintptr_t)(p != 0 && k < KE ? p + (uint64_t)k0 * 4 : zline));
      f32x4_t v;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        v[q] = *reinterpret_cast<const float*>((uintptr_t)(p != 0 && k + q < KE ? p + (uint64_t)(k0 + q) * ld * 4 : zline));
      return v;
    };
    f32x4_t x[2][TM], y[2][TN];
    auto fetch8 = [&](int k0, int u) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i) x[u][i] = load(A_KC, ap[i], k0, R);
#pragma unroll
      for (int j = 0; j < TN; ++j) y[u][j] = load(B_KC, bp[j], k0, N);
    };
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) c[i][j][v] = 0.f;
    fetch8(0, 0);
#pragma unroll 1
    for (int k0 = 0; k0 < KE; k0 += 16) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        fetch8(k0 + 8 * (u + 1), 1 - u);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              c[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[u][i][q], y[u][j][q], c[i][j], 0, 0, 0);
      }
    }
  };

  // anything but finite numbers (0 x number is 0 else): this wavefront's tiles again, in fp32 products
  float zero = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        zero = fmaf(main[i][j][v], 0.f, zero);
        main[i][j][v] *= kDown;
      }
  if (__builtin_amdgcn_ballot_w64(!(zero == 0.f)) != 0) fp32_products(main);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) store_tile(i, j, main[i][j], masks[i][j]);
}

template <int TM, int TN, int PD, int KG, int EPI, bool A_KC, bool B_KC, bool K_KEPT>
int prepare_tiles() {
  static LdsLimitOnce once;
  return ensure_lds_limit(
      once, reinterpret_cast<const void*>(gemm_f32_mfma_kernel<TM, TN, PD, KG, EPI, A_KC, B_KC, K_KEPT>),
      F32Smem<TM, TN, KG, A_KC, B_KC>::kBytes);
}

template <int TM, int TN, int PD, int KG, int EPI, bool A_KC, bool B_KC, bool K_KEPT>
int launch_tiles(const GemmArgs& a, int E, int R, int N, int K, hipStream_t st) {
  if (prepare_tiles<TM, TN, PD, KG, EPI, A_KC, B_KC, K_KEPT>() != MOE_OK) return MOE_EHIP;
  constexpr size_t kLds = F32Smem<TM, TN, KG, A_KC, B_KC>::kBytes;
  const int tiles_r = (R + 64 * TM - 1) / (64 * TM), tiles_n = (N + 64 * TN - 1) / (64 * TN);
  const long long nblk = (long long)E * tiles_r * tiles_n;
  if (nblk > 0x7fffffffLL) return MOE_EUNSUPPORTED;
  hipLaunchKernelGGL((gemm_f32_mfma_kernel<TM, TN, PD, KG, EPI, A_KC, B_KC, K_KEPT>), dim3((unsigned)nblk),
                     dim3(256 * KG), kLds, st, static_cast<const float*>(a.A), static_cast<const float*>(a.B),
                     static_cast<float*>(a.C), static_cast<const float*>(a.mask), R, N, K, tiles_r,
                     tiles_n, a.gather, a.kept);
  return check_launch();
}

// Tile and groups: the shape's time on the fullest compute unit.  The tables hold what 16 k of n tiles that
// share a unit take, in ns, n up to what fits a unit (mean of shapes whose blocks share operands and shapes
// that stream weights, K 1024); a tile's ends take about 2.5 us more.  A lone tile's step is a chain that no
// form shortens much, so more groups help until the tiles fill the units.
//   us, tiles 64 x 64 with 1 / 2 / 4 groups, 64 x 128, 128 x 128 (both expert products):
//   E 3  R 64  M 1024 H 4096  112 / 89 / 77 / 136 / 206    E 16 R 128 M 512 H 1024    47 / 44 / 45 / 51 / 73
//   E 66 R 12  M 848  H 3424  393 / 403 / 438 / 341 / 523  E 40 R 100 M 600 H 1500  169 / 184 / 224 / 148 / 142
//   E 16 R 512 M 1024 H 2048  543 / 567 / 628 / 469 / 426  E 2  R 300 M 512 H 2048    67 / 56 / 56 / 75 / 109
enum F32Form { k64x64, k64x64x2, k64x64x4, k64x128, k128x128 };
F32Form f32_form(int E, int R, int N, int K, int cus) {
  static const double t64[] = {425, 635, 915, 1230}, t64x2[] = {375, 615}, t64x4[] = {345}, t64x128[] = {590, 990, 1550},
                      t128[] = {890, 1700};
  F32Form form = k64x64;
  double best = 0;
  auto consider = [&](F32Form f, int bm, int bn, int groups, int res, const double* t) {
    const long long n = (long long)E * ((R + bm - 1) / bm) * ((N + bn - 1) / bn), full = n / ((long long)res * cus);
    const int left = (int)((n - full * res * cus + cus - 1) / cus);
    const double steps = (double)((K + 16 * groups - 1) / (16 * groups)) * groups;
    const double us = steps * (full * t[res - 1] + (left > 0 ? t[left - 1] : 0.0)) + 2500.0 * (double)(full + (left > 0));
    if (f == k64x64 || us < best) { best = us; form = f; }
  };
  consider(k64x64, 64, 64, 1, 4, t64);
  consider(k64x64x2, 64, 64, 2, 2, t64x2);
  consider(k64x64x4, 64, 64, 4, 1, t64x4);
  consider(k64x128, 64, 128, 1, 3, t64x128);
  consider(k128x128, 128, 128, 1, 2, t128);
  return form;
}

template <int EPI, bool A_KC, bool B_KC, bool K_KEPT = false>
int launch_form(const GemmArgs& a, int E, int R, int N, int K, hipStream_t st) {
  int cus = 0;
  if (compute_units(&cus) != MOE_OK) return MOE_EHIP;
  switch (f32_form(E, R, N, K, cus)) {
    case k64x64: return launch_tiles<1, 1, 4, 1, EPI, A_KC, B_KC, K_KEPT>(a, E, R, N, K, st);
    case k64x64x2: return launch_tiles<1, 1, 2, 2, EPI, A_KC, B_KC, K_KEPT>(a, E, R, N, K, st);
    case k64x64x4: return launch_tiles<1, 1, 2, 4, EPI, A_KC, B_KC, K_KEPT>(a, E, R, N, K, st);
    case k64x128: return launch_tiles<1, 2, 2, 1, EPI, A_KC, B_KC, K_KEPT>(a, E, R, N, K, st);
    default: return launch_tiles<2, 2, 2, 1, EPI, A_KC, B_KC, K_KEPT>(a, E, R, N, K, st);
  }
}

}  // namespace

int prepare_gemm_f32() {
  const int rcs[] = {
#define MOE_F32_ALL(...)                                                                              \
  prepare_tiles<1, 1, 4, 1, __VA_ARGS__>(), prepare_tiles<1, 1, 2, 2, __VA_ARGS__>(),                \
      prepare_tiles<1, 1, 2, 4, __VA_ARGS__>(), prepare_tiles<1, 2, 2, 1, __VA_ARGS__>(),            \
      prepare_tiles<2, 2, 2, 1, __VA_ARGS__>()
      MOE_F32_ALL(0, true, false, false), MOE_F32_ALL(1, true, false, false), MOE_F32_ALL(0, true, true, false),
      MOE_F32_ALL(2, true, true, false), MOE_F32_ALL(0, false, false, true), MOE_F32_ALL(0, false, false, false)};
#undef MOE_F32_ALL
  for (int rc : rcs)
    if (rc != MOE_OK) return rc;
  return MOE_OK;
}

int launch_gemm_f32(GemmKind kind, const GemmArgs& a, int E, int R, int N, int K, hipStream_t st) {
  // unit strides along K (kForward: A; kDataGrad: A and B), N and R in whole 16-byte pieces
  if (E < 1 || R < 1 || N < 1 || K < 1 || N % 4 != 0 || (kind == kWeightGrad ? R : K) % 4 != 0)
    return MOE_EUNSUPPORTED;
  switch (kind) {
    case kForward: return launch_form<0, true, false>(a, E, R, N, K, st);
    case kForwardRelu: return launch_form<1, true, false>(a, E, R, N, K, st);
    case kDataGrad: return launch_form<0, true, true>(a, E, R, N, K, st);
    case kDataGradMask: return launch_form<2, true, true>(a, E, R, N, K, st);
    case kWeightGrad:
      return a.kept != nullptr ? launch_form<0, false, false, true>(a, E, R, N, K, st)
                               : launch_form<0, false, false>(a, E, R, N, K, st);
  }
  return MOE_EINVAL;
}

}  // namespace moe
