// fp32 expert GEMMs on the matrix cores (v_mfma_f32_32x32x2_f32: full fp32 products, fp32
// accumulation).  The paper trained its experts in fp32 (Section 4, "Model Details"); bf16 is
// this library's fast path, this kernel is the fp32 one for all six expert GEMMs of the forward
// and backward pass and the dense layers around them.
//
// Built like the bf16 kernel of expert_gemm.hip that takes any shape: one block of four wavefronts
// (2 x 2) per tile, operands travel global -> LDS without passing the registers
// (global_load_lds_dwordx4, 1 KB per wavefront instruction, three stages of 16 k), every lane with its
// own source address, and a row, column or k past an edge, or an unoccupied packed row, reads a zero
// line.  Unit strides run along dimensions that are multiples of 4 elements.
//
//   K-contiguous operand [rows][K]: stage [rows][4 chunks of 4 k], chunk c of row r at position
//     c ^ ((r>>2)&3); a lane reads 16 bytes = the 4 k of four MFMA steps.
//   row-of-k operand [K][rows]: stage [16 k][rows / 4 chunks], chunk c of row k at c ^ (8 ((k>>2)&1));
//     one 4-byte read per step.  (64 banks: both reads touch every bank once)
// Lane half h of step j of an 8-wide group of k takes k = 4 h + j in both operands.
//
// Bound: the matrix pipes (one instruction occupies its pipe for 64 cycles, so LDS and issue rates
// are far from binding); what the kernel has to do is keep them fed across the barrier and the tile's
// ends, which takes several blocks per compute unit.  The 128 x 128 kernel before this one staged
// through registers and waited for each load where it was issued.
// Forward products of 8 experts of 2048 rows, M 1024, H 4096: 111 TFLOP/s with that kernel, 132 with
// this one (0.84 of the fp32 matrix peak); 16 experts of 512 rows, M 1024, H 2048: 97 -> 129.
#include "common.h"

namespace moe {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

static __device__ const f32x4_t f32_zero_line = {0.f, 0.f, 0.f, 0.f};

constexpr int kF32Stages = 3, kBK = 16;

// T: 64 T x 64 T tile, 32 T x 32 T per wavefront.  The other parameters are those of GemmArgs and of
// the bf16 kernel: EPI 0 plain, 1 relu, 2 zero where mask[e,r,n] <= 0; gathered rows of A, kept rows
// of an expert (or, K_KEPT, the length of its sum).
template <int T, int EPI, bool A_KC, bool B_KC, bool K_KEPT>
__global__ __launch_bounds__(256, T == 2 ? 3 : 4) void gemm_f32_mfma_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ Cout,
    const float* __restrict__ mask, int R, int N, int K, int tiles_r, int tiles_n,
    const int32_t* __restrict__ gather, const int32_t* __restrict__ kept) {
  constexpr int kTile = 64 * T, kAStage = kTile * kBK * 4, kStage = 2 * kAStage, ST = kF32Stages;
  __shared__ __attribute__((aligned(16))) unsigned char smem[ST * kStage];
  typedef unsigned char __attribute__((address_space(3))) * lds_ptr;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_ptr)smem);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
  const int r0 = rt * kTile, n0 = ct * kTile;
  const int rows = kept != nullptr && !K_KEPT ? kept[e] : R;
  if (r0 >= rows) return;                                      // block-uniform
  const int KE = K_KEPT ? kept[e] : K;
  const int KT = (KE + kBK - 1) / kBK;
  const int wm0 = (wave >> 1) * 32 * T, wn0 = (wave & 1) * 32 * T;
  const int l32 = lane & 31, hf = lane >> 5;

  // per-lane sources: T copies of each operand per wavefront and step.  A copy fills 16 rows of 4
  // chunks (K-contiguous) or 4 / T k rows of 16 T chunks (row-of-k)
  constexpr int CH = 16 * T, RPC = 64 / CH;
  const uint64_t zline = (uint64_t)(uintptr_t)&f32_zero_line;
  uint64_t a_addr[T], b_addr[T];
  uint32_t a_inc[T], b_inc[T];
  int a_k[T], b_k[T];                                          // the lane's first k inside a step
#pragma unroll
  for (int q = 0; q < T; ++q) {
    const int c = wave * T + q;
    const int krow = RPC * c + lane / CH, kcol = 4 * ((lane % CH) ^ (8 * ((krow >> 2) & 1)));
    const int row = 16 * c + (lane >> 2), kch = 4 * ((lane & 3) ^ ((row >> 2) & 3));
    bool ok;
    const float* src;
    if (A_KC) {
      a_k[q] = kch;
      ok = r0 + row < rows && kch < KE;
      long long arow = (long long)e * R + r0 + row;
      if (gather != nullptr) {
        const int tok = ok ? gather[arow] : -1;
        ok = tok >= 0;
        arow = tok;
      }
      src = A + arow * K + kch;
    } else {
      a_k[q] = krow;
      ok = r0 + kcol < R && krow < KE;
      src = A + ((size_t)e * K + krow) * R + r0 + kcol;
    }
    a_addr[q] = ok ? (uint64_t)(uintptr_t)src : zline;
    a_inc[q] = ok ? (A_KC ? kBK * 4 : (uint32_t)R * kBK * 4) : 0u;
    if (B_KC) {
      b_k[q] = kch;
      ok = n0 + row < N && kch < KE;
      src = B + ((size_t)e * N + n0 + row) * K + kch;
    } else {
      b_k[q] = krow;
      ok = n0 + kcol < N && krow < KE;
      src = B + ((size_t)e * K + krow) * N + n0 + kcol;
    }
    b_addr[q] = ok ? (uint64_t)(uintptr_t)src : zline;
    b_inc[q] = ok ? (B_KC ? kBK * 4 : (uint32_t)N * kBK * 4) : 0u;
  }
#define MOE_F32_COPY(LDS_U32, ADDR_U64)                                                      \
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"            \
               :: "s"(LDS_U32), "v"(ADDR_U64) : "memory")
  auto start_step = [&](int p, int stage) {                    // the next step in order
    if (p > 0) {
#pragma unroll
      for (int q = 0; q < T; ++q) { a_addr[q] += a_inc[q]; b_addr[q] += b_inc[q]; }
      const int kl = KE - p * kBK;                             // k left, this step's included
      if (kl < kBK) {                                          // block-uniform, last step only
#pragma unroll
        for (int q = 0; q < T; ++q) {
          if (a_k[q] >= kl) a_addr[q] = zline;
          if (b_k[q] >= kl) b_addr[q] = zline;
        }
      }
    }
    const uint32_t la = lds0 + stage * kStage + wave * (T * 1024);
#pragma unroll
    for (int q = 0; q < T; ++q) {
      MOE_F32_COPY(la + q * 1024, a_addr[q]);
      MOE_F32_COPY(la + kAStage + q * 1024, b_addr[q]);
    }
  };

  // fragment reads of k group kg (8 k): value j is step j's operand
  typedef f32x4_t __attribute__((address_space(3))) * lds_f4_ptr;
  typedef float __attribute__((address_space(3))) * lds_f_ptr;
  auto read_frag = [&](bool kc, uint32_t base, int w0, int i, int kg) {
    const int row = w0 + 32 * i + l32;
    if (kc)
      return *(lds_f4_ptr)(uintptr_t)(base + row * 64 + (((2 * kg + hf) ^ ((row >> 2) & 3)) * 16));
    f32x4_t v;
    const uint32_t p = base + (8 * kg + 4 * hf) * (kTile * 4) + (((row >> 2) ^ (8 * hf)) * 16) + 4 * (row & 3);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = *(lds_f_ptr)(uintptr_t)(p + j * (kTile * 4));
    return v;
  };

  f32x16_t acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  int p = 0, pstage = 0;
  for (; p < ST - 1 && p < KT; ++p) {
    start_step(p, pstage);
    ++pstage;
  }
  int stage = 0;
  for (int s = 0; s < KT; ++s) {
    // own copies of step s landed (step s + 1 may still fly), then everybody's; the stage of step
    // s - 1 is free after the barrier
    if (s + 1 < KT) {
      if (T == 2) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
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
    for (int kg = 0; kg < 2; ++kg) {
      f32x4_t a[T], b[T];
#pragma unroll
      for (int i = 0; i < T; ++i) {
        a[i] = read_frag(A_KC, sb, wm0, i, kg);
        b[i] = read_frag(B_KC, sb + kAStage, wn0, i, kg);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][q], b[j][q], acc[i][j], 0, 0, 0);
    }
  }
  // acc[i][j][v]: row 32 i + 8 (v/4) + 4 hf + v%4, column 32 j + lane%32 of the wavefront tile: a store
  // covers whole 128-byte pieces of two rows
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = r0 + wm0 + 32 * i + 8 * (v >> 2) + 4 * hf + (v & 3);
      if (r >= rows) continue;
      const size_t o = ((size_t)e * R + r) * N;
#pragma unroll
      for (int j = 0; j < T; ++j) {
        const int n = n0 + wn0 + 32 * j + l32;
        if (n >= N) continue;
        float x = acc[i][j][v];
        if (EPI == 1) x = fmaxf(x, 0.f);
        if (EPI == 2) x = mask[o + n] > 0.f ? x : 0.f;
        Cout[o + n] = x;
      }
    }
#undef MOE_F32_COPY
}

template <int T, int EPI, bool A_KC, bool B_KC, bool K_KEPT>
int launch_tiles(const GemmArgs& a, int E, int R, int N, int K, hipStream_t st) {
  const int tiles_r = (R + 64 * T - 1) / (64 * T), tiles_n = (N + 64 * T - 1) / (64 * T);
  const long long nblk = (long long)E * tiles_r * tiles_n;
  if (nblk > 0x7fffffffLL) return MOE_EUNSUPPORTED;
  hipLaunchKernelGGL((gemm_f32_mfma_kernel<T, EPI, A_KC, B_KC, K_KEPT>), dim3((unsigned)nblk), dim3(256), 0,
                     st, static_cast<const float*>(a.A), static_cast<const float*>(a.B),
                     static_cast<float*>(a.C), static_cast<const float*>(a.mask), R, N, K, tiles_r,
                     tiles_n, a.gather, a.kept);
  return check_launch();
}

// 128 x 128 or 64 x 64 tiles: whichever keeps the fullest compute unit busy for a shorter time.  Of the
// larger three share a unit, one alone reaches 0.74 of the fp32 matrix rate, three 0.84; of the smaller
// six share it, 0.5 for one, 0.74 from four on.  (h = relu(buf wi), out = h wo, 128 / 64, us:
//   E 16 R 512 M 1024 H 2048  533 / 604    E 8  R 2048 M 1024 H 4096  2090 / 2365
//   E 24 R 295 M 768  H 3072  732 / 663    E 16 R 128  M 512  H 1024   114 / 48.7
//   E 4  R 512 M 512  H 2048  183 / 90.3   E 32 R 64   M 1024 H 2048   278 / 174)
template <int EPI, bool A_KC, bool B_KC, bool K_KEPT = false>
int launch_form(const GemmArgs& a, int E, int R, int N, int K, hipStream_t st) {
  int cus = 0;
  if (compute_units(&cus) != MOE_OK) return MOE_EHIP;
  auto tiles = [&](int edge) { return (long long)E * ((R + edge - 1) / edge) * ((N + edge - 1) / edge); };
  static const double t128[] = {4 / 0.74, 8 / 0.80, 12 / 0.84},
                      t64[] = {1 / 0.5, 2 / 0.65, 3 / 0.7, 4 / 0.74, 5 / 0.74, 6 / 0.74};
  const bool small = tiles_time(tiles(64), cus, 6, t64) < tiles_time(tiles(128), cus, 3, t128);
  return small ? launch_tiles<1, EPI, A_KC, B_KC, K_KEPT>(a, E, R, N, K, st)
               : launch_tiles<2, EPI, A_KC, B_KC, K_KEPT>(a, E, R, N, K, st);
}

}  // namespace

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
