// Expert networks (Eq. 2 of the paper; Algorithm 2: EGCM,EMH->EGCH, relu,
// EGCH,EHM->EGCM) as two grouped GEMMs over the experts, and the four GEMMs of
// their backward pass:
//
//   h[e]   = relu(buf[e] . wi[e])     [R, M] x [M, H],  R = G*C rows per expert
//   out[e] = h[e] . wo[e]             [R, H] x [H, M]
//
// bf16, v_mfma_f32_32x32x16_bf16 with fp32 accumulation, in two kernels:
//
//   expert_gemm_bf16_dma_kernel   column counts of whole 256-wide tiles with K % 32 == 0, any
//     number of rows of a K-contiguous operand (the large layers): persistent, one block per CU walks its share of the
//     tiles as one stream of K steps; operands travel global -> LDS without passing
//     the registers; either operand in either layout; gathered rows, packed rows,
//     scattered result rows and a per-expert k range as template options.
//   expert_gemm_bf16_edge_kernel  every other shape, and outputs of few tiles: one block per
//     tile of 128 x 256 down to 64 x 64, two to four blocks per CU, the same register-bypassing
//     copies with per-lane source addresses (pieces past an edge come from a zero line).
//     expert_gemm_bf16_pair_kernel runs the tiles of two such products in one launch.
//
// In all, activation tiles (K contiguous) sit in LDS as [m][k] and are read with
// 16-byte loads; weight tiles are [k][n] in memory (N contiguous), stay that way in
// LDS and are read with ds_read_b64_tr_b16, which hands every lane the 4 consecutive
// k of its column that the MFMA operand wants.  Blocks of one XCD (own L2) take
// neighbouring tiles so that they share operand panels.
//
// fp32 layers run the kernel of gemm_f32.hip.
#include "common.h"

namespace moe {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));   // native 16-byte vector
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

constexpr int kXcds = 8;

__device__ __forceinline__ int xcd_remap(int bid, int nblk) {
  const int q = nblk / kXcds, r = nblk % kXcds;
  const int xcd = bid % kXcds, idx = bid / kXcds;
  return xcd * q + (xcd < r ? xcd : r) + idx;
}

// ----------------------------------------------------------------------------
// 256x256 tiles: a persistent kernel (one block per CU) that walks its share
// of the tiles as ONE stream of 32-wide K steps.
//
// Global -> LDS copies bypass the registers (global_load_lds_dwordx4), ST stages of
// 32 KB, the copy of step g+ST-1 is started during step g, also across a tile
// boundary: the next tile's first stages land while the current tile is finished
// and stored, so neither the fill of the pipeline nor the drain of the stores is
// paid per tile.
//
// One wavefront copy instruction fills 1 KB of LDS (lane l -> bytes 16 l ..), which
// fixes the LDS layout to unpadded rows; bank conflicts are avoided by permuting
// which 16-byte chunk of a row a lane fetches:
//   A stage [256 rows][4 chunks of 8 k]:  chunk c of row r sits at position c ^ ((r>>2)&3)
//   B stage [32 k][32 chunks of 8 n]:     chunk c of row k sits at position c ^ (4 (k&3))
// (64 banks of 4 bytes: a 16-lane group of a 16-byte read, or a 32-lane group of an
// 8-byte transposing read, then touches every bank exactly once)
//
// Step g: fetch the fragments of the second k half, multiply the first half; wait
// for the own copies of step g+1 and barrier (step g+1 is now visible to all, the
// stage of step g-1 is free); then, spread between the four MFMA rows of the second
// half, start the copies of step g+ST-1 and fetch the first fragments of step g+1.
// ----------------------------------------------------------------------------
template <int ST>
struct DmaSmem {
  static constexpr int kAStage = 256 * 32 * 2, kBStage = 32 * 256 * 2;
  static constexpr int kStage = kAStage + kBStage;
  static constexpr size_t kBytes = (size_t)ST * kStage;
};

#define MOE_DMA16(LDS_U32, VOFF_U32, SBASE)                                         \
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"     \
               :: "s"(LDS_U32), "v"(VOFF_U32), "s"(SBASE) : "memory")

// GATHER: the A rows are not a dense [E,R,K] buffer but rows of the matrix A ([rows, K]) picked by
// index (row p of expert e is A[src_token[e R + p], :], a zero row from kept[e] on), i.e. the
// dispatch of Algorithm 2 folded into the first GEMM's copies.
//
// Operand layouts.  "K-contiguous" (KC): the operand is stored [rows][K] (row = its index in
// the output) and staged as [256 rows][4 chunks]; "row-of-k" (MNC): stored [K][rows] and
// staged as [32 k][32 chunks], read with the transposing LDS load.  Either operand can have
// either layout; both fragment kinds hand a lane the 8 consecutive k of its row:
//   forward       C = A . B        A KC  [R,K],  B MNC [K,N]
//   data gradient C = A . B^T      A KC  [R,K],  B KC  [N,K]      (A_MNC = false, B_KC = true)
//   weight grad.  C = A^T . B      A MNC [K,R],  B MNC [K,N]      (A_MNC = true,  B_KC = false)
// EPI: 0 plain, 1 relu, 2 zero every element whose `mask` element (same [E,R,N] index as C)
// is zero -- the derivative of relu taken from the stored activations, 3 plain with an fp32
// result (Cout points to floats), 4 relu that also records which results are non-zero, one
// bit per element in `signbits`, 5 zero every element whose recorded bit is clear.
// The bit record is private to this kernel: 8 KB per 256x256 tile (tile index
// (e * tiles_m + row tile) * tiles_n + column tile), inside a tile 2 KB per wavefront laid
// out as [2][64 lanes][16 bytes] = the 32 bytes a lane meets in its own store phase (4 row
// groups x 8 stores, one byte each: bit b = column 8 c + b of that store).  Writer and reader
// are the same tiling of the same [E,R,N] matrix, so no lane ever needs another lane's bits.
// The reader fetches a tile's 8 KB into spare LDS with two register-bypassing copies issued
// in the tile's first K step; the waits of the next two steps cover them.
// PACKED: expert e has only its first ceil(kept[e] / 256) row tiles multiplied (kept[e] = its
// occupied rows): every block copies kept to LDS and forms the running tile counts there when it
// starts; the tiles of all experts are numbered consecutively in expert order, and since a
// block's tile numbers only grow it finds a tile's expert by stepping a cursor forward.  Rows
// from kept[e] to the end of the last tile are multiplied as zero rows.  SCATTER (with PACKED):
// the rows of C go to the absolute rows src_token[e * R + p] of Cout ([rows, N]), -1 = not stored.
// ROWS: R is no multiple of 256.  The last row tile of an expert reads its last row in place of those past it and
// does not store them.  Before, such layers ran 128 x 256 tiles of the edge kernel (us, before / after): 16 000 rows,
// 1024 x 6144 264 / 240, 2048 x 1024 81 / 66; out and dbuf of 10 experts of 2852 rows, M 1024, H 8192 540 / 482
// and 591 / 518, dh 671 / 584.
// DYNK: the sum over k of expert e stops at 256 ceil(kept[e] / 256) instead of K (the weight
// gradients, whose k runs over an expert's packed rows); an expert with no rows gets zeros.
template <int ST, int EPI, bool GATHER, bool A_MNC, bool B_KC, bool PACKED, bool SCATTER, bool DYNK, bool ROWS>
__global__ __launch_bounds__(256) void expert_gemm_bf16_dma_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, bf16_t* __restrict__ Cout,
    int R, int N, int K, int tiles_m, int tiles_n, int ntiles_static,
    const int32_t* __restrict__ src_token, const bf16_t* __restrict__ zero_row,
    const bf16_t* __restrict__ mask, unsigned char* __restrict__ signbits, const int32_t* __restrict__ kept, int E) {
  static_assert(!(GATHER && A_MNC), "the gather form addresses whole rows of a K-contiguous A");
  static_assert(!GATHER || PACKED, "gathered rows are packed rows");
  static_assert(!SCATTER || (PACKED && EPI == 0), "scattered rows: plain bf16 result of a packed launch");
  static_assert(!(DYNK && (PACKED || GATHER)), "a shortened k range comes with the full list of output tiles");
  static_assert(!ROWS || !(A_MNC || SCATTER || DYNK || EPI == 3), "rows of a K-contiguous A and of C");
  constexpr bool RELU = EPI == 1 || EPI == 4;
  using SM = DmaSmem<ST>;
  constexpr int BM = 256, BN = 256, BK = 32, TM = 4, TN = 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  typedef unsigned char __attribute__((address_space(3))) * lds_ptr;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_ptr)smem_raw);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * 128, wn0 = (wave & 1) * 128;
  const int per_e = tiles_m * tiles_n;
  const int KT = K / BK;
  // Tile t of an expert -> (row tile, column tile): bands of kBand row tiles, inside a band
  // row tile fastest, then column tile.  The ~32 tiles an XCD works on at a time then span
  // about 8 row tiles x 4 column tiles, the split that shares the most operand panels in that
  // XCD's L2 (a tall output, as in the weight gradients, would otherwise re-read its A panel
  // once per column tile).
  constexpr int kBand = 8;   // bands of 2 or 4 row tiles measured the same on the forward shapes
  // PACKED: kept_s[e] = occupied rows of expert e, rts_s[e] = occupied row tiles of the experts
  // before e (rts_s[E] = all of them), behind the stages and the token / bit areas in LDS
  int* const kept_s = reinterpret_cast<int*>(smem_raw + SM::kBytes + (GATHER ? 1024 : 0) + (EPI == 5 ? 8192 : 0));
  int* const rts_s = kept_s + E;
  if (PACKED || DYNK) {
    for (int e = tid; e < E; e += 256) kept_s[e] = kept[e];
    __syncthreads();
  }
  if (PACKED) {
    if (wave == 0) {
      // lane l scans experts [l per, (l+1) per); the lanes' sums meet in a wavefront scan
      const int per = (E + 63) / 64, b0 = lane * per;
      int sum = 0;
      for (int j = 0; j < per; ++j)
        if (b0 + j < E) sum += (kept_s[b0 + j] + 255) >> 8;
      int incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      int run = incl - sum;
      for (int j = 0; j < per; ++j)
        if (b0 + j < E) {
          rts_s[b0 + j] = run;
          run += (kept_s[b0 + j] + 255) >> 8;
        }
      if (lane == 63) rts_s[E] = incl;
    }
    __syncthreads();
  }
  const int ntiles = PACKED ? __builtin_amdgcn_readfirstlane(rts_s[E]) * tiles_n : ntiles_static;
  // PACKED: expert of the tile located last and its range of row tiles [rs, re) in the global
  // numbering; one cursor for the copies (producer side), one for the epilogues
  struct TileCursor { int e, rs, re; };
  TileCursor pcur{-1, 0, 0}, ccur{-1, 0, 0};
#define MOE_DMA_TILE(T_, CUR_, e_, rt_, ct_)                                                 \
  int e_, rt_, ct_;                                                                          \
  {                                                                                          \
    int t_, tm_;                                                                             \
    if (PACKED) {                                                                            \
      /* ends at the latest with e = E - 1: T_ < ntiles = rts_s[E] * tiles_n */              \
      while ((T_) >= CUR_.re * tiles_n && CUR_.e + 1 < E) {                                  \
        ++CUR_.e;                                                                            \
        CUR_.rs = CUR_.re;                                                                   \
        CUR_.re = __builtin_amdgcn_readfirstlane(rts_s[CUR_.e + 1]);                         \
      }                                                                                      \
      e_ = CUR_.e;                                                                           \
      t_ = (T_) - CUR_.rs * tiles_n;                                                         \
      tm_ = CUR_.re - CUR_.rs;                                                               \
    } else {                                                                                 \
      e_ = (T_) / per_e;                                                                     \
      t_ = (T_) - e_ * per_e;                                                                \
      tm_ = tiles_m;                                                                         \
    }                                                                                        \
    const int band_ = t_ / (kBand * tiles_n), rem_ = t_ - band_ * kBand * tiles_n;           \
    const int left_ = tm_ - band_ * kBand, rows_ = left_ < kBand ? left_ : kBand;            \
    ct_ = rem_ / rows_;                                                                      \
    rt_ = band_ * kBand + (rem_ - ct_ * rows_);                                              \
  }

  // This block's tiles: XCD x = blockIdx % 8 owns a contiguous range of tiles; its
  // blocks take them round-robin, so at any time they work on neighbouring tiles
  // (row tile fastest: neighbours share a weight panel in that XCD's L2).
  const int nb = gridDim.x;
  const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int xq = ntiles / kXcds, xr = ntiles % kXcds;
  const int t_begin = xcd * xq + (xcd < xr ? xcd : xr);
  const int t_end = t_begin + xq + (xcd < xr ? 1 : 0);
  const int stride = (nb - xcd + kXcds - 1) / kXcds;           // blocks on this XCD
  const int first = t_begin + slot;
  if (first >= t_end) return;                                  // block-uniform
  // K steps of a tile of expert e_
#define MOE_DMA_STEPS(e_) (DYNK ? ((kept_s[e_] + 255) >> 8) * (256 / BK) : KT)

  // per-lane source byte offsets of the 4 + 4 copy instructions of this wavefront
  uint32_t a_voff[4], b_voff[4], a_last[4];                    // a_last: of the tile being copied (ROWS)
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = 16 * (wave * 4 + q) + (lane >> 2);
    const int ca = (lane & 3) ^ ((row >> 2) & 3);
    const int krow = 2 * (wave * 4 + q) + (lane >> 5);
    const int cb = (lane & 31) ^ (4 * (krow & 3));
    a_voff[q] = A_MNC ? (uint32_t)((krow * R + 8 * cb) * 2) : (uint32_t)((row * K + 8 * ca) * 2);
    b_voff[q] = B_KC ? (uint32_t)((row * K + 8 * ca) * 2) : (uint32_t)((krow * N + 8 * cb) * 2);
  }

  // producer cursor: the next step to copy (tile p_tile, k step p_kt) and its sources
  // (p_steps: steps of that tile; p_more: such a step exists; p_g: steps started so far)
  int p_tile = first, p_kt = 0, p_stage = 0, p_g = 0, p_steps = KT, p_more = 1;
  const bf16_t* p_a;
  const bf16_t* p_b;
  // GATHER: per-lane source addresses of the 4 row copies.  The 64 dispatch indices of this
  // wavefront's rows of a tile are copied to LDS (one more register-bypassing copy, issued
  // 4 steps before the tile's first step, so the regular waits of the steps in between
  // cover it) and read from there when the producer moves on to that tile.
  uint64_t a_addr[4];
  const uint32_t lds_tok = lds0 + (uint32_t)SM::kBytes + wave * 256;
  const uint32_t lds_bits = lds0 + (uint32_t)SM::kBytes + wave * 2048;   // EPI 5 (never with GATHER)
  typedef int __attribute__((address_space(3))) * lds_int_ptr;
#define MOE_DMA_TOKENS(TILE)                                                                 \
  {                                                                                          \
    MOE_DMA_TILE(TILE, pcur, e_, rt_, ct_)                                                   \
    (void)ct_;                                                                               \
    int p_ = rt_ * BM + 64 * wave + lane;                                                    \
    if (ROWS) p_ = p_ < R ? p_ : R - 1;                                                      \
    const uint64_t ta_ = (uint64_t)(uintptr_t)(src_token + (size_t)e_ * R + p_);             \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"            \
                 :: "s"(lds_tok), "v"(ta_) : "memory");                                      \
  }
#define MOE_DMA_GATHER_ROWS(e_, m0_)                                                         \
  {                                                                                          \
    _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                          \
      const int rl_ = 16 * q + (lane >> 2);                                                  \
      const int tok_ = *(lds_int_ptr)(uintptr_t)(lds_tok + 4 * rl_);                         \
      const int row_ = 64 * wave + rl_;                                                      \
      const int ca_ = (lane & 3) ^ ((row_ >> 2) & 3);                                        \
      const bf16_t* src_ = (m0_) + row_ < kept_s[e_] && tok_ >= 0 ? A + (size_t)tok_ * K : zero_row; \
      a_addr[q] = (uint64_t)(uintptr_t)(src_ + 8 * ca_);                                     \
    }                                                                                        \
  }
#define MOE_DMA16_ADDR(LDS_U32, ADDR_U64)                                                    \
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"            \
               :: "s"(LDS_U32), "v"(ADDR_U64) : "memory")
#define MOE_DMA_COPY_A(LDS_U32, q)                                                           \
  if (GATHER) { MOE_DMA16_ADDR(LDS_U32, a_addr[q]); }                                         \
  else { MOE_DMA16(LDS_U32, (ROWS ? a_last[q] : a_voff[q]), p_a); }
#define MOE_DMA_SET_SOURCES()                                                                \
  {                                                                                          \
    if (DYNK) {                                 /* pass over tiles without a single k step */ \
      while (p_tile < t_end && MOE_DMA_STEPS(p_tile / per_e) == 0) p_tile += stride;         \
    }                                                                                        \
    p_more = __builtin_amdgcn_readfirstlane(p_tile < t_end);                                 \
    if (p_more) {                                                                            \
      MOE_DMA_TILE(p_tile, pcur, e_, rt_, ct_)                                               \
      p_steps = __builtin_amdgcn_readfirstlane(MOE_DMA_STEPS(e_));                           \
      if (GATHER) MOE_DMA_GATHER_ROWS(e_, rt_ * BM)                                          \
      else if (A_MNC) p_a = A + (size_t)e_ * K * R + (size_t)rt_ * BM;                       \
      else {                                                                                 \
        p_a = A + ((size_t)e_ * R + (size_t)rt_ * BM) * K;                                   \
        if (ROWS) {                                                                          \
          _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                    \
            const int row_ = 16 * (wave * 4 + q) + (lane >> 2), past_ = row_ - (R - 1 - rt_ * BM); \
            a_last[q] = a_voff[q] - (past_ > 0 ? (uint32_t)(past_ * K * 2) : 0u);            \
          }                                                                                  \
        }                                                                                    \
      }                                                                                      \
      if (B_KC) p_b = B + ((size_t)e_ * N + (size_t)ct_ * BN) * K;                           \
      else p_b = B + (size_t)e_ * K * N + (size_t)ct_ * BN;                                  \
    }                                                                                        \
  }
#define MOE_DMA_ADVANCE()                                                                    \
  {                                                                                          \
    ++p_g;                                                                                   \
    p_stage = p_stage + 1 == ST ? 0 : p_stage + 1;                                           \
    if (GATHER) {                                                                            \
      _Pragma("unroll") for (int q = 0; q < 4; ++q) a_addr[q] += BK * 2;                     \
      if (p_kt == KT - 4 && p_tile + stride < t_end) MOE_DMA_TOKENS(p_tile + stride)         \
    } else p_a += A_MNC ? (size_t)BK * R : (size_t)BK;                                       \
    p_b += B_KC ? (size_t)BK : (size_t)BK * N;                                               \
    if (++p_kt == p_steps) { p_kt = 0; p_tile += stride; MOE_DMA_SET_SOURCES() }             \
  }
  if (GATHER) {
    MOE_DMA_TOKENS(first)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  MOE_DMA_SET_SOURCES()

  // fragment read offsets (bytes inside a stage); w0 = the wavefront's first row of the operand
  //   KC operand: row w0 + 32 i + lane%32, chunk 2 kk + lane/32 at its permuted position
  //   MNC operand (transposing read): 16-lane block b = lane/16 covers k rows
  //   8 (b/2) + (lane%16)/4 (+4), rows w0 + 32 j + 16 (b%2) + 4 (lane%4) .. +3; chunk = row / 8
  const int ar = lane & 31;
  const int p16 = lane & 15, bb = lane >> 4;
  const int bk = 8 * (bb >> 1) + (p16 >> 2);                   // k row inside a 16-wide step
  const int bsw = 4 * (bk & 3);                                // permutation of that row
  uint32_t a_rd[4], b_rd[4];                                   // KC: [kk], MNC: [sub-tile]
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int kc_chunk = (2 * (j & 1) + (lane >> 5)) ^ ((ar >> 2) & 3);
    const int ca = (wm0 >> 3) + 4 * j + 2 * (bb & 1) + ((p16 & 3) >> 1);
    const int cb = (wn0 >> 3) + 4 * j + 2 * (bb & 1) + ((p16 & 3) >> 1);
    a_rd[j] = A_MNC ? (uint32_t)(bk * 512 + ((ca ^ bsw) * 16) + (p16 & 1) * 8)
                    : (uint32_t)((wm0 + ar) * 64 + kc_chunk * 16);
    b_rd[j] = B_KC ? (uint32_t)(SM::kAStage + (wn0 + ar) * 64 + kc_chunk * 16)
                   : (uint32_t)(SM::kAStage + bk * 512 + ((cb ^ bsw) * 16) + (p16 & 1) * 8);
  }
  typedef s16x4_t __attribute__((address_space(3))) * lds_s16x4_ptr;
  typedef bf16x8_t __attribute__((address_space(3))) * lds_bf16x8_ptr;
  struct Frags { bf16x8_t a[TM]; bf16x8_t b[TN]; };
#define MOE_DMA_READ_KC(DST, STAGE, RD, kk, i)                                               \
  DST = *(lds_bf16x8_ptr)(uintptr_t)(lds0 + (STAGE) * SM::kStage + RD[kk] + (i) * 32 * 64);
#define MOE_DMA_READ_MNC(DST, STAGE, RD, kk, j)                                              \
  {                                                                                          \
    const uint32_t pb_ = lds0 + (STAGE) * SM::kStage + RD[j] + (kk) * 16 * 512;              \
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)pb_); \
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(                              \
        (lds_s16x4_ptr)(uintptr_t)(pb_ + 4 * 512));                                          \
    DST = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)); \
  }
#define MOE_DMA_READ_A(F, STAGE, kk, i)                                                      \
  { if (A_MNC) MOE_DMA_READ_MNC((F).a[i], STAGE, a_rd, kk, i) else { MOE_DMA_READ_KC((F).a[i], STAGE, a_rd, kk, i) } }
#define MOE_DMA_READ_B(F, STAGE, kk, j)                                                      \
  { if (B_KC) { MOE_DMA_READ_KC((F).b[j], STAGE, b_rd, kk, j) } else MOE_DMA_READ_MNC((F).b[j], STAGE, b_rd, kk, j) }
  // The weight fragment goes in as the first MFMA operand: the 32x32 result is then
  // the transposed tile, i.e. a lane owns 4 consecutive columns of one row of C.
#define MOE_DMA_MFMA_ROW(F, i)                                                               \
  _Pragma("unroll") for (int j = 0; j < TN; ++j)                                             \
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16((F).b[j], (F).a[i], acc[i][j], 0, 0, 0);

  Frags fr[2];
  // start the first ST-1 steps (as many as there are), wait for step 0
  for (int tl = 0; tl < ST - 1 && p_more; ++tl) {
    const uint32_t la_ = lds0 + p_stage * SM::kStage + wave * 4096;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      MOE_DMA_COPY_A(la_ + q * 1024, q)
      MOE_DMA16(la_ + SM::kAStage + q * 1024, b_voff[q], p_b);
    }
    MOE_DMA_ADVANCE()
  }
  if (p_g >= 3) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
  else if (p_g == 2) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TM; ++i) { MOE_DMA_READ_A(fr[0], 0, 0, i) MOE_DMA_READ_B(fr[0], 0, 0, i) }

  int stage = 0, g = 0;                                        // consumer cursor
  // The fragment reads are unconditional (the very last step fetches fragments nobody
  // multiplies, from a valid stage): a conditional read would make every later wait
  // for LDS data wait for all outstanding reads instead of the older ones only.
  for (int c_tile = first; c_tile < t_end; c_tile += stride) {
    MOE_DMA_TILE(c_tile, ccur, e, rt, ct)
    const int c_steps = __builtin_amdgcn_readfirstlane(MOE_DMA_STEPS(e));
    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    for (int kt = 0; kt < c_steps; ++kt, ++g) {
      // (a fragment row's reads go out right before the MFMA row of the other k half: pinned,
      // it measures 0.6-0.8 % faster than leaving the order to the compiler)
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        MOE_DMA_READ_A(fr[1], stage, 1, i) MOE_DMA_READ_B(fr[1], stage, 1, i)
        MOE_DMA_MFMA_ROW(fr[0], i)
        __builtin_amdgcn_sched_barrier(0);
      }
      // The own copies of step g+1 must have landed; younger steps (8 copies each) may
      // still fly.  p_g steps have been started.  Copies land in the order they were issued,
      // but stores complete in no fixed order relative to them: "at most n operations
      // outstanding" therefore still proves that all but the n youngest copies have landed,
      // it just may wait for stores as well.  An epilogue first awaits every copy issued so
      // far (steps up to g+3) and only then issues its stores, so the first two steps of the
      // following tile need no wait at all and the stores drain behind their MFMAs.
      // (The counts pass through an empty asm so that the optimiser cannot peel or
      // duplicate the loop body around these conditions: copies of the body would shuffle
      // the 256 accumulator registers between them.)
      // the step to await is g+1, or the last one when the producer has started them all
      int younger = p_g - 1 - (p_more || g + 1 < p_g ? g + 1 : p_g - 1);
      if (kt < 2 && c_tile != first) younger = 3;              // landed before the last epilogue
      younger = __builtin_amdgcn_readfirstlane(younger);
      asm volatile("" : "+s"(younger));
      if (younger <= 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      else if (younger == 1) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      else if (younger == 2) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
      __syncthreads();
      if (EPI == 5 && kt == 0) {
        const unsigned char* src5 = signbits + ((size_t)(e * tiles_m + rt) * tiles_n + ct) * 8192 +
                                    wave * 2048 + lane * 16;
        MOE_DMA16_ADDR(lds_bits, (uint64_t)(uintptr_t)src5);
        MOE_DMA16_ADDR(lds_bits + 1024, (uint64_t)(uintptr_t)(src5 + 1024));
      }
      const int nstage = stage + 1 == ST ? 0 : stage + 1;      // stage of step g+1
      int more = p_more;                                       // p_stage: stage of step g-1, free now
      asm volatile("" : "+s"(more));
      const uint32_t la_ = lds0 + p_stage * SM::kStage + wave * 4096;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (more) {
          MOE_DMA_COPY_A(la_ + q * 1024, q)
          MOE_DMA16(la_ + SM::kAStage + q * 1024, b_voff[q], p_b);
        }
        MOE_DMA_READ_A(fr[0], nstage, 0, q)
        MOE_DMA_READ_B(fr[0], nstage, 0, q)
        MOE_DMA_MFMA_ROW(fr[1], q)
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more) MOE_DMA_ADVANCE()
      stage = nstage;
    }

    // Tile finished: acc[i][j][4 q + r] = C[32 i + r32][32 j + 8 q + 4 h + r], r32 = lane%32,
    // h = lane/32.  The stage of the step just consumed is free until the next step's
    // barrier, so each wavefront turns its tile through 8 KB of it, 32 rows at a time, into
    // full-row 16-byte stores.  Staging layout: [32 rows][16 chunks of 16 bytes], chunk c of
    // row r at position c ^ (r & 15), its two 8-byte halves swapped when r >= 16 (then the
    // 32 lanes of a half-wave write 256 distinct bytes: no bank conflict).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // every copy issued so far
    const int m0 = rt * BM, n0 = ct * BN;
    const size_t c_off = ((size_t)e * R + m0 + wm0) * N + n0 + wn0;
    bf16_t* Ce = Cout + c_off;
    // ROWS: stores past the wavefront's last row are past the end of this buffer, and dropped there (branches
    // around them cost registers that the K loop does not have)
    const int rows_left = R - m0 - wm0 < 128 ? R - m0 - wm0 : 128;
    __amdgpu_buffer_rsrc_t c_rsrc;
    if (ROWS)
      c_rsrc = __builtin_amdgcn_make_buffer_rsrc(Ce, 0, rows_left > 0 ? ((rows_left - 1) * N + 128) * 2 : 0, 0x00027000);
    const uint32_t st_base = lds0 + (stage == 0 ? ST - 1 : stage - 1) * SM::kStage + wave * 8192;
    const int r32 = lane & 31, hh = lane >> 5;
    const uint32_t st_wr = st_base + r32 * 256 + 8 * (hh ^ (r32 >> 4));
    typedef u32x2_t __attribute__((address_space(3))) * lds_u2_ptr;
    typedef u32x4_t __attribute__((address_space(3))) * lds_u4_ptr;
    if (EPI == 3) {
      // fp32 result: Cout is a float array; each lane stores its 4 consecutive columns
      float* Cf = reinterpret_cast<float*>(Cout) + c_off;
      typedef float f32x4_t __attribute__((ext_vector_type(4)));
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4_t*>(Cf + (size_t)(32 * i + r32) * N + 32 * j + 8 * q + 4 * hh) =
                f32x4_t{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2],
                        acc[i][j][4 * q + 3]};
        __builtin_amdgcn_sched_barrier(0);
      }
      continue;
    }
    u32x4_t bits[2] = {u32x4_t{0u, 0u, 0u, 0u}, u32x4_t{0u, 0u, 0u, 0u}};
    if (EPI == 5) {
      bits[0] = *(lds_u4_ptr)(uintptr_t)(lds_bits + lane * 16);
      bits[1] = *(lds_u4_ptr)(uintptr_t)(lds_bits + 1024 + lane * 16);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      int drow[8];                                             // SCATTER: destination rows
      if (SCATTER) {
#pragma unroll
        for (int ps = 0; ps < 8; ++ps) {
          const int pr = m0 + wm0 + 32 * i + 4 * ps + (lane >> 4);
          drow[ps] = pr < kept_s[e] ? src_token[(size_t)e * R + pr] : -1;
        }
      }
      u32x4_t mk[8];
      if (EPI == 2) {
#pragma unroll
        for (int ps = 0; ps < 8; ++ps) {
          int mrow = m0 + wm0 + 32 * i + 4 * ps + (lane >> 4);
          if (ROWS) mrow = mrow < R ? mrow : R - 1;            // (the result of such a row is not stored)
          mk[ps] = *reinterpret_cast<const u32x4_t*>(
              mask + ((size_t)e * R + mrow) * N + n0 + wn0 + 8 * (lane & 15));
        }
      }
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t lo = pack_bf16x2(acc[i][j][4 * q], acc[i][j][4 * q + 1]);
          uint32_t hi = pack_bf16x2(acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
          if (RELU) { lo = relu_bf16x2(lo); hi = relu_bf16x2(hi); }
          *(lds_u2_ptr)(uintptr_t)(st_wr + (((4 * j + q) ^ (r32 & 15)) * 16)) = u32x2_t{lo, hi};
        }
#pragma unroll
      for (int ps = 0; ps < 8; ++ps) {
        const int rr = 4 * ps + (lane >> 4), c = lane & 15;
        u32x4_t d = *(lds_u4_ptr)(uintptr_t)(st_base + rr * 256 + ((c ^ (rr & 15)) * 16));
        if (ps >= 4) d = u32x4_t{d[2], d[3], d[0], d[1]};      // rows 16..31: halves were swapped
        if (EPI == 2) {
#pragma unroll
          for (int w = 0; w < 4; ++w)
            d[w] &= ((mk[ps][w] & 0xffffu) ? 0xffffu : 0u) | ((mk[ps][w] >> 16) ? 0xffff0000u : 0u);
        }
        if (EPI == 4) {
          uint32_t byte = 0;
#pragma unroll
          for (int w = 0; w < 4; ++w)
            byte |= ((d[w] & 0xffffu) ? 1u : 0u) << (2 * w) | ((d[w] >> 16) ? 2u : 0u) << (2 * w);
          bits[i >> 1][2 * (i & 1) + (ps >> 2)] |= byte << (8 * (ps & 3));
        }
        if (EPI == 5) {
          const uint32_t byte = bits[i >> 1][2 * (i & 1) + (ps >> 2)] >> (8 * (ps & 3));
#pragma unroll
          for (int w = 0; w < 4; ++w)
            d[w] &= ((byte >> (2 * w)) & 1u ? 0xffffu : 0u) | ((byte >> (2 * w + 1)) & 1u ? 0xffff0000u : 0u);
        }
        if (SCATTER) {
          if (drow[ps] >= 0)
            *reinterpret_cast<u32x4_t*>(Cout + (size_t)drow[ps] * N + n0 + wn0 + 8 * c) = d;
        } else if (ROWS) {
          __builtin_amdgcn_raw_buffer_store_b128(d, c_rsrc, ((32 * i + rr) * N + 8 * c) * 2, 0, 0);
        } else {
          *reinterpret_cast<u32x4_t*>(Ce + (size_t)(32 * i + rr) * N + 8 * c) = d;
        }
      }
      __builtin_amdgcn_sched_barrier(0);   // one row group at a time: small register need
    }
    if (EPI == 4) {
      unsigned char* dst4 = signbits + ((size_t)(e * tiles_m + rt) * tiles_n + ct) * 8192 +
                            wave * 2048 + lane * 16;
      *reinterpret_cast<u32x4_t*>(dst4) = bits[0];
      *reinterpret_cast<u32x4_t*>(dst4 + 1024) = bits[1];
    }
  }
#undef MOE_DMA_SET_SOURCES
#undef MOE_DMA_STEPS
#undef MOE_DMA_TILE
#undef MOE_DMA_GATHER_ROWS
#undef MOE_DMA_TOKENS
#undef MOE_DMA16_ADDR
#undef MOE_DMA_COPY_A
#undef MOE_DMA_ADVANCE
#undef MOE_DMA_READ_A
#undef MOE_DMA_READ_KC
#undef MOE_DMA_READ_MNC
#undef MOE_DMA_READ_B
#undef MOE_DMA_MFMA_ROW
}

// ----------------------------------------------------------------------------
// Tiles of any shape: C [E,R,N] with R, N, K arbitrary (contiguous dimensions multiples of 8
// elements), either operand in either layout (the products of the table above).
//
// One block of four wavefronts (2 x 2) per BM x BN tile, wavefront tile BM/2 x BN/2, K steps of BK = 32
// or 64 in ST LDS stages (which, and why: gemm_form).  The copies are those
// of the persistent kernel (1 KB per wavefront instruction, the same source permutation against bank
// conflicts), but every lane carries its own 64-bit source address: a row, column or k past an edge,
// an unoccupied packed row, reads a zero line instead, so the inner loop knows no edges and nothing
// outside an operand is touched.
// Two (BN = 256, deep forms) to four (64 x 64) blocks share a compute unit: while one waits for its step or
// stores its tile the others multiply, and the dispatcher evens out tiles of different length,
// which a persistent block cannot.
//
// gather: NULL, or the rows of A (K-contiguous) are the absolute rows gather[e R + p].
// kept:   NULL, or occupied rows of each expert (packed layout): row tiles past them are left
//         alone; row_pad 255: up to 255 rows of zeros follow them, to the next multiple of 256, which
//         the persistent kernel's DYNK sums run over.  K_KEPT: kept[e] limits the sum over k instead
//         (weight gradients).
// scatter: NULL, or row p of expert e goes to the absolute row scatter[e R + p] of C.
// EPI: 0 plain, 1 relu, 2 zero every element whose `mask` element (same index as C) is <= 0, 3 plain with an
// fp32 result, "expert" e summing the k from e K on, up to k_total in all (row-of-k operands).
//
// The k order of a sum is the persistent kernel's, so a layer gets the same bits from either.
//
// Bound: the copies of a step (24 KB for 2 x 128 x 256 x 32 flop, a third more per flop than 256 x 256
// tiles) and the power they draw; 0.95 PFLOP/s on shapes of whole tiles where the persistent kernel
// reaches 1.07.  Layer of 5 x 700 tokens, M 768, H 3072, 24 experts of 295 positions: 299 us with the
// kernel it replaced (256 x 256 tiles through registers, one block per unit, every position
// multiplied), 146 us with this one, 145 us over the occupied rows only.  Few tiles: what a unit fetches,
// about 50 bytes per ns (neither more stages nor fragment reads moved under the MFMAs changed the time),
// hence the smaller tiles; sides measured at gemm_form.
// ----------------------------------------------------------------------------
static __device__ const u32x4_t edge_zero_line = {0u, 0u, 0u, 0u};

template <int BM, int BN, int BK, int ST>
struct EdgeSmem {
  static constexpr int kAStage = BM * BK * 2, kBStage = BN * BK * 2;
  static constexpr int kStage = kAStage + kBStage;
  static constexpr size_t kBytes = (size_t)ST * kStage;
};

// Position of the 16-byte chunks of row k of a row-of-k stage: chunk c sits at c ^ edge_swizzle(k).  The
// transposing read of a half-wavefront takes 64 bytes of four consecutive rows; rows of 64 columns are half
// the banks long, so two of them share a line of banks.
template <int COLS>
__device__ __forceinline__ constexpr int edge_swizzle(int k) {
  return COLS == 64 ? 4 * ((k >> 1) & 1) : 4 * (k & 3);
}

// The arguments of a product, of one launch or of one of the two of a pair (below).
struct EdgeArgs {
  const bf16_t *A, *B;
  bf16_t* C;
  const bf16_t* mask;
  int R, N, K, tiles_m, tiles_n, nblk;
  const int32_t *gather, *kept;
  int row_pad;
  const int32_t* scatter;
  int k_total;
};
// EPI of the products of a pair: decided by their arguments
constexpr int kEpiMaskIfAny = 6;       // 2 with a mask, else 0
constexpr int kEpiRangesIfAny = 7;     // 3 with a k_total, else 0; kept is K_KEPT's

template <int BM, int BN, int BK, int ST, int EPI, bool A_MNC, bool B_KC, bool K_KEPT>
__device__ __forceinline__ void edge_tile(const EdgeArgs& arg, const int logical) {
  const bf16_t *const __restrict__ A = arg.A, *const __restrict__ B = arg.B, *const __restrict__ mask = arg.mask;
  bf16_t* const __restrict__ Cout = arg.C;
  const int R = arg.R, N = arg.N, K = arg.K, tiles_m = arg.tiles_m, tiles_n = arg.tiles_n, row_pad = arg.row_pad;
  const int32_t *const __restrict__ gather = arg.gather, *const __restrict__ kept = arg.kept, *const __restrict__ scatter = arg.scatter;
  const int k_total = arg.k_total;
  const bool masked = EPI == 2 || (EPI == kEpiMaskIfAny && mask != nullptr);
  const bool ranges = EPI == 3 || (EPI == kEpiRangesIfAny && k_total != 0);
  const bool k_kept = K_KEPT || (EPI == kEpiRangesIfAny && kept != nullptr);
  constexpr bool MASKS = EPI == 2 || EPI == kEpiMaskIfAny, RANGES = EPI == 3 || EPI == kEpiRangesIfAny;
  static_assert(EPI != 3 || (A_MNC && !B_KC && !K_KEPT), "ranges of k: of row-of-k operands");
  using SM = EdgeSmem<BM, BN, BK, ST>;
  constexpr int TM = BM / 64, TN = BN / 64;
  constexpr int WN = BN / 2;                                   // columns of a wavefront tile
  constexpr int AC = BM * BK / 2048, BC = BN * BK / 2048;      // copies per wavefront and step
  constexpr int KCH = BK / 8, KRPC = 64 / KCH;                 // K-contiguous rows: chunks, rows per copy
  auto kc_swizzle = [](int row) { return BK == 64 ? (row >> 1) & 7 : (row >> 2) & 3; };
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  typedef unsigned char __attribute__((address_space(3))) * lds_ptr;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_ptr)smem_raw);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * (BM / 2), wn0 = (wave & 1) * WN;

  // Neighbouring tiles on one XCD; inside an expert bands of 8 row tiles, row tile fastest, so
  // that the tiles an XCD works on at a time share row and column panels in its L2.
  const int per_e = tiles_m * tiles_n;
  const int e = logical / per_e;
  const int t = logical - e * per_e;
  constexpr int kBand = 8;
  const int band = t / (kBand * tiles_n), rem = t - band * kBand * tiles_n;
  const int left = tiles_m - band * kBand, brows = left < kBand ? left : kBand;
  const int ct = rem / brows, rt = band * kBand + (rem - ct * brows);
  const int m0 = rt * BM, n0 = ct * BN;
  int rows = R, rows_out = R;                                  // rows of A that count, of C that are stored
  if (kept != nullptr && !k_kept) {
    rows = kept[e];
    rows_out = (rows + row_pad) & ~row_pad;
    rows_out = rows_out < R ? rows_out : R;
  }
  if (m0 >= rows_out) return;                                  // block-uniform
  int KE = k_kept ? kept[e] : K;                               // length of the sum
  if (ranges) KE = k_total - e * K < K ? k_total - e * K : K;
  const int KT = (KE + BK - 1) / BK;

  // Per-lane source addresses of the copies and their advance per K step (0 for a lane that reads
  // the zero line).  k_of: the lane's first k inside a step.
  const uint64_t zline = (uint64_t)(uintptr_t)&edge_zero_line;
  uint64_t a_addr[AC], b_addr[BC];
  uint32_t a_inc[AC], b_inc[BC];
  constexpr int ACH = BM / 8, ARPC = 64 / ACH, BCH = BN / 8, BRPC = 64 / BCH;   // row-of-k operands
#pragma unroll
  for (int q = 0; q < AC; ++q) {
    const int c = wave * AC + q;
    bool ok;
    const bf16_t* src;
    if (A_MNC) {                                               // 512 / BM k rows of BM / 8 chunks per copy
      const int kr = ARPC * c + lane / ACH, col = m0 + 8 * ((lane % ACH) ^ edge_swizzle<BM>(kr));
      ok = col < R && kr < KE;
      src = A + ((size_t)e * K + kr) * R + col;
    } else {
      const int row = KRPC * c + lane / KCH, ch = (lane % KCH) ^ kc_swizzle(row);
      ok = m0 + row < rows && 8 * ch < KE;
      long long arow = (long long)e * R + m0 + row;
      if (gather != nullptr) {
        const int tok = ok ? gather[arow] : -1;
        ok = tok >= 0;
        arow = tok;
      }
      src = A + arow * K + 8 * ch;
    }
    a_addr[q] = ok ? (uint64_t)(uintptr_t)src : zline;
    a_inc[q] = ok ? (A_MNC ? (uint32_t)R * BK * 2 : BK * 2) : 0u;
  }
#pragma unroll
  for (int q = 0; q < BC; ++q) {
    const int c = wave * BC + q;
    bool ok;
    const bf16_t* src;
    if (B_KC) {
      const int row = KRPC * c + lane / KCH, ch = (lane % KCH) ^ kc_swizzle(row);
      ok = n0 + row < N && 8 * ch < KE;
      src = B + ((size_t)e * N + n0 + row) * K + 8 * ch;
    } else {
      const int kr = BRPC * c + lane / BCH, col = n0 + 8 * ((lane % BCH) ^ edge_swizzle<BN>(kr));
      ok = col < N && kr < KE;
      src = B + ((size_t)e * K + kr) * N + col;
    }
    b_addr[q] = ok ? (uint64_t)(uintptr_t)src : zline;
    b_inc[q] = ok ? (B_KC ? BK * 2 : (uint32_t)N * BK * 2) : 0u;
  }
#define MOE_EDGE_COPY(LDS_U32, ADDR_U64)                                                     \
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"            \
               :: "s"(LDS_U32), "v"(ADDR_U64) : "memory")
  // start the copies of step `p` (the next one in order) and move the addresses on; lanes whose
  // k is past the end in the last step go to the zero line
  auto start_step = [&](int p, int stage) {
    if (p > 0) {
#pragma unroll
      for (int q = 0; q < AC; ++q) a_addr[q] += a_inc[q];
#pragma unroll
      for (int q = 0; q < BC; ++q) b_addr[q] += b_inc[q];
      const int kl = KE - p * BK;                              // k left, this step's included
      if (kl < BK) {                                           // block-uniform, last step only
#pragma unroll
        for (int q = 0; q < AC; ++q) {
          const int c = wave * AC + q;
          const int k = A_MNC ? ARPC * c + lane / ACH : 8 * ((lane % KCH) ^ kc_swizzle(KRPC * c + lane / KCH));
          if (k >= kl) a_addr[q] = zline;
        }
#pragma unroll
        for (int q = 0; q < BC; ++q) {
          const int c = wave * BC + q;
          const int k = B_KC ? 8 * ((lane % KCH) ^ kc_swizzle(KRPC * c + lane / KCH)) : BRPC * c + lane / BCH;
          if (k >= kl) b_addr[q] = zline;
        }
      }
    }
    const uint32_t la = lds0 + stage * SM::kStage + wave * (AC * 1024);
    const uint32_t lb = lds0 + stage * SM::kStage + SM::kAStage + wave * (BC * 1024);
#pragma unroll
    for (int q = 0; q < AC; ++q) MOE_EDGE_COPY(la + q * 1024, a_addr[q]);
#pragma unroll
    for (int q = 0; q < BC; ++q) MOE_EDGE_COPY(lb + q * 1024, b_addr[q]);
  };

  // fragment read offsets, as in the persistent kernel (row pitch of a row-of-k stage: 2 x rows)
  const int ar = lane & 31;
  const int p16 = lane & 15, bb = lane >> 4;
  const int bk = 8 * (bb >> 1) + (p16 >> 2);
  // K-contiguous: per 16 k of a step, row-of-k: per 32-row tile
  constexpr int KK = BK / 16;
  uint32_t a_rd[A_MNC ? TM : KK], b_rd[B_KC ? KK : TN];
  auto kc_rd = [&](int w0, int kk) { return (uint32_t)((w0 + ar) * (BK * 2) + ((2 * kk + (lane >> 5)) ^ kc_swizzle(ar)) * 16); };
#pragma unroll
  for (int j = 0; j < (A_MNC ? TM : KK); ++j) {
    const int ca = (wm0 >> 3) + 4 * j + 2 * (bb & 1) + ((p16 & 3) >> 1);
    a_rd[j] = A_MNC ? (uint32_t)(bk * (BM * 2) + ((ca ^ edge_swizzle<BM>(bk)) * 16) + (p16 & 1) * 8) : kc_rd(wm0, j);
  }
#pragma unroll
  for (int j = 0; j < (B_KC ? KK : TN); ++j) {
    const int cb = (wn0 >> 3) + 4 * j + 2 * (bb & 1) + ((p16 & 3) >> 1);
    b_rd[j] = SM::kAStage + (B_KC ? kc_rd(wn0, j)
                                  : (uint32_t)(bk * (BN * 2) + ((cb ^ edge_swizzle<BN>(bk)) * 16) + (p16 & 1) * 8));
  }
  typedef s16x4_t __attribute__((address_space(3))) * lds_s16x4_ptr;
  typedef bf16x8_t __attribute__((address_space(3))) * lds_bf16x8_ptr;
  auto read_kc = [&](uint32_t stage_base, uint32_t rd, int i) {
    return *(lds_bf16x8_ptr)(uintptr_t)(stage_base + rd + i * 32 * (BK * 2));
  };
  auto read_mnc = [&](uint32_t stage_base, uint32_t rd, int kk, int pitch) {
    const uint32_t p = stage_base + rd + kk * 16 * pitch;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)p);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(p + 4 * pitch));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  int p = 0, pstage = 0;
#pragma unroll 1
  for (; p < ST - 1 && p < KT; ++p) {
    start_step(p, pstage);
    ++pstage;
  }
  int stage = 0;
  // A step: the fragments of its first kAhead pieces of 16 k are asked for at once and each product is followed by the fetch
  // of the piece kAhead on, so that a step waits for LDS once and not once per piece: it is this chain of waits that bounds
  // tiles alone on their unit (48 tiles of K 3072, 0.24 us a step of 64 k, of which 0.05 are products).
  // Where three stages or more leave them time the copies of a later step are started under that wait.  They go first with two
  // stages, in the forward products, whose weights may come from memory (64 x 128 deep of 40 us and more lost 3 %), and in the
  // dense layers' 128 x 128 weight gradients, whose long sums lost 5 %.
  // Over the products of 60 drawn training and encoder steps, sums of us before / after: 64 x 64 deep 1129 / 1062, pairs of
  // 64 x 64 tiles 1501 / 1389, weight gradients of 64 x 64 tiles 269 / 245, of 128 x 128 of kept rows 411 / 392.
  // As before: 128 x 256 tiles (two blocks of 128 accumulators fill the unit) and the forward products on 128 x 128 tiles or in
  // two stages: 64 tokens through 32 experts of M 1024, H 8192, whose weights stream, took 200 us with it instead of 194.
  constexpr int kAhead = BN == 256 || (!A_MNC && !B_KC && (ST == 2 || BM == 128)) ? 0 : BM == 128 && KK > 2 ? 2 : KK;
  constexpr bool kReadFirst = ST > 2 && (A_MNC ? BM == 64 || K_KEPT || EPI == kEpiRangesIfAny : B_KC);
  bf16x8_t fa[KK][TM], fb[KK][TN];
  auto fetch = [&](uint32_t sb, int kk) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[kk][i] = A_MNC ? read_mnc(sb, a_rd[i], kk, BM * 2) : read_kc(sb, a_rd[kk], i);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[kk][j] = B_KC ? read_kc(sb, b_rd[kk], j) : read_mnc(sb, b_rd[j], kk, BN * 2);
  };
  auto begin = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < kAhead; ++kk) fetch(lds0 + stage * SM::kStage, kk);
    if (kAhead > 0) __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&]() __attribute__((always_inline)) {
    const uint32_t sb = lds0 + stage * SM::kStage;
    stage = stage + 1 == ST ? 0 : stage + 1;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if constexpr (kAhead == 0) {                             // (by itself: fa and fb in their place cost address arithmetic)
        bf16x8_t ga[TM], gb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) ga[i] = A_MNC ? read_mnc(sb, a_rd[i], kk, BM * 2) : read_kc(sb, a_rd[kk], i);
#pragma unroll
        for (int j = 0; j < TN; ++j) gb[j] = B_KC ? read_kc(sb, b_rd[kk], j) : read_mnc(sb, b_rd[j], kk, BN * 2);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gb[j], ga[i], acc[i][j], 0, 0, 0);
        continue;
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[kk][j], fa[kk][i], acc[i][j], 0, 0, 0);
      if (kk + kAhead < KK) {
        fetch(sb, kk + kAhead);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // The last step of a masked tile stands by itself (k is never empty there): a loop that the masks' loads may have
  // preceded waits for them in every turn.
  const int loop_steps = MASKS ? KT - 1 : KT;
  for (int g = 0; g < loop_steps; ++g) {
    // own copies of step g landed (the steps started after it may still fly), then everybody's; the
    // stage of step g - 1 is free after the barrier
    wait_copies<AC + BC, ST - 2>(KT - 1 - g);
    __syncthreads();
    if (kReadFirst) begin();
    if (p < KT) {
      start_step(p, pstage);
      pstage = pstage + 1 == ST ? 0 : pstage + 1;
      ++p;
    }
    if (!kReadFirst) begin();
    multiply();
  }
  constexpr int CH = WN / 8, RPP = 64 / CH;                    // chunks per row of the wavefront tile, rows per store
  u32x4_t mk[MASKS ? TM : 1][MASKS ? 32 / RPP : 1];
  if constexpr (MASKS) {
    wait_copies<0, 0>(0);
    __syncthreads();
    begin();
    if (masked) {
      // The masks of a tile, all at once and under the last step: fetched store by store, they wait for one another
      // (training step of 76 experts of 309 rows, M 512, H 4096 1072 / 1058 us, of 12 of 669, M 520, H 2056 266.0 / 263.8).
      // Those of rows and columns that are not stored come from the last ones.
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int ps = 0; ps < 32 / RPP; ++ps) {
          const int row = m0 + wm0 + 32 * i + RPP * ps + lane / CH, col = n0 + wn0 + 8 * (lane % CH);
          mk[i][ps] = *reinterpret_cast<const u32x4_t*>(mask + ((size_t)e * R + (row < rows_out ? row : rows_out - 1)) * N +
                                                        (col < N ? col : N - 8));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    multiply();
  }
  if (RANGES && ranges) {                                      // a lane owns four consecutive columns of a row
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    float* const Cf = reinterpret_cast<float*>(Cout) + (size_t)e * R * N;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = m0 + wm0 + 32 * i + (lane & 31);
      if (row >= R) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = n0 + wn0 + 32 * j + 8 * q + 4 * (lane >> 5);
          if (col < N)
            *reinterpret_cast<f32x4_t*>(Cf + (size_t)row * N + col) =
                f32x4_t{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        }
    }
    return;
  }
  __syncthreads();                                             // the stages are free

  // acc[i][j][4 q + r] = C[32 i + r32][32 j + 8 q + 4 h + r] of the wavefront tile: 32 rows at a time
  // through the wavefront's own LDS into whole-row 16-byte stores.  Chunk c of row r sits at
  // position c ^ (r % chunks), its 8-byte halves swapped in every other group of rows.
  const uint32_t st_base = lds0 + wave * (32 * WN * 2);
  const int r32 = lane & 31, hh = lane >> 5;
  const uint32_t st_wr = st_base + r32 * (WN * 2) + 8 * (hh ^ ((r32 / CH) & 1));
  typedef u32x2_t __attribute__((address_space(3))) * lds_u2_ptr;
  typedef u32x4_t __attribute__((address_space(3))) * lds_u4_ptr;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t lo = pack_bf16x2(acc[i][j][4 * q], acc[i][j][4 * q + 1]);
        uint32_t hi = pack_bf16x2(acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        if (EPI == 1) { lo = relu_bf16x2(lo); hi = relu_bf16x2(hi); }
        *(lds_u2_ptr)(uintptr_t)(st_wr + (((4 * j + q) ^ (r32 & (CH - 1))) * 16)) = u32x2_t{lo, hi};
      }
#pragma unroll
    for (int ps = 0; ps < 32 / RPP; ++ps) {
      const int rr = RPP * ps + lane / CH, c = lane % CH;
      u32x4_t d = *(lds_u4_ptr)(uintptr_t)(st_base + rr * (WN * 2) + ((c ^ (rr & (CH - 1))) * 16));
      if ((rr / CH) & 1) d = u32x4_t{d[2], d[3], d[0], d[1]};
      const int row = m0 + wm0 + 32 * i + rr, col = n0 + wn0 + 8 * c;
      if (row < rows_out && col < N) {
        const size_t o = ((size_t)e * R + row) * N + col;
        if (MASKS && masked) {
#pragma unroll
          for (int w = 0; w < 4; ++w)          // a bf16 is positive iff its bits, as an integer, are
            d[w] &= ((int16_t)(mk[i][ps][w] & 0xffffu) > 0 ? 0xffffu : 0u) |
                    ((int16_t)(mk[i][ps][w] >> 16) > 0 ? 0xffff0000u : 0u);
        }
        if (scatter != nullptr)
          *reinterpret_cast<u32x4_t*>(Cout + (size_t)scatter[(size_t)e * R + row] * N + col) = d;
        else
          *reinterpret_cast<u32x4_t*>(Cout + o) = d;
      }
    }
  }
#undef MOE_EDGE_COPY
}

template <int BM, int BN> constexpr int kEdgeBlocks = BN == 256 ? 2 : BM == 128 ? 3 : 4;      // per compute unit
template <int BM, int BN, int BK, int ST, int EPI, bool A_MNC, bool B_KC, bool K_KEPT>
__global__ __launch_bounds__(256, (kEdgeBlocks<BM, BN>)) void expert_gemm_bf16_edge_kernel(EdgeArgs arg) {
  edge_tile<BM, BN, BK, ST, EPI, A_MNC, B_KC, K_KEPT>(arg, xcd_remap(blockIdx.x, arg.nblk));
}

// The data gradient and the weight gradient of one linear layer in one launch: both read the layer's upstream gradient,
// neither needs the other (pair_ok below says when).  The arguments decide what the forms of a launch of its own know when
// they are compiled (masks, ranges, kept rows), which keeps them at nine kernels; a tile does the same arithmetic either way.
template <int BMD, int BND, int STD, int BMW, int BNW, int STW>
__global__ __launch_bounds__(256, (kEdgeBlocks<BMD, BND> < kEdgeBlocks<BMW, BNW> ? kEdgeBlocks<BMD, BND> : kEdgeBlocks<BMW, BNW>))
void expert_gemm_bf16_pair_kernel(EdgeArgs data, EdgeArgs weight) {
  const int id = blockIdx.x;
  if (id < data.nblk) edge_tile<BMD, BND, 64, STD, kEpiMaskIfAny, false, true, false>(data, xcd_remap(id, data.nblk));
  else edge_tile<BMW, BNW, 32, STW, kEpiRangesIfAny, true, false, false>(weight, xcd_remap(id - data.nblk, weight.nblk));
}

// LDS limit of one instantiation of the persistent kernel on the current device (all of the
// 160 KB when the size depends on the number of experts)
template <int ST, int EPI, bool GATHER, bool A_MNC = false, bool B_KC = false, bool PACKED = false,
          bool SCATTER = false, bool DYNK = false, bool ROWS = false>
int prepare_dma() {
  static LdsLimitOnce once;
  constexpr int kFixed = (int)DmaSmem<ST>::kBytes + (GATHER ? 1024 : 0) + (EPI == 5 ? 8192 : 0);
  return ensure_lds_limit(
      once, reinterpret_cast<const void*>(
                expert_gemm_bf16_dma_kernel<ST, EPI, GATHER, A_MNC, B_KC, PACKED, SCATTER, DYNK, ROWS>),
      PACKED || DYNK ? 160 * 1024 : kFixed);
}

template <int ST, int EPI, bool GATHER, bool A_MNC, bool B_KC, bool PACKED, bool SCATTER, bool DYNK, bool ROWS>
int launch_bf16_dma_rows(const bf16_t* A, const bf16_t* B, bf16_t* Cout, int E, int R, int N, int K,
                         const int32_t* src_token, const bf16_t* zero_row, hipStream_t st,
                         const bf16_t* mask, unsigned char* signbits, const int32_t* kept) {
  using SM = DmaSmem<ST>;
  static_assert(!(GATHER && EPI == 5), "the two users of the spare LDS exclude each other");
  // PACKED / DYNK: 2 E + 1 more integers of LDS (row counts and running tile counts of the experts)
  const size_t kLds = SM::kBytes + (GATHER ? 4 * 64 * sizeof(int32_t) : 0) + (EPI == 5 ? 8192 : 0) +
                      (PACKED || DYNK ? align_up(((size_t)2 * E + 1) * sizeof(int32_t), 16) : 0);
  if (kLds > 160 * 1024) return MOE_EUNSUPPORTED;
  if ((PACKED || DYNK) && kept == nullptr) return MOE_EINVAL;
  auto kern = expert_gemm_bf16_dma_kernel<ST, EPI, GATHER, A_MNC, B_KC, PACKED, SCATTER, DYNK, ROWS>;
  int cus = 0;
  if (prepare_dma<ST, EPI, GATHER, A_MNC, B_KC, PACKED, SCATTER, DYNK, ROWS>() != MOE_OK ||
      compute_units(&cus) != MOE_OK)
    return MOE_EHIP;
  const int tiles_m = (R + 255) / 256, tiles_n = N / 256;
  const long long ntiles = (long long)E * tiles_m * tiles_n;
  if (ntiles > 0x7fffffffLL) return MOE_EUNSUPPORTED;
  const unsigned grid = (unsigned)(ntiles < cus ? ntiles : cus);   // one block per CU (LDS-bound)
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), kLds, st, A, B, Cout, R, N, K, tiles_m,
                     tiles_n, (int)ntiles, src_token, zero_row, mask, signbits,
                     kept, E);
  return check_launch();
}

template <int ST, int EPI, bool GATHER, bool A_MNC = false, bool B_KC = false, bool PACKED = false,
          bool SCATTER = false, bool DYNK = false>
int launch_bf16_dma(const bf16_t* A, const bf16_t* B, bf16_t* Cout, int E, int R, int N, int K,
                    const int32_t* src_token, const bf16_t* zero_row, hipStream_t st,
                    const bf16_t* mask = nullptr, unsigned char* signbits = nullptr,
                    const int32_t* kept = nullptr) {
  if (R % 256 != 0) {
    if constexpr (!A_MNC && !SCATTER && !DYNK && EPI != 3)
      return launch_bf16_dma_rows<ST, EPI, GATHER, A_MNC, B_KC, PACKED, SCATTER, DYNK, true>(
          A, B, Cout, E, R, N, K, src_token, zero_row, st, mask, signbits, kept);
    return MOE_EUNSUPPORTED;
  }
  return launch_bf16_dma_rows<ST, EPI, GATHER, A_MNC, B_KC, PACKED, SCATTER, DYNK, false>(
      A, B, Cout, E, R, N, K, src_token, zero_row, st, mask, signbits, kept);
}

// shapes the persistent 256x256 kernel takes (its per-lane byte offsets are 32-bit); rows of a K-contiguous A
// may be any number
inline bool dma_columns_ok(int R, int N, int K) {
  const long long big = R > N ? (R > K ? R : K) : (N > K ? N : K);
  return N % 256 == 0 && K % 32 == 0 && K >= 128 && 256 * big * 2 < (1LL << 31);
}
inline bool dma_shape_ok(int R, int N, int K) {
  const long long big = R > N ? (R > K ? R : K) : (N > K ? N : K);
  return R % 256 == 0 && N % 256 == 0 && K % 32 == 0 && 256 * big * 2 < (1LL << 31);
}

// Which kernel multiplies C [E,R,N]: the persistent one on 256 x 256 tiles (shapes it takes), or the
// edge kernel in one of its forms.  All have the same k order, so the choice changes no bit.
//
// Operands that are K-contiguous (both in the data gradients, A in the forward products) come in pieces of
// a row of one step: 64-wide steps fetch whole 128-byte lines where 32-wide ones fetch halves.  They cost
// twice the LDS per stage, so 128 x 256 tiles, which would be left alone on a unit, stay at 32 and the others
// have a form of fewer stages for shapes of many tiles and a deep one for tiles that are alone on their
// unit, or where the weights stream from memory.  (us of one product, 32-wide / 64-wide steps, tiles 128 x 128:
// dbuf of 10 experts of 2852 rows, M 1024, H 8192 617 / 506, of 52 of 880, M 664, H 1384 174 / 150; tiles 64 x 64,
// dbuf of 10 of 81, M 1024, H 4096 43.6 / 33.2, of 4 of 64 29.3 / 21.8.)  The weight gradients' operands are both
// row-of-k, whose pieces are whole lines anyway, and their sums often short: 32 wide.
enum GemmForm { kPersistent, kEdge128x256, kEdge128x128, kEdge128x128Deep, kEdge64x128, kEdge64x128Deep, kEdge64x64,
                kEdge64x64Deep };
enum GemmLayout { kLayoutForward, kLayoutDataGrad, kLayoutWeightGrad, kLayoutMaskedDataGrad };

// The rule compares what the fullest compute unit needs: 32 k of the tiles that share it (ns; up to as many as
// fit), the ends of the tiles (us; `more` of it for every further round), and the time in which the form streams the
// weights from memory (TB/s).  dh, whose sums are short and whose results are long, is often bound by its rows and
// masks instead, so all its bytes count there (positions are 0.85 full in the mean; the persistent kernel reads the masks
// as bits).
// Fitted to the choices among the forms for the products of 430 shapes (E 1 to 192, R 1 to 16384, M 130 to 1024, H 260 to
// 8192; two states of operands in turn).  On 110 others its choice was 3.0 % from the best form in the mean; with the
// constants before, which took the persistent kernel too often where N or K is a few hundred and 128 x 256 tiles for long
// sums of few tiles, 3.9 %.
//   us, 64x64 deep / 64x64 / 64x128 deep / 64x128 / 128x128 deep / 128x128 / 128x256 / persistent:
//   out  E 16  R 15   M 1024 H 4096    54 /   47 /   55 /   66 /   57 /   71 /   74 /   88
//   out  E 24  R 295  M 768  H 3072    79 /   77 /   70 /   61 /   70 /   58 /   69 /  100
//   out  E 100 R 290  M 256  H 512     24 /   22 /   21 /   24 /   25 /   24 /   23 /   36
//   h    E 81  R 456  M 512  H 1024   112 /   96 /   87 /   82 /   94 /   75 /   64 /   78
//   h    E 32  R 2048 M 1024 H 8192  2096 / 1740 / 1607 / 1402 / 1804 / 1335 / 1160 / 1147
//   dbuf E 81  R 456  M 512  H 1024    96 /   90 /   79 /   77 /   81 /   69 /   69 /   88
//   dh   E 5   R 612  M 512  H 1024    13 /   14 /   11 /   11 /   14 /   14 /   20 /   21
//   dh   E 51  R 862  M 512  H 4096   545 /  454 /  455 /  402 /  537 /  392 /  370 /  291
struct FormCost { int bm, bn, bk, res; double step[4], ends, more, stream; };
const FormCost* form_costs(GemmLayout layout) {
  static const FormCost forward[] = {{256, 256, 32, 1, {840}, 7.5, 1, 6.0},             {128, 256, 32, 2, {595, 980}, 8.3, 0.5, 6.0},
                                     {128, 128, 64, 2, {360, 605}, 7, 0.5, 5.6},        {128, 128, 64, 1, {280}, 6.1, 0.5, 5.7},
                                     {64, 128, 64, 3, {250, 288, 555}, 4.9, 0.47, 4.6}, {64, 128, 64, 2, {227, 405}, 4.1, 0.48, 4.6},
                                     {64, 64, 64, 3, {168, 242, 340}, 4.6, 0.37, 4.8},  {64, 64, 64, 2, {119, 230}, 4, 0.5, 4.3}};
  static const FormCost datagrad[] = {{256, 256, 32, 1, {930}, 6.5, 1, 5.5},          {128, 256, 32, 2, {640, 1110}, 8.6, 0.5, 5.0},
                                      {128, 128, 64, 2, {283, 500}, 6.2, 0.5, 4.1},   {128, 128, 64, 1, {280}, 5.8, 0.5, 5.2},
                                      {64, 128, 64, 3, {265, 322, 565}, 4, 0.5, 3.9}, {64, 128, 64, 2, {190, 393}, 3.7, 0.5, 5.1},
                                      {64, 64, 64, 3, {152, 242, 330}, 3.4, 0.5, 5.1}, {64, 64, 64, 2, {123, 268}, 3.6, 0.5, 5.15}};
  static const FormCost masked[] = {{256, 256, 32, 1, {767}, 6.9, 0.82, 5.5},          {128, 256, 32, 2, {580, 1245}, 10.7, 0.5, 5.2},
                                    {128, 128, 64, 2, {289, 590}, 6.7, 0.5, 6.7},      {128, 128, 64, 1, {235}, 7.1, 0.5, 5.2},
                                    {64, 128, 64, 3, {265, 268, 543}, 4.1, 0.44, 6.3}, {64, 128, 64, 2, {213, 390}, 4.6, 0.5, 6.5},
                                    {64, 64, 64, 3, {152, 242, 300}, 3.5, 0.43, 6.5},  {64, 64, 64, 2, {142, 242}, 3.9, 0.5, 6.0}};
  static const FormCost weightgrad[] = {{256, 256, 32, 1, {840}, 12, 0.38, 0},            {128, 256, 32, 2, {480, 950}, 11, 0.3, 0},
                                        {128, 128, 32, 3, {272, 505, 760}, 5.6, 0.5, 0},  {0},
                                        {64, 128, 32, 3, {230, 350, 530}, 4.1, 0.6, 0},   {0},
                                        {64, 64, 32, 4, {162, 220, 320, 395}, 4, 0.5, 0}, {0}};
  switch (layout) {
    case kLayoutForward: return forward;
    case kLayoutDataGrad: return datagrad;
    case kLayoutMaskedDataGrad: return masked;
    default: return weightgrad;
  }
}
// us of a form, 0: not one for this shape (the persistent kernel's shapes are the caller's to check)
double form_time(GemmForm f, int E, int R, int N, int K, GemmLayout layout, int cus) {
  const FormCost* const cost = form_costs(layout);
  const FormCost& c = cost[f];
  if (c.bm == 0) return 0;
  const long long n = (long long)E * ((R + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn), round = (long long)c.res * cus;
  // few tiles: the deep form, many: the other (64 x 128 tiles of any count may be deep, for weights that stream)
  if ((f == kEdge64x64Deep || f == kEdge128x128Deep) && n > round) return 0;
  if ((f == kEdge64x64 || f == kEdge128x128 || f == kEdge64x128) && n <= (long long)cost[f + 1].res * cus) return 0;
  const int steps = (K + c.bk - 1) / c.bk * (c.bk / 32);
  const long long full = n / round, rounds = (n + round - 1) / round;
  const int left = (int)((n - full * round + cus - 1) / cus);
  double part = left > 0 ? c.step[left - 1] : 0.0;
  // (the weight gradients' last round starts while the one before it ends)
  if (layout == kLayoutWeightGrad && full > 0 && left > 0)
    part = 0.5 * (part + (double)(n - full * round) / round * c.step[c.res - 1]);
  double us = 1e-3 * steps * (full * c.step[c.res - 1] + part);
  us += c.ends * (1 + c.more * (double)(rounds - 1));
  if (c.stream > 0) {
    double elems = (double)N * K;
    if (layout == kLayoutMaskedDataGrad) elems += 0.85 * R * ((double)K + (f == kPersistent ? 1.0 : 2.0) * N);
    const double stream = 2e-6 * E * elems / c.stream + 0.5 * c.ends;
    us = stream > us ? stream : us;
  }
  return us;
}
GemmForm gemm_form(bool persistent_ok, int E, int R, int N, int K, GemmLayout layout, int cus, double* time = nullptr) {
  GemmForm form = kEdge128x256;
  double best = 0;
  for (int f = kEdge64x64Deep; f >= (persistent_ok ? kPersistent : kEdge128x256); --f) {
    const double us = form_time((GemmForm)f, E, R, N, K, layout, cus);
    if (us > 0 && (best == 0 || us < best)) { best = us; form = (GemmForm)f; }
  }
  if (time != nullptr) *time = best;
  return form;
}
// h of a training pass over packed rows: the persistent kernel takes relu' of dh from the bits that only it records
// with h, so the two products are chosen together.  A dh that reads h leaves it in the last-level cache for dwo, unless it
// is too large to stay there: an h that is slower persistent has to be that large, and gain 4 % of both.  A dh that shares its
// launch with dwo (pair_ok, below: small layers) masks by h after all and leaves the bits unread.  us of h / dh / dwo,
// each by its own best form, then h and dh persistent (MB of h at 0.85 full):
//   E 12 R 4352 M 256  H 2048 (182)   80 / 162 /  83    97 /  93 /  91
//   E 51 R 862  M 512  H 4096 (306)  234 / 346 / 198   259 / 265 / 205
//   E 4  R 3376 M 512  H 4096  (94)   72 /  94 /  63    70 /  67 /  66
//   E 10 R 602  M 768  H 6144  (63)   78 /  88 /  64    90 /  85 /  76
//   E 5  R 1048 M 1024 H 4096  (36)   58 /  63 /  45    68 /  66 /  46
bool persistent_h(int E, int R, int H, int M, int cus) {
  double h = 0, dh = 0;
  gemm_form(false, E, R, H, M, kLayoutForward, cus, &h);
  gemm_form(false, E, R, H, M, kLayoutMaskedDataGrad, cus, &dh);
  const double hp = form_time(kPersistent, E, R, H, M, kLayoutForward, cus);
  const double dhp = form_time(kPersistent, E, R, H, M, kLayoutMaskedDataGrad, cus);
  const double both = hp + (dhp < dh ? dhp : dh);
  return hp < h ? both < h + dh : both < 0.96 * (h + dh) && 0.85 * 2 * E * R * H > 80e6;
}
// the form of this shape on a device of `cus` units, or the current one; k_kept: the sum over k runs over packed rows, of
// which the persistent kernel takes whole 256-row tiles
GemmForm form_of(int E, int R, int N, int K, GemmLayout layout, bool k_kept, int cus, double* us = nullptr) {
  const bool persistent = dma_shape_ok(R, N, K) || (layout != kLayoutWeightGrad && dma_columns_ok(R, N, K));
  return gemm_form(persistent && (!k_kept || K % 256 == 0), E, R, N, K, layout, cus, us);
}
int choose_form(int E, int R, int N, int K, GemmLayout layout, GemmForm* form, bool k_kept = false) {
  int cus = 0;
  if (compute_units(&cus) != MOE_OK) return MOE_EHIP;
  *form = form_of(E, R, N, K, layout, k_kept, cus);
  return MOE_OK;
}
// h and dh of a training pass over packed rows
void train_forms_of(const moe_config& c, int cus, GemmForm* h, GemmForm* dh, double* dh_us = nullptr) {
  const int R = c.G * c.C;
  const bool bits = (dma_shape_ok(R, c.H, c.M) || dma_columns_ok(R, c.H, c.M)) && persistent_h(c.E, R, c.H, c.M, cus);
  *h = bits ? kPersistent : gemm_form(false, c.E, R, c.H, c.M, kLayoutForward, cus);
  *dh = gemm_form(bits, c.E, R, c.H, c.M, kLayoutMaskedDataGrad, cus, dh_us);
}
int choose_train_forms(const moe_config& c, GemmForm* h, GemmForm* dh) {
  int cus = 0;
  if (compute_units(&cus) != MOE_OK) return MOE_EHIP;
  train_forms_of(c, cus, h, dh);
  return MOE_OK;
}

template <int BM, int BN, int BK, int ST, int EPI, bool A_MNC, bool B_KC, bool K_KEPT>
int prepare_edge() {
  static LdsLimitOnce once;
  return ensure_lds_limit(
      once, reinterpret_cast<const void*>(expert_gemm_bf16_edge_kernel<BM, BN, BK, ST, EPI, A_MNC, B_KC, K_KEPT>),
      (int)EdgeSmem<BM, BN, BK, ST>::kBytes);
}

inline bool edge_args(EdgeArgs* out, int BM, int BN, const GemmArgs& a, int E, int R, int N, int K, int k_total) {
  const int tiles_m = (R + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  const long long nblk = (long long)E * tiles_m * tiles_n;
  if (nblk > 0x7fffffffLL) return false;
  *out = EdgeArgs{static_cast<const bf16_t*>(a.A), static_cast<const bf16_t*>(a.B), static_cast<bf16_t*>(a.C),
                  static_cast<const bf16_t*>(a.mask), R, N, K, tiles_m, tiles_n, (int)nblk, a.gather, a.kept, a.row_pad,
                  a.scatter, k_total};
  return true;
}
template <int BM, int BN, int BK, int ST, int EPI, bool A_MNC, bool B_KC, bool K_KEPT>
int launch_edge(const GemmArgs& a, int E, int R, int N, int K, hipStream_t st, int k_total = 0) {
  if (prepare_edge<BM, BN, BK, ST, EPI, A_MNC, B_KC, K_KEPT>() != MOE_OK) return MOE_EHIP;
  constexpr size_t kLds = EdgeSmem<BM, BN, BK, ST>::kBytes;
  EdgeArgs arg;
  if (!edge_args(&arg, BM, BN, a, E, R, N, K, k_total) || (K_KEPT && a.kept == nullptr)) return MOE_EUNSUPPORTED;
  hipLaunchKernelGGL((expert_gemm_bf16_edge_kernel<BM, BN, BK, ST, EPI, A_MNC, B_KC, K_KEPT>), dim3((unsigned)arg.nblk),
                     dim3(256), kLds, st, arg);
  return check_launch();
}

// C [E,R,N] for any R, N, K with N % 8 == 0 and the operands' contiguous dimensions % 8 == 0
// (K for a K-contiguous operand, R / N for a row-of-k one)
template <int EPI, bool A_MNC, bool B_KC, bool K_KEPT = false>
int gemm_bf16_edge(GemmForm form, const GemmArgs& a, int E, int R, int N, int K, hipStream_t st, int k_total = 0) {
  if constexpr (A_MNC) {
    switch (form) {
      case kEdge64x64: return launch_edge<64, 64, 32, 5, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st, k_total);
      case kEdge64x128: return launch_edge<64, 128, 32, 4, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st, k_total);
      case kEdge128x128: return launch_edge<128, 128, 32, 3, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st, k_total);
      default: return launch_edge<128, 256, 32, 3, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st, k_total);
    }
  } else {
    switch (form) {
      case kEdge64x64: return launch_edge<64, 64, 64, 3, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st);
      case kEdge64x64Deep: return launch_edge<64, 64, 64, 4, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st);
      case kEdge64x128: return launch_edge<64, 128, 64, 2, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st);
      case kEdge64x128Deep: return launch_edge<64, 128, 64, 3, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st);
      case kEdge128x128: return launch_edge<128, 128, 64, 2, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st);
      case kEdge128x128Deep: return launch_edge<128, 128, 64, 3, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st);
      default: return launch_edge<128, 256, 32, 3, EPI, A_MNC, B_KC, K_KEPT>(a, E, R, N, K, st);
    }
  }
}

// One product of a pair: its operands and sizes as for gemm_bf16_edge, its form and the rule's time (us).
struct PairProduct {
  GemmArgs a;
  int E, R, N, K;
  GemmForm form;
  double us;
  int k_total = 0;
};
template <int BMD, int BND, int STD, int BMW, int BNW, int STW>
int prepare_pair() {
  static LdsLimitOnce once;
  constexpr size_t d = EdgeSmem<BMD, BND, 64, STD>::kBytes, w = EdgeSmem<BMW, BNW, 32, STW>::kBytes;
  return ensure_lds_limit(once, reinterpret_cast<const void*>(expert_gemm_bf16_pair_kernel<BMD, BND, STD, BMW, BNW, STW>),
                          (int)(d > w ? d : w));
}
template <int BMD, int BND, int STD, int BMW, int BNW, int STW>
int launch_pair_as(const PairProduct& d, const PairProduct& w, hipStream_t st) {
  if (prepare_pair<BMD, BND, STD, BMW, BNW, STW>() != MOE_OK) return MOE_EHIP;
  constexpr size_t kLdsD = EdgeSmem<BMD, BND, 64, STD>::kBytes, kLdsW = EdgeSmem<BMW, BNW, 32, STW>::kBytes;
  EdgeArgs da, wa;
  if (!edge_args(&da, BMD, BND, d.a, d.E, d.R, d.N, d.K, 0) || !edge_args(&wa, BMW, BNW, w.a, w.E, w.R, w.N, w.K, w.k_total) ||
      (long long)da.nblk + wa.nblk > 0x7fffffffLL)
    return MOE_EUNSUPPORTED;
  hipLaunchKernelGGL((expert_gemm_bf16_pair_kernel<BMD, BND, STD, BMW, BNW, STW>), dim3((unsigned)(da.nblk + wa.nblk)), dim3(256),
                     kLdsD > kLdsW ? kLdsD : kLdsW, st, da, wa);
  return check_launch();
}
// as many stages as leave a unit the blocks that its larger tiles would have alone
template <int BMD, int BND>
int launch_pair_weight(const PairProduct& d, const PairProduct& w, hipStream_t st) {
  constexpr int kDeep = BND == 64 ? 4 : 2, kFlat = BND == 64 ? 3 : 2;
  switch (w.form) {
    case kEdge64x64: return launch_pair_as<BMD, BND, kDeep, 64, 64, 5>(d, w, st);
    case kEdge64x128: return launch_pair_as<BMD, BND, kDeep, 64, 128, 4>(d, w, st);
    default: return launch_pair_as<BMD, BND, kFlat, 128, 128, 3>(d, w, st);
  }
}
// Which pairs of gradients share a launch.  A small product leaves units idle at its start and end and its successor waits
// for the last of its tiles; in one launch the second product's tiles fill the units that the first leaves, and one launch
// and its gap go away.  With 160 products of 60 drawn training steps and encoder backward passes (us, two launches / one,
// without the gap): 64 x 64 tiles 13.9 / 8.3, 18.1 / 12.0, 25.5 / 24.5, mixed ones 24.5 / 19.9, 60.5 / 53.8,
// 162 / 147, 128 x 128 tiles 31.1 / 22.4, 57.8 / 52.4, 121 / 101, at worst 64.3 / 69.7.  The line is drawn (kPairMost, both
// products by the rule) under the sizes from which pairs were as often slower as faster, 140 us: both then fill the chip alone.
// The persistent kernel and 128 x 256 tiles take too much of a unit's LDS to share it.  Products that the rule would give to
// them are paired in their best other form unless that looks more than kPairGain slower, which a shared launch is worth
// (us, with such a form / paired, 7 of 90 drawn layers: 69.8 / 62.2, 66.2 / 58.2, 60.0 / 56.6, 49.0 / 44.4, 48.8 / 47.4,
// 42.2 / 35.8, 62.1 / 62.7; at 4 us instead of 12 only one of them was paired).
// What one product writes the other must not read: a caller may pass a gradient's buffer that is also an operand of the
// product that comes first otherwise (wi as dwi: an expert's data gradient; a dense layer's comes second), which one launch
// after the other allows.
bool disjoint(const void* p, size_t pn, const void* q, size_t qn) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
  return p == nullptr || q == nullptr || a + pn <= b || b + qn <= a;
}
bool independent(const PairProduct& writer, const PairProduct& reader) {
  auto bytes = [](long long e, long long r, long long n, size_t elt) { return (size_t)(e * r * n) * elt; };
  const PairProduct &w = writer, &r = reader;
  const size_t out = bytes(w.E, w.R, w.N, w.k_total != 0 ? sizeof(float) : sizeof(bf16_t));
  const long long k = r.k_total != 0 ? r.k_total : (long long)r.E * r.K;        // of all experts or ranges
  return disjoint(w.a.C, out, r.a.A, bytes(k, r.R, 1, sizeof(bf16_t))) &&
         disjoint(w.a.C, out, r.a.B, bytes(k, r.N, 1, sizeof(bf16_t))) &&
         disjoint(w.a.C, out, r.a.mask, bytes(r.E, r.R, r.N, sizeof(bf16_t)));
}
constexpr double kPairMost = 120.0, kPairGain = 12.0;          // us
// sets the forms that the pair runs in; both products' times are for `cus` units
bool pair_ok(PairProduct* d, GemmLayout data, PairProduct* w, int cus) {
  const double alone = d->us + w->us;
  for (PairProduct* p : {d, w})
    if (p->form == kPersistent || p->form == kEdge128x256) {
      p->us = 1e30;
      for (int f = kEdge64x64Deep; f >= kEdge128x128; --f) {
        const double us = form_time((GemmForm)f, p->E, p->R, p->N, p->K, p == d ? data : kLayoutWeightGrad, cus);
        if (us > 0 && us < p->us) { p->us = us; p->form = (GemmForm)f; }
      }
    }
  const double us = d->us + w->us;
  return us < kPairMost && us < alone + kPairGain;
}
// one launch, unless the products are not independent
int launch_pair(const PairProduct& d, const PairProduct& w, hipStream_t st, bool* done) {
  *done = independent(d, w) && independent(w, d);
  if (!*done) return MOE_OK;
  switch (d.form) {
    case kEdge64x64: case kEdge64x64Deep: return launch_pair_weight<64, 64>(d, w, st);
    case kEdge64x128: case kEdge64x128Deep: return launch_pair_weight<64, 128>(d, w, st);
    default: return launch_pair_weight<128, 128>(d, w, st);
  }
}

template <bool RELU>
int gemm_bf16(const bf16_t* A, const bf16_t* B, bf16_t* Cout, int E, int R, int N, int K,
              hipStream_t st) {
  GemmForm form;
  if (choose_form(E, R, N, K, kLayoutForward, &form) != MOE_OK) return MOE_EHIP;
  if (form == kPersistent)
    return launch_bf16_dma<4, RELU ? 1 : 0, false>(A, B, Cout, E, R, N, K, nullptr, nullptr, st);
  return gemm_bf16_edge<RELU ? 1 : 0, false, false>(form, GemmArgs{A, B, Cout}, E, R, N, K, st);
}

}  // namespace

int compute_units(int* cus) {
  static std::atomic<int> cus_of[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MOE_EHIP;
  int n = cus_of[dev].load(std::memory_order_acquire);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
      return MOE_EHIP;
    cus_of[dev].store(n, std::memory_order_release);
  }
  *cus = n;
  return MOE_OK;
}

// Every instantiation the launchers of this file use (a kernel missing from this list is
// still set up by its launcher's first call).
int prepare_expert_gemm() {
  const int rcs[] = {
      // forward
      prepare_dma<4, 0, false, false, false, true, true>(),
      // fp32 results (gate logits and gate gradients)
      prepare_dma<4, 3, false, true, false>(), prepare_dma<4, 3, false, false, true>(),
      // weight gradients
      prepare_dma<4, 0, false, true, false>(), prepare_dma<4, 0, false, true, false, false, false, true>(),
      // whole 256-row tiles and any number of rows: forward, data gradients
#define MOE_DMA_BOTH(...) prepare_dma<__VA_ARGS__, false>(), prepare_dma<__VA_ARGS__, true>()
      MOE_DMA_BOTH(4, 1, false, false, false, false, false, false), MOE_DMA_BOTH(4, 0, false, false, false, false, false, false),
      MOE_DMA_BOTH(4, 1, true, false, false, true, false, false), MOE_DMA_BOTH(4, 4, true, false, false, true, false, false),
      MOE_DMA_BOTH(4, 0, false, false, false, true, false, false), MOE_DMA_BOTH(4, 2, false, false, true, false, false, false),
      MOE_DMA_BOTH(4, 0, false, false, true, false, false, false), MOE_DMA_BOTH(4, 5, false, false, true, true, false, false),
      MOE_DMA_BOTH(4, 0, false, false, true, true, false, false),
#undef MOE_DMA_BOTH
      // other shapes: forward (relu / plain), data gradients (plain / masked), weight gradients
#define MOE_EDGE_KC(...)                                                                       \
  prepare_edge<128, 256, 32, 3, __VA_ARGS__>(), prepare_edge<128, 128, 64, 2, __VA_ARGS__>(),  \
      prepare_edge<128, 128, 64, 3, __VA_ARGS__>(), prepare_edge<64, 128, 64, 2, __VA_ARGS__>(), \
      prepare_edge<64, 128, 64, 3, __VA_ARGS__>(), prepare_edge<64, 64, 64, 3, __VA_ARGS__>(), \
      prepare_edge<64, 64, 64, 4, __VA_ARGS__>()
#define MOE_EDGE_MNC(...)                                                                      \
  prepare_edge<128, 256, 32, 3, __VA_ARGS__>(), prepare_edge<128, 128, 32, 3, __VA_ARGS__>(),  \
      prepare_edge<64, 128, 32, 4, __VA_ARGS__>(), prepare_edge<64, 64, 32, 5, __VA_ARGS__>()
      MOE_EDGE_KC(1, false, false, false), MOE_EDGE_KC(0, false, false, false), MOE_EDGE_KC(0, false, true, false),
      MOE_EDGE_KC(2, false, true, false), MOE_EDGE_MNC(0, true, false, false), MOE_EDGE_MNC(0, true, false, true),
      MOE_EDGE_MNC(3, true, false, false),
#define MOE_PAIR(BM, BN, DEEP, FLAT) \
  prepare_pair<BM, BN, DEEP, 64, 64, 5>(), prepare_pair<BM, BN, DEEP, 64, 128, 4>(), prepare_pair<BM, BN, FLAT, 128, 128, 3>()
      MOE_PAIR(64, 64, 4, 3), MOE_PAIR(64, 128, 2, 2), MOE_PAIR(128, 128, 2, 2)};
#undef MOE_PAIR
#undef MOE_EDGE_KC
#undef MOE_EDGE_MNC
  int cus = 0;
  if (compute_units(&cus) != MOE_OK) return MOE_EHIP;
  for (int rc : rcs)
    if (rc != MOE_OK) return rc;
  return MOE_OK;
}

static int rows_per_expert(const moe_config& c, int* R) {
  const long long rows = (long long)c.G * c.C;
  if (rows > 0x7fffffffLL) return MOE_EUNSUPPORTED;
  *R = (int)rows;
  return MOE_OK;
}

int launch_expert_gemm1(const moe_config& c, const void* buf, const void* wi, void* h,
                        hipStream_t st) {
  int R;
  const int rc = rows_per_expert(c, &R);
  if (rc != MOE_OK) return rc;
  if (c.act_dtype == MOE_F32)
    return launch_gemm_f32(kForwardRelu, GemmArgs{buf, wi, h}, c.E, R, c.H, c.M, st);
  return gemm_bf16<true>(static_cast<const bf16_t*>(buf), static_cast<const bf16_t*>(wi),
                         static_cast<bf16_t*>(h), c.E, R, c.H, c.M, st);
}

// Batched bf16 GEMM with an fp32 result for the gate gradients (A, B, C as in the kernel's
// layout table; batch plays the role of the expert index).
bool gemm_bf16_f32out_ok(int R, int N, int K) { return dma_shape_ok(R, N, K); }

int launch_gemm_bf16_f32out(bool transposed_a, const void* A, const void* B, float* Cout,
                            int batch, int R, int N, int K, hipStream_t st) {
  if (!dma_shape_ok(R, N, K)) return MOE_EUNSUPPORTED;
  auto a = static_cast<const bf16_t*>(A);
  auto b = static_cast<const bf16_t*>(B);
  auto c = reinterpret_cast<bf16_t*>(Cout);
  // transposed_a: C = A^T . B with A [K,R], B [K,N];  else C = A . B^T with A [R,K], B [N,K]
  return transposed_a
             ? launch_bf16_dma<4, 3, false, true, false>(a, b, c, batch, R, N, K, nullptr, nullptr, st)
             : launch_bf16_dma<4, 3, false, false, true>(a, b, c, batch, R, N, K, nullptr, nullptr, st);
}

// Which layers take the packed row layout, gathering the rows of x in the first GEMM: those with
// M >= 128 (the persistent kernel fetches a tile's row indices 4 K steps of 32 ahead of its first copy)
// and row counts of the experts that fit the LDS left over by its stages.
bool expert_ffn_can_pack(const moe_config& c) {
  return (long long)c.G * c.C <= 0x7fffffffLL && c.M >= 128 && c.E <= 2048;
}

bool expert_ffn_whole_tiles(const moe_config& c) {
  return c.act_dtype == MOE_BF16 && expert_ffn_can_pack(c) && dma_shape_ok(c.G * c.C, c.H, c.M) &&
         dma_shape_ok(c.G * c.C, c.M, c.H);
}

size_t expert_signbits_bytes(const moe_config& c) {
  const bool kept = c.act_dtype == MOE_BF16 && expert_ffn_can_pack(c) && dma_columns_ok(c.G * c.C, c.H, c.M);
  return kept ? (size_t)c.E * align_up((size_t)c.G * c.C, 256) * c.H / 8 : 0;      // of whole 256-row tiles
}

// The weight gradients sum over whole 256-row tiles when the persistent kernel forms them: the rows of
// h and dh behind the occupied ones then have to be zeros up to there.
static int packed_row_pad(const moe_config& c) {
  GemmForm f1, f2;
  const int R = c.G * c.C;
  if (choose_form(c.E, c.H, c.M, R, kLayoutWeightGrad, &f1, true) != MOE_OK || choose_form(c.E, c.M, c.H, R, kLayoutWeightGrad, &f2, true) != MOE_OK)
    return 255;
  return f1 == kPersistent || f2 == kPersistent ? 255 : 0;
}

// Packed row layout: both GEMMs walk the occupied row tiles.  The first gathers its rows
// through pk.packed_src (absolute rows of `a`: token rows of x, or rows of an [E,G,C,M] buffer),
// h and (scatter_out == false) out hold packed rows; scatter_out sends the rows of out back to
// the absolute rows pk.packed_src names.
int launch_expert_ffn_packed(const moe_config& c, const void* a, const RowPacking& pk,
                             const void* zero_row, const void* wi, const void* wo, void* h,
                             void* out, bool scatter_out, bool train, void* signbits, hipStream_t st,
                             void* event_between) {
  if (!expert_ffn_can_pack(c)) return MOE_EUNSUPPORTED;
  const int R = c.G * c.C;
  auto between = [&] {
    return event_between == nullptr || hipEventRecord(static_cast<hipEvent_t>(event_between), st) == hipSuccess;
  };
  GemmArgs g1{a, wi, h}, g2{h, wo, out};
  g1.gather = pk.packed_src;
  g1.kept = g2.kept = pk.kept;
  g2.scatter = scatter_out ? pk.packed_src : nullptr;
  int rc;
  if (c.act_dtype == MOE_F32) {
    if (scatter_out) return MOE_EUNSUPPORTED;
    rc = launch_gemm_f32(kForwardRelu, g1, c.E, R, c.H, c.M, st);
    if (rc != MOE_OK) return rc;
    if (!between()) return MOE_EHIP;
    return launch_gemm_f32(kForward, g2, c.E, R, c.M, c.H, st);
  }
  GemmForm f1, f2, dh;
  if ((train ? choose_train_forms(c, &f1, &dh) : choose_form(c.E, R, c.H, c.M, kLayoutForward, &f1)) != MOE_OK ||
      choose_form(c.E, R, c.M, c.H, kLayoutForward, &f2) != MOE_OK)
    return MOE_EHIP;
  if (f1 != kPersistent) {
    g1.row_pad = train ? packed_row_pad(c) : 0;
    rc = gemm_bf16_edge<1, false, false>(f1, g1, c.E, R, c.H, c.M, st);
  } else if (signbits != nullptr) {
    rc = launch_bf16_dma<4, 4, true, false, false, true>(
        static_cast<const bf16_t*>(a), static_cast<const bf16_t*>(wi), static_cast<bf16_t*>(h), c.E, R,
        c.H, c.M, pk.packed_src, static_cast<const bf16_t*>(zero_row), st, nullptr,
        static_cast<unsigned char*>(signbits), pk.kept);
  } else {
    rc = launch_bf16_dma<4, 1, true, false, false, true>(
        static_cast<const bf16_t*>(a), static_cast<const bf16_t*>(wi), static_cast<bf16_t*>(h), c.E, R,
        c.H, c.M, pk.packed_src, static_cast<const bf16_t*>(zero_row), st, nullptr, nullptr,
        pk.kept);
  }
  if (rc != MOE_OK) return rc;
  if (!between()) return MOE_EHIP;
  if (f2 != kPersistent) return gemm_bf16_edge<0, false, false>(f2, g2, c.E, R, c.M, c.H, st);
  if (scatter_out)
    return launch_bf16_dma<4, 0, false, false, false, true, true>(
        static_cast<const bf16_t*>(h), static_cast<const bf16_t*>(wo), static_cast<bf16_t*>(out), c.E,
        R, c.M, c.H, pk.packed_src, nullptr, st, nullptr, nullptr, pk.kept);
  return launch_bf16_dma<4, 0, false, false, false, true, false>(
      static_cast<const bf16_t*>(h), static_cast<const bf16_t*>(wo), static_cast<bf16_t*>(out), c.E, R,
      c.M, c.H, nullptr, nullptr, st, nullptr, nullptr, pk.kept);
}

// dW [in,out] = X^T dY over rows tokens: few tiles and a long sum.  The ranges run as a batch with fp32 results,
// at the rule's time for that batch, and adding them up costs a launch and their bytes at about 6 TB/s (they
// are in the last-level cache).  The ranges size a workspace, so they are those of a whole device on any partition.
constexpr int kPlanUnits = 256;
DenseWgradPlan dense_wgrad_plan(long long rows, int in, int out) {
  DenseWgradPlan best{1, (int)rows};
  double best_us = 0;
  for (int want = 1; want <= 16; want += want < 4 ? 1 : want < 8 ? 2 : 4) {
    const int k = (int)(((rows + want - 1) / want + 31) / 32 * 32), sp = (int)((rows + k - 1) / k);
    if (want > 1 && (k < 128 || sp < want)) continue;
    const bool persistent = dma_shape_ok(in, out, k) && (long long)sp * k == rows;
    double us = 0;
    gemm_form(persistent, sp, in, out, sp == 1 ? (int)rows : k, kLayoutWeightGrad, kPlanUnits, &us);
    if (sp > 1) us += 3.0 + 4e-6 * sp * in * out / 6.0;
    if (want == 1 || us < best_us) { best_us = us; best = DenseWgradPlan{sp, sp == 1 ? (int)rows : k}; }
  }
  return best;
}

// the batch of the plan: partial [splits, in, out]
int launch_dense_wgrad_ranges(const DenseWgradPlan& p, long long rows, int in, int out, const void* X, const void* dY,
                              float* partial, hipStream_t st) {
  const bool persistent = dma_shape_ok(in, out, p.k) && (long long)p.splits * p.k == rows;
  const GemmForm form = gemm_form(persistent, p.splits, in, out, p.k, kLayoutWeightGrad, kPlanUnits);
  if (form == kPersistent) return launch_gemm_bf16_f32out(true, X, dY, partial, p.splits, in, out, p.k, st);
  return gemm_bf16_edge<3, true, false>(form, GemmArgs{X, dY, partial}, p.splits, in, out, p.k, st, (int)rows);
}

int launch_expert_gemm2(const moe_config& c, const void* h, const void* wo, void* out,
                        hipStream_t st) {
  int R;
  const int rc = rows_per_expert(c, &R);
  if (rc != MOE_OK) return rc;
  if (c.act_dtype == MOE_F32)
    return launch_gemm_f32(kForward, GemmArgs{h, wo, out}, c.E, R, c.M, c.H, st);
  return gemm_bf16<false>(static_cast<const bf16_t*>(h), static_cast<const bf16_t*>(wo),
                          static_cast<bf16_t*>(out), c.E, R, c.M, c.H, st);
}

// ---- backward pass: A K-contiguous x B K-contiguous (dgrad), A and B row(k)-major (wgrad) ----
int launch_expert_dgrad2(const moe_config& c, const void* dout, const void* wo, const void* h,
                         const void* signbits, void* dh, const int32_t* kept, hipStream_t st) {
  const long long R = (long long)c.G * c.C;
  if (R > 0x7fffffffLL) return MOE_EUNSUPPORTED;
  GemmArgs g{dout, wo, dh, h};
  g.kept = kept;
  if (c.act_dtype == MOE_F32) return launch_gemm_f32(kDataGradMask, g, c.E, (int)R, c.H, c.M, st);
  auto a = static_cast<const bf16_t*>(dout);
  auto b = static_cast<const bf16_t*>(wo);
  auto o = static_cast<bf16_t*>(dh);
  auto sign = const_cast<unsigned char*>(static_cast<const unsigned char*>(signbits));
  GemmForm form, h_form;
  if ((kept != nullptr ? choose_train_forms(c, &h_form, &form)
                       : choose_form(c.E, (int)R, c.H, c.M, kLayoutMaskedDataGrad, &form)) != MOE_OK)
    return MOE_EHIP;
  if (form != kPersistent) {
    g.row_pad = kept != nullptr ? packed_row_pad(c) : 0;
    return gemm_bf16_edge<2, false, true>(form, g, c.E, (int)R, c.H, c.M, st);
  }
  if (kept != nullptr) {
    if (signbits == nullptr) return MOE_EINVAL;
    return launch_bf16_dma<4, 5, false, false, true, true>(a, b, o, c.E, (int)R, c.H, c.M, nullptr, nullptr,
                                                       st, nullptr, sign, kept);
  }
  return launch_bf16_dma<4, 2, false, false, true>(a, b, o, c.E, (int)R, c.H, c.M, nullptr, nullptr, st,
                                               static_cast<const bf16_t*>(h));
}

// C = A^T . B of a weight gradient, [N1,N2] per expert summed over its rows (kept: packed rows)
static int wgrad(const moe_config& c, const void* A, const void* B, void* dw, int N1, int N2,
                 const int32_t* kept, hipStream_t st) {
  const long long R = (long long)c.G * c.C;
  if (R > 0x7fffffffLL) return MOE_EUNSUPPORTED;
  GemmArgs g{A, B, dw};
  g.kept = kept;
  if (c.act_dtype == MOE_F32) return launch_gemm_f32(kWeightGrad, g, c.E, N1, N2, (int)R, st);
  GemmForm form;
  if (choose_form(c.E, N1, N2, (int)R, kLayoutWeightGrad, &form, kept != nullptr) != MOE_OK) return MOE_EHIP;
  if (form != kPersistent)
    return kept != nullptr ? gemm_bf16_edge<0, true, false, true>(form, g, c.E, N1, N2, (int)R, st)
                           : gemm_bf16_edge<0, true, false>(form, g, c.E, N1, N2, (int)R, st);
  auto a = static_cast<const bf16_t*>(A);
  auto b = static_cast<const bf16_t*>(B);
  auto o = static_cast<bf16_t*>(dw);
  if (kept != nullptr)
    return launch_bf16_dma<4, 0, false, true, false, false, false, true>(a, b, o, c.E, N1, N2, (int)R, nullptr,
                                                                     nullptr, st, nullptr, nullptr,
                                                                     kept);
  return launch_bf16_dma<4, 0, false, true, false>(a, b, o, c.E, N1, N2, (int)R, nullptr, nullptr, st);
}

int launch_expert_wgrad2(const moe_config& c, const void* h, const void* dout, void* dwo,
                         const int32_t* kept, hipStream_t st) {
  return wgrad(c, h, dout, dwo, c.H, c.M, kept, st);
}

int launch_expert_dgrad1(const moe_config& c, const void* dh, const void* wi, void* dbuf,
                         const int32_t* kept, hipStream_t st) {
  const long long R = (long long)c.G * c.C;
  if (R > 0x7fffffffLL) return MOE_EUNSUPPORTED;
  GemmArgs g{dh, wi, dbuf};
  g.kept = kept;
  if (c.act_dtype == MOE_F32) return launch_gemm_f32(kDataGrad, g, c.E, (int)R, c.M, c.H, st);
  auto a = static_cast<const bf16_t*>(dh);
  auto b = static_cast<const bf16_t*>(wi);
  auto o = static_cast<bf16_t*>(dbuf);
  GemmForm form;
  if (choose_form(c.E, (int)R, c.M, c.H, kLayoutDataGrad, &form) != MOE_OK) return MOE_EHIP;
  if (form != kPersistent) return gemm_bf16_edge<0, false, true>(form, g, c.E, (int)R, c.M, c.H, st);
  if (kept != nullptr)
    return launch_bf16_dma<4, 0, false, false, true, true>(a, b, o, c.E, (int)R, c.M, c.H, nullptr, nullptr,
                                                       st, nullptr, nullptr, kept);
  return launch_bf16_dma<4, 0, false, false, true>(a, b, o, c.E, (int)R, c.M, c.H, nullptr, nullptr, st);
}

int launch_expert_wgrad1(const moe_config& c, const void* buf, const void* dh, void* dwi,
                         const int32_t* kept, hipStream_t st) {
  return wgrad(c, buf, dh, dwi, c.M, c.H, kept, st);
}

// The gradients of out = h . wo (dh, dwo; masked) and of h = relu(x . wi) (dbuf, dwi), in one launch where that is faster.
// upstream [R,K], weight [N,K]: [R,K] . [N,K]^T -> [R,N] and [R,N]^T . [R,K] -> [N,K]
static bool expert_pair(const moe_config& c, bool masked, bool packed, int cus, PairProduct* d, PairProduct* w) {
  const int R = c.G * c.C, N = masked ? c.H : c.M, K = masked ? c.M : c.H;
  const GemmLayout layout = masked ? kLayoutMaskedDataGrad : kLayoutDataGrad;
  d->E = w->E = c.E;
  d->R = w->K = R; d->N = w->R = N; d->K = w->N = K;
  GemmForm h;
  if (masked && packed) train_forms_of(c, cus, &h, &d->form, &d->us);
  else d->form = form_of(c.E, R, N, K, layout, false, cus, &d->us);
  w->form = form_of(c.E, N, K, R, kLayoutWeightGrad, packed, cus, &w->us);
  return pair_ok(d, layout, w, cus);
}
static int pair_or_none(const moe_config& c, bool masked, const GemmArgs& data, const GemmArgs& weight, const int32_t* kept,
                        hipStream_t st, bool* done) {
  int cus = 0;
  if (compute_units(&cus) != MOE_OK) return MOE_EHIP;
  PairProduct d{data}, w{weight};
  return expert_pair(c, masked, kept != nullptr, cus, &d, &w) ? launch_pair(d, w, st, done) : MOE_OK;
}
bool gradient_pair_forms(const moe_config& c, bool masked, int cus, int* data, int* weight) {
  PairProduct d{}, w{};
  if (c.act_dtype != MOE_BF16 || !expert_pair(c, masked, expert_ffn_can_pack(c), cus, &d, &w)) return false;
  *data = d.form;
  *weight = w.form;
  return true;
}

int launch_expert_grads2(const moe_config& c, const void* dout, const void* wo, const void* h, const void* signbits, void* dh,
                         void* dwo, const int32_t* kept, hipStream_t st) {
  if (c.act_dtype == MOE_BF16 && (long long)c.G * c.C <= 0x7fffffffLL) {
    GemmArgs d{dout, wo, dh, h}, w{h, dout, dwo};
    d.kept = w.kept = kept;
    if (kept != nullptr) d.row_pad = packed_row_pad(c);
    bool done = false;
    const int rc = pair_or_none(c, true, d, w, kept, st, &done);
    if (rc != MOE_OK || done) return rc;
  }
  const int rc = launch_expert_dgrad2(c, dout, wo, h, signbits, dh, kept, st);
  return rc != MOE_OK ? rc : launch_expert_wgrad2(c, h, dout, dwo, kept, st);
}

int launch_expert_grads1(const moe_config& c, const void* dh, const void* wi, void* dbuf, const void* buf, void* dwi,
                         const int32_t* kept, hipStream_t st) {
  if (c.act_dtype == MOE_BF16 && (long long)c.G * c.C <= 0x7fffffffLL) {
    GemmArgs d{dh, wi, dbuf}, w{buf, dh, dwi};
    d.kept = w.kept = kept;
    bool done = false;
    const int rc = pair_or_none(c, false, d, w, kept, st, &done);
    if (rc != MOE_OK || done) return rc;
  }
  const int rc = launch_expert_dgrad1(c, dh, wi, dbuf, kept, st);
  return rc != MOE_OK ? rc : launch_expert_wgrad1(c, buf, dh, dwi, kept, st);
}

// dX [rows,in] = dY . W^T (0 where mask <= 0) and dW [in,out] = X^T . dY of a dense layer in one launch, dW in the plan's
// ranges (partial); false: to be launched one after the other
int launch_dense_grads_pair(const DenseWgradPlan& p, long long rows, int in, int out, const void* X, const void* dY,
                            const void* W, const void* mask, void* dX, void* dW, float* partial, hipStream_t st, bool* done) {
  *done = false;
  PairProduct d{GemmArgs{dY, W, dX, mask}, 1, (int)rows, in, out, kPersistent, 0};
  PairProduct w{GemmArgs{X, dY, p.splits > 1 ? static_cast<void*>(partial) : dW}, p.splits, in, out, p.splits > 1 ? p.k : (int)rows, kPersistent, 0};
  w.k_total = p.splits > 1 ? (int)rows : 0;
  int cus = 0;
  if (compute_units(&cus) != MOE_OK) return MOE_EHIP;
  const GemmLayout layout = mask != nullptr ? kLayoutMaskedDataGrad : kLayoutDataGrad;
  const bool persistent = dma_shape_ok(in, out, w.K) && (long long)p.splits * w.K == rows;
  d.form = form_of(1, (int)rows, in, out, layout, false, cus, &d.us);
  w.form = gemm_form(persistent, p.splits, in, out, w.K, kLayoutWeightGrad, cus, &w.us);
  return pair_ok(&d, layout, &w, cus) ? launch_pair(d, w, st, done) : MOE_OK;
}

}  // namespace moe
