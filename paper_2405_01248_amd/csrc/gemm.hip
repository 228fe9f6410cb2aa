// GEMM kernels for the projections and MLPs of a stage (forward y = x W^T, backward
// dx = dy W and dW = dy^T x), fp32 accumulation, with fused epilogues.
//
// bf16 path: MFMA tiles fed from LDS.  An operand whose contraction index is
// contiguous in memory is staged [rows][BK] and read with 16-byte LDS loads; an operand
// whose contraction index is the slow one (both operands in dW, weights in dx where a stage
// reads them as they are stored) is staged [BK][cols] exactly as it sits in HBM and read with
// the transposing LDS load.  Workgroup ids are remapped so that the tiles running on one XCD
// (one L2) are neighbours in the output.
// Elsewhere: the weight gradients of a block in one launch (gemm_dw.hip), at most 48 rows
// (gemm_few_rows.hip), fp32 (gemm_f32.hip).
#include "dp_device.h"
#include "dp_kernels.h"
#include "dp_errors.h"
#include "dp_ktime.h"
#include "dp_gemm_epilogue.h"
#include "dp_gemm_pp.h"
#include "dp_gemm_ring.h"
#include "dp_host.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>

namespace dp {

// ------------------------------------------------------------------ bf16 MFMA kernel
struct GemmBf16Params {
  const bf16* A; const bf16* B;
  int M, N, K, lda, ldb;
  int k_tiles_per_split;
  int tiles_m, tiles_n;
  int group_m;                 // tile-rows per group of the workgroup-to-tile map (choose_group_m)
  int split_major;             // register-staged kernel: number of splits of a 1-D grid over (split, tile) pairs, 0 = plain grid of tiles
  // Column sums of the A operand over the contraction (register-staged kernel, contraction-strided A only: the
  // bias gradient next to a weight gradient).  colsum[blockIdx.z * colsum_stride + m]; colsum_acc: add to what is there.
  float* colsum; int colsum_stride; int colsum_acc;
  uint32_t a_bytes, b_bytes;   // extent of each operand in bytes (direct-to-LDS kernels address it with 32-bit offsets)
  EpiParams<bf16> epi;
  // gemm_wave_kernel with NORM: the rows operand is LN(norm_x)
  const float* norm_x; const bf16* norm_gamma; const bf16* norm_beta; float norm_eps;
};

// The direct-to-LDS kernels need both operands below 4 GiB.
static inline bool dtl_addressable(const GemmArgs& a) {
  const size_t ab = a.a_mc ? operand_extent_bytes(a.K, a.M, a.lda) : operand_extent_bytes(a.M, a.K, a.lda);
  const size_t bb = a.b_mc ? operand_extent_bytes(a.K, a.N, a.ldb) : operand_extent_bytes(a.N, a.K, a.ldb);
  return ab < (1ull << 32) && bb < (1ull << 32);
}

template <int BM, int BN, int BK, int WGM, int WGN, bool A_MC, bool B_MC>
struct GemmSmem {
  // [rows][BK + 8] for contraction-contiguous operands; [BK][cols], unpadded with permuted 16-byte
  // chunks (mc_swizzle), for the others
  static constexpr int A_LD = A_MC ? BM : (BK + 8);
  static constexpr int B_LD = B_MC ? BN : (BK + 8);
  static constexpr int A_ELEMS = A_MC ? BK * A_LD : BM * A_LD;
  static constexpr int B_ELEMS = B_MC ? BK * B_LD : BN * B_LD;
  static constexpr int WN = BN / WGN;
  static constexpr int C_LD = WN + 4;                                   // per-wave fp32 staging [32][WN + 4]
  static constexpr size_t TILE_BYTES = 2 * (size_t)(A_ELEMS + B_ELEMS) * 2;
  static constexpr size_t EPI_BYTES = (size_t)WGM * WGN * 32 * C_LD * 4;
  static constexpr size_t BYTES = TILE_BYTES > EPI_BYTES ? TILE_BYTES : EPI_BYTES;
};

template <int BM, int BN, int BK, int WGM, int WGN, bool A_MC, bool B_MC>
__global__ void __launch_bounds__(WGM * WGN * 64)
gemm_bf16_kernel(const GemmBf16Params p) {
  using S = GemmSmem<BM, BN, BK, WGM, WGN, A_MC, B_MC>;
  constexpr int NT = WGM * WGN * 64;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int A_CHUNKS = BM * BK / 8, B_CHUNKS = BN * BK / 8;
  constexpr int A_PER = A_CHUNKS / NT, B_PER = B_CHUNKS / NT;
  static_assert(A_CHUNKS % NT == 0 && B_CHUNKS % NT == 0, "tile/threads mismatch");

  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16* As = reinterpret_cast<bf16*>(smem_raw);
  bf16* Bs = As + 2 * S::A_ELEMS;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 5, l32 = lane & 31;
  const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;
  // Split-K launches come as a 1-D grid over (split, tile) pairs in split-major order, of which every XCD takes a
  // contiguous range (the hardware deals consecutive workgroups round-robin to the 8 XCDs): the tiles of one split,
  // which read the same slice of both operands, run on one or two XCDs instead of all eight.
  int split = 0, tile_m, tile_n;
  if (p.split_major) {
    const int T = p.tiles_m * p.tiles_n;
    const int id = xcd_contiguous_id(blockIdx.x, T * p.split_major);
    split = id / T;
    tile_of_id(id % T, p.tiles_m, p.tiles_n, p.group_m, tile_m, tile_n);
  } else {
    tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tile_m, tile_n);
  }
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  EpiParams<bf16> epi = p.epi;
  if (p.split_major && epi.partial) epi.partial += (size_t)split * p.M * p.N;   // blockIdx.z is 0 in the 1-D grid

  const int total_kt = (p.K + BK - 1) / BK;
  const int kt_begin = split * p.k_tiles_per_split;
  const int kt_end = min(total_kt, kt_begin + p.k_tiles_per_split);

  // staged tile chunks; out-of-range chunks are loaded from a clamped (valid) address and
  // zeroed only when they are written to LDS, so nothing waits on the loads before the MFMAs
  bf16x8 ra[A_PER], rb[B_PER];
  unsigned oka = 0, okb = 0;
  // bias gradient: every thread always stages the same 8 columns of A (NT is a multiple of BM / 8), so it keeps
  // their running sums; only the workgroups of the first tile column do
  const bool do_colsum = A_MC && p.colsum != nullptr && tile_n == 0;
  float csum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#define DP_GEMM_LOAD_GLOBAL(kt_)                                                              \
  {                                                                                           \
    const int k0_ = (kt_) * BK;                                                               \
    oka = 0; okb = 0;                                                                         \
    _Pragma("unroll") for (int i = 0; i < A_PER; ++i) {                                       \
      const int id = tid + i * NT;                                                            \
      if (A_MC) {                                                                             \
        const int kk = id / (BM / 8), c = id % (BM / 8);                                      \
        const int gk = k0_ + kk, gm = m0 + c * 8;                                             \
        ra[i] = *reinterpret_cast<const bf16x8*>(p.A + (size_t)min(gk, p.K - 1) * p.lda + min(gm, p.M - 8)); \
        oka |= (unsigned)(gk < p.K && gm < p.M) << i;                                         \
      } else {                                                                                \
        const int r = id / (BK / 8), c = id % (BK / 8);                                       \
        const int gm = m0 + r, gk = k0_ + c * 8;                                              \
        ra[i] = *reinterpret_cast<const bf16x8*>(p.A + (size_t)min(gm, p.M - 1) * p.lda + min(gk, p.K - 8)); \
        oka |= (unsigned)(gm < p.M && gk < p.K) << i;                                         \
      }                                                                                       \
    }                                                                                         \
    _Pragma("unroll") for (int i = 0; i < B_PER; ++i) {                                       \
      const int id = tid + i * NT;                                                            \
      if (B_MC) {                                                                             \
        const int kk = id / (BN / 8), c = id % (BN / 8);                                      \
        const int gk = k0_ + kk, gn = n0 + c * 8;                                             \
        rb[i] = *reinterpret_cast<const bf16x8*>(p.B + (size_t)min(gk, p.K - 1) * p.ldb + min(gn, p.N - 8)); \
        okb |= (unsigned)(gk < p.K && gn < p.N) << i;                                         \
      } else {                                                                                \
        const int r = id / (BK / 8), c = id % (BK / 8);                                       \
        const int gn = n0 + r, gk = k0_ + c * 8;                                              \
        rb[i] = *reinterpret_cast<const bf16x8*>(p.B + (size_t)min(gn, p.N - 1) * p.ldb + min(gk, p.K - 8)); \
        okb |= (unsigned)(gn < p.N && gk < p.K) << i;                                         \
      }                                                                                       \
    }                                                                                         \
  }
#define DP_GEMM_STORE_LDS(buf_)                                                               \
  {                                                                                           \
    bf16* as_ = As + (buf_) * S::A_ELEMS;                                                     \
    bf16* bs_ = Bs + (buf_) * S::B_ELEMS;                                                     \
    _Pragma("unroll") for (int i = 0; i < A_PER; ++i) {                                       \
      const int id = tid + i * NT;                                                            \
      if (A_MC) { const int kk = id / (BM / 8), c = id % (BM / 8); const bf16x8 v_ = ((oka >> i) & 1) ? ra[i] : zero8(); \
                  *reinterpret_cast<bf16x8*>(as_ + kk * S::A_LD + mc_swizzle(c, kk) * 8) = v_;                \
                  if (do_colsum) { _Pragma("unroll") for (int t_ = 0; t_ < 8; ++t_) csum[t_] += (float)v_[t_]; } } \
      else      { const int r = id / (BK / 8), c = id % (BK / 8);  *reinterpret_cast<bf16x8*>(as_ + r * S::A_LD + c * 8) = ((oka >> i) & 1) ? ra[i] : zero8(); }  \
    }                                                                                         \
    _Pragma("unroll") for (int i = 0; i < B_PER; ++i) {                                       \
      const int id = tid + i * NT;                                                            \
      if (B_MC) { const int kk = id / (BN / 8), c = id % (BN / 8); *reinterpret_cast<bf16x8*>(bs_ + kk * S::B_LD + mc_swizzle(c, kk) * 8) = ((okb >> i) & 1) ? rb[i] : zero8(); } \
      else      { const int r = id / (BK / 8), c = id % (BK / 8);  *reinterpret_cast<bf16x8*>(bs_ + r * S::B_LD + c * 8) = ((okb >> i) & 1) ? rb[i] : zero8(); }  \
    }                                                                                         \
  }

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  if (kt_begin < kt_end) {
    DP_GEMM_LOAD_GLOBAL(kt_begin);
    DP_GEMM_STORE_LDS(0);
  }
  __syncthreads();

  for (int kt = kt_begin; kt < kt_end; ++kt) {
    const int buf = (kt - kt_begin) & 1;
    const bool more = kt + 1 < kt_end;
    if (more) DP_GEMM_LOAD_GLOBAL(kt + 1);
    const bf16* as = As + buf * S::A_ELEMS;
    const bf16* bs = Bs + buf * S::B_ELEMS;
    // fragments of k-step ks + 1 are fetched from LDS before the MFMAs of k-step ks are issued
    bf16x8 fa[2][TM], fb[2][TN];
#define DP_GEMM_LOAD_FRAGS(ks_, set_)                                                                                   \
    {                                                                                                                     \
      _Pragma("unroll") for (int i = 0; i < TM; ++i) {                                                                   \
        if (A_MC) fa[set_][i] = frag_from_mc_swz(as, S::A_LD, (ks_) * 16, wm0 + i * 32, lane);                 \
        else      fa[set_][i] = *reinterpret_cast<const bf16x8*>(as + (wm0 + i * 32 + l32) * S::A_LD + (ks_) * 16 + 8 * g); \
      }                                                                                                                   \
      _Pragma("unroll") for (int j = 0; j < TN; ++j) {                                                                   \
        if (B_MC) fb[set_][j] = frag_from_mc_swz(bs, S::B_LD, (ks_) * 16, wn0 + j * 32, lane);                 \
        else      fb[set_][j] = *reinterpret_cast<const bf16x8*>(bs + (wn0 + j * 32 + l32) * S::B_LD + (ks_) * 16 + 8 * g); \
      }                                                                                                                   \
    }
    DP_GEMM_LOAD_FRAGS(0, 0);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      if (ks + 1 < BK / 16) DP_GEMM_LOAD_FRAGS(ks + 1, (ks + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma32(fa[ks & 1][i], fb[ks & 1][j], acc[i][j]);
    }
#undef DP_GEMM_LOAD_FRAGS
    if (more) DP_GEMM_STORE_LDS(buf ^ 1);
    __syncthreads();
  }

  if (A_MC && do_colsum) {      // workgroup-uniform
    // fixed order: a thread's rows in k order (above), then the NT / (BM / 8) row groups in ascending order
    constexpr int GROUPS = NT / (BM / 8);
    float* red = reinterpret_cast<float*>(smem_raw);
    const int c = tid % (BM / 8), grp = tid / (BM / 8);
#pragma unroll
    for (int t = 0; t < 8; ++t) red[grp * BM + c * 8 + t] = csum[t];
    __syncthreads();
    if (tid < BM && m0 + tid < p.M) {
      float sum = 0.f;
      for (int g2 = 0; g2 < GROUPS; ++g2) sum += red[g2 * BM + tid];
      float* o = p.colsum + (size_t)split * p.colsum_stride + m0 + tid;
      *o = p.colsum_acc ? *o + sum : sum;
    }
    __syncthreads();
  }
  float* Cw = reinterpret_cast<float*>(smem_raw) + wave * 32 * S::C_LD;
  wave_epilogue<TM, TN, WN, S::C_LD>(acc, Cw, epi, m0 + wm0, n0 + wn0, lane);
}

#undef DP_GEMM_LOAD_GLOBAL
#undef DP_GEMM_STORE_LDS

// ------------------------------------------------------------------ bf16 MFMA kernel, direct-to-LDS pipeline
// Same tiling and epilogue, but the operand tiles travel global -> LDS without passing through
// registers (buffer_load_dwordx4 ... lds: every lane fetches 16 bytes, the wave's 1 KB lands
// contiguously in LDS) in a ring of three or four buffers, two or three k-tiles ahead of the
// MFMAs.  What bounds this loop on MI355X is not one pipe but three at once: per k-tile a
// 256x128 workgroup needs about as many LDS cycles (fragment reads plus the incoming copies) and
// three quarters as many L1 address cycles as MFMA cycles, so copies, fragment reads and MFMAs
// are interleaved finely and every wait names exactly the data it needs.  The copies use the
// buffer-descriptor form because a flat-address LDS copy in flight makes the compiler treat the
// LDS counter as unordered (every wait for one fragment becomes a wait for all).  LDS tiles are unpadded; bank conflicts
// are avoided by permuting 16-byte chunks inside a row (the permutation is applied through
// the per-lane global address, and undone when fragments are read).
//   K-contiguous operand:  tile [rows][32], chunk c of row r stored at c ^ ((r >> 2) & 3).
//   K-strided operand:     tile [BK][cols], chunk c of k-row k stored at c ^ (4 * (k & 3)).
// Requires K % 32 == 0.  Rows / columns beyond M / N are fetched from a clamped address; they
// only feed accumulators whose outputs are never stored.

template <int BM, int BN, int BK, int STAGES, int WGM, int WGN>
struct DtlSmem {
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
  static constexpr int WN = BN / WGN;
  static constexpr int C_LD = WN + 4;
  static constexpr size_t TILE_BYTES = (size_t)STAGES * STAGE;
  static constexpr size_t EPI_BYTES = (size_t)WGM * WGN * 32 * C_LD * 4;
  static constexpr size_t BYTES = TILE_BYTES > EPI_BYTES ? TILE_BYTES : EPI_BYTES;
};

// Chunk permutation of a K-contiguous tile row r (BK / 8 chunks per row): conflict-free 16-byte
// reads by 16 consecutive rows.  BK = 32: 4 chunks, key (r >> 2) & 3; BK = 64: 8 chunks, key (r >> 1) & 7.
template <int BK> __device__ __forceinline__ int kc_key(int r) { return BK == 32 ? ((r >> 2) & 3) : ((r >> 1) & 7); }

// FP8: the operands are OCP E4M3 bytes.  The copy pipeline only moves bytes, so an fp8 row of K bytes is handled as a
// row of K / 2 two-byte elements (all sizes and strides in the parameters are given in those units); what changes is the
// k-step (64 bytes instead of 32: two 16-byte chunks per lane) and the instruction, v_mfma_f32_32x32x64_f8f6f4 with both
// block scales at 2^0.  Any assignment of the 64 bytes of a k-step to lanes and byte slots gives the right product as
// long as it is the same for both operands, which it is by symmetry.
// SEG: the sums of the contraction's segments of k_tiles_per_split k-tiles are formed apart and added in order, the additions of a split-K
// launch and its reduction without the partial tiles' way through memory.
// KIND: the kind of epilogue (PpEpi), whose operands are then requested before the main loop; -1: any, each group of columns requests its own when
// its turn comes.  Few tiles of a short
// contraction end with two to four such waits one after the other: 12 layers on 924 rows of width 768 in the batch-invariant mode 843 -> 811 us.
template <int BM, int BN, int BK, int STAGES, int WGM, int WGN, bool A_MC, bool B_MC, bool FP8 = false, bool SEG = false, int KIND = -1>
__global__ void __launch_bounds__(WGM * WGN * 64)
gemm_bf16_dtl_kernel(const GemmBf16Params p) {
  using S = DtlSmem<BM, BN, BK, STAGES, WGM, WGN>;
  constexpr int NW = WGM * WGN, KS = FP8 ? BK / 32 : BK / 16, CPR = BK / 8;      // k-steps per tile, chunks per K-contiguous row
  static_assert(!FP8 || (!A_MC && !B_MC && BK == 64), "the fp8 variant takes contraction-contiguous operands and 128-byte k-tiles");
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int A_LOADS = S::A_BYTES / 1024 / NW, B_LOADS = S::B_BYTES / 1024 / NW, LOADS = A_LOADS + B_LOADS;
  static_assert(S::A_BYTES % (1024 * NW) == 0 && S::B_BYTES % (1024 * NW) == 0, "tile/waves mismatch");
  static_assert(KS % 2 == 0 && STAGES >= 2, "pipeline shape");
  // 64x64 tiles with four buffers on ring_main_loop (us, K = 768 / 3072 / 4608, 180 tiles: 7.1 -> 5.9 / 17.1 -> 12.4 / 23.8 -> 15.8; as dear with three, where two and more workgroups share
  // a CU, 26.2 -> 28.2 with 612 tiles of K = 3072, and with 128x128 tiles, 8.6 -> 8.8 / 21.3 -> 21.2 / 29.9 -> 29.8 with 72)
  constexpr bool INTERLEAVE = BK == 64 && !FP8 && !A_MC && !B_MC, RING = INTERLEAVE && BM == 64 && BN == 64 && STAGES == 4;

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, l32 = lane & 31;
  const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;
  int tile_m, tile_n;
  tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int kt_begin = blockIdx.z * p.k_tiles_per_split;
  const int kt_end = SEG ? p.K / BK : min(p.K / BK, kt_begin + p.k_tiles_per_split);
  const int nk = kt_end - kt_begin;

  // per-lane byte offset (inside the operand) of each of this wave's 1 KB pieces at k-tile 0;
  // advancing by one k-tile adds a wave-uniform constant.  Rows / column chunks past the matrix edge
  // are clamped to the last valid one (they only feed outputs that are never stored).
  const rsrc_t ra = make_rsrc(p.A, p.a_bytes), rb = make_rsrc(p.B, p.b_bytes);
  uint32_t va[A_LOADS], vb[B_LOADS];
#pragma unroll
  for (int j = 0; j < A_LOADS; ++j) {
    const int blk = wave * A_LOADS + j;
    if (A_MC) {
      const int k = blk * (1024 / (BM * 2)) + lane / (BM / 8), pc = lane % (BM / 8), c = mc_swizzle(pc, k);
      va[j] = 2u * ((uint32_t)(kt_begin * BK + k) * p.lda + min(m0 + c * 8, p.M - 8));
    } else {
      const int r = blk * (512 / BK) + lane / CPR, pc = lane % CPR, c = pc ^ kc_key<BK>(r);
      va[j] = 2u * ((uint32_t)min(m0 + r, p.M - 1) * p.lda + kt_begin * BK + c * 8);
    }
  }
#pragma unroll
  for (int j = 0; j < B_LOADS; ++j) {
    const int blk = wave * B_LOADS + j;
    if (B_MC) {
      const int k = blk * (1024 / (BN * 2)) + lane / (BN / 8), pc = lane % (BN / 8), c = mc_swizzle(pc, k);
      vb[j] = 2u * ((uint32_t)(kt_begin * BK + k) * p.ldb + min(n0 + c * 8, p.N - 8));
    } else {
      const int r = blk * (512 / BK) + lane / CPR, pc = lane % CPR, c = pc ^ kc_key<BK>(r);
      int brow = min(n0 + r, p.N - 1);
      if (p.epi.geglu == 1)   // tile row r: 32-row blocks alternate value / gate rows of the same outputs
        brow = ((r >> 5) & 1) * p.epi.geglu_inner + min(n0 / 2 + (r >> 6) * 32 + (r & 31), p.epi.geglu_inner - 1);
      vb[j] = 2u * ((uint32_t)brow * p.ldb + kt_begin * BK + c * 8);
    }
  }
  const uint32_t a_step = 2u * (A_MC ? (uint32_t)BK * p.lda : BK), b_step = 2u * (B_MC ? (uint32_t)BK * p.ldb : BK);

  // Copies of k-tile t_, to buffer buf_, whose index j (A pieces first, then B) satisfies j % parts_ == part_.
#define DP_DTL_ISSUE_PART(t_, buf_, part_, parts_)                                                                    \
  {                                                                                                                   \
    unsigned char* st_ = smem_raw + (buf_) * S::STAGE;                                                                \
    _Pragma("unroll") for (int j = 0; j < A_LOADS; ++j)                                                               \
      if (j % (parts_) == (part_))                                                                                    \
        async_copy_16B_buf(ra, va[j], (uint32_t)(t_) * a_step, st_ + (wave * A_LOADS + j) * 1024);                    \
    _Pragma("unroll") for (int j = 0; j < B_LOADS; ++j)                                                               \
      if ((A_LOADS + j) % (parts_) == (part_))                                                                        \
        async_copy_16B_buf(rb, vb[j], (uint32_t)(t_) * b_step, st_ + S::A_BYTES + (wave * B_LOADS + j) * 1024);       \
  }

  // What the epilogue reads beside the sums: a lane has the same eight columns of every (512 / WN)-th row
  constexpr int EPI = KIND < 0 ? PE_PLAIN : KIND, CH = WN / 8, NIT = 32 * CH / 64;
  static_assert(KIND < 0 || 64 % CH == 0, "epilogue by kind");
  PpIn<EPI> in[KIND < 0 ? 1 : TM][KIND < 0 ? 1 : NIT];
  float bias[8];
  if constexpr (KIND >= 0) {
    const int n = n0 + wn0 + lane % CH * 8;
    pp_bias(KIND == PE_F32 ? nullptr : p.epi.bias, min(n, p.N - 8), bias);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int it = 0; it < NIT; ++it) pp_load<EPI>(p.epi, m0 + wm0 + i * 32 + (it * 64 + lane) / CH, n, in[i][it]);
    __builtin_amdgcn_sched_barrier(0);
  }

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // (from -0 on, the first segment's sums stay as they are, zeros of either sign included)
  f32x16 total[SEG ? TM : 1][SEG ? TN : 1];
#pragma unroll
  for (int i = 0; i < (SEG ? TM : 0); ++i)
#pragma unroll
    for (int j = 0; j < (SEG ? TN : 0); ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) total[i][j][r] = -0.0f;
  int seg_left = p.k_tiles_per_split;
  // In place, by instructions that name the same register twice: as ordinary additions, both sets of sums are copied on the way round the loop in every
  // k-tile, closed or not (32 instructions, 924 x 768, K = 3072 in eight segments 18.2 -> 14.5 us).  The compiler does not count wait states for
  // inline assembly: 19 after the last product, and the ones behind for the next to take the zeros.
  auto close_segment = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < (SEG ? TM : 0); ++i)
#pragma unroll
      for (int j = 0; j < (SEG ? TN : 0); ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float t = total[i][j][r], a = acc[i][j][r];
          asm volatile("v_add_f32 %0, %0, %1\n\tv_mov_b32 %1, 0" : "+v"(t), "+v"(a));
          total[i][j][r] = t; acc[i][j][r] = a;
        }
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    seg_left = p.k_tiles_per_split;
  };
  if constexpr (RING) {
    ring_main_loop<STAGES, S::STAGE, S::A_BYTES, LOADS>(acc[0], smem_raw, nk, wm0, wn0, lane,
        [&](int t, unsigned char* st) {
          const rsrc_t a = make_rsrc(p.A, t < nk ? p.a_bytes : 0u), b = make_rsrc(p.B, t < nk ? p.b_bytes : 0u);
#pragma unroll
          for (int j = 0; j < A_LOADS; ++j) async_copy_16B_buf(a, va[j], (uint32_t)t * a_step, st + (wave * A_LOADS + j) * 1024);
#pragma unroll
          for (int j = 0; j < B_LOADS; ++j) async_copy_16B_buf(b, vb[j], (uint32_t)t * b_step, st + S::A_BYTES + (wave * B_LOADS + j) * 1024);
        },
        [&]() { if (SEG && --seg_left == 0) close_segment(); });
  } else {
  // Fragment fetch of k-step ks_ of the k-tile in stage st_ into register set set_.
  bf16x8 fa[2][TM], fb[2][TN];
  i32x8 qa[2][FP8 ? TM : 1], qb[2][FP8 ? TN : 1];     // fp8: 32 bytes per lane and fragment
#define DP_DTL_FRAGS(st_, ks_, set_)                                                                                  \
  { if (FP8) {                                                                                                        \
    const unsigned char* as = smem_raw + (st_) * S::STAGE;                                                            \
    const unsigned char* bs = smem_raw + (st_) * S::STAGE + S::A_BYTES;                                               \
    _Pragma("unroll") for (int i = 0; i < (FP8 ? TM : 0); ++i) {                                                      \
      const int r = wm0 + i * 32 + l32, c0 = 4 * (ks_) + 2 * g, key = kc_key<BK>(r);                                  \
      const u32x4 lo = *reinterpret_cast<const u32x4*>(as + r * (2 * BK) + ((c0 ^ key) * 16));                        \
      const u32x4 hi = *reinterpret_cast<const u32x4*>(as + r * (2 * BK) + (((c0 + 1) ^ key) * 16));                  \
      qa[set_][i] = __builtin_bit_cast(i32x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));              \
    }                                                                                                                 \
    _Pragma("unroll") for (int j2 = 0; j2 < (FP8 ? TN : 0); ++j2) {                                                   \
      const int r = wn0 + j2 * 32 + l32, c0 = 4 * (ks_) + 2 * g, key = kc_key<BK>(r);                                 \
      const u32x4 lo = *reinterpret_cast<const u32x4*>(bs + r * (2 * BK) + ((c0 ^ key) * 16));                        \
      const u32x4 hi = *reinterpret_cast<const u32x4*>(bs + r * (2 * BK) + (((c0 + 1) ^ key) * 16));                  \
      qb[set_][j2] = __builtin_bit_cast(i32x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));             \
    }                                                                                                                 \
  } else {                                                                                                            \
    const bf16* as = reinterpret_cast<const bf16*>(smem_raw + (st_) * S::STAGE);                                      \
    const bf16* bs = reinterpret_cast<const bf16*>(smem_raw + (st_) * S::STAGE + S::A_BYTES);                         \
    _Pragma("unroll") for (int i = 0; i < TM; ++i) {                                                                  \
      if (A_MC) {                                                                                                     \
        fa[set_][i] = frag_from_mc_swz(as, BM, (ks_) * 16, wm0 + i * 32, lane);                                       \
      } else {                                                                                                        \
        const int r = wm0 + i * 32 + l32;                                                                             \
        fa[set_][i] = *reinterpret_cast<const bf16x8*>(as + r * BK + (((2 * (ks_) + g) ^ kc_key<BK>(r)) * 8));        \
      }                                                                                                               \
    }                                                                                                                 \
    _Pragma("unroll") for (int j2 = 0; j2 < TN; ++j2) {                                                               \
      if (B_MC) {                                                                                                     \
        fb[set_][j2] = frag_from_mc_swz(bs, BN, (ks_) * 16, wn0 + j2 * 32, lane);                                     \
      } else {                                                                                                        \
        const int r = wn0 + j2 * 32 + l32;                                                                            \
        fb[set_][j2] = *reinterpret_cast<const bf16x8*>(bs + r * BK + (((2 * (ks_) + g) ^ kc_key<BK>(r)) * 8));       \
      }                                                                                                               \
    }                                                                                                                 \
  } }
#define DP_DTL_MFMAS(set_)                                                                                            \
  _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                                      \
    _Pragma("unroll") for (int j2 = 0; j2 < TN; ++j2) {                                                               \
      if (FP8) acc[i][j2] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(qa[set_][FP8 ? i : 0], qb[set_][FP8 ? j2 : 0], acc[i][j2], 0, 0, 0, 127, 0, 127); \
      else acc[i][j2] = mfma32(fa[set_][i], fb[set_][j2], acc[i][j2]);                                                \
    }

  // Software pipeline.  All STAGES buffers are filled up front.  Fragments are fetched one k-step
  // ahead of the MFMAs that use them, also across the k-tile boundary: before the last MFMA group
  // of k-tile t every wave waits for its own fragment reads of that tile and for its share of
  // k-tile t + 1 to land, then meets the others at a barrier.  Past it, k-tile t + 1 is visible to
  // all and nobody reads k-tile t from LDS any more, so its buffer is free for k-tile t + STAGES.
  // Those copies are not issued in one burst behind the barrier (all waves would queue up at the
  // texture addresser together while the MFMA pipes drain) but spread over the k-steps of
  // k-tile t + 1, a few per MFMA group; they still run STAGES - 2 k-tiles ahead of their use.
  constexpr int PART_LAST = LOADS / KS;   // number of copies with index % KS == KS - 1
  static_assert(STAGES >= 3 && (STAGES - 1) * LOADS < 64, "pipeline shape");
  for (int t = 0; t < STAGES && t < nk; ++t) DP_DTL_ISSUE_PART(t, t, 0, 1);
  {
    const int y = min(nk, STAGES) - 1;
    static_for<STAGES>([&](auto n) { if (y == n) wait_vmcnt<n * LOADS>(); });
  }
  barrier_nofence();
  DP_DTL_FRAGS(0, 0, 0);
  // all k-tiles but the last: no branch between the fragment reads and the MFMAs, so the waits for
  // LDS data stay exact (a merge of paths with different numbers of reads in flight would make the
  // compiler wait for all of them)
  // buffers of k-tile t and its neighbours; the remainder by 3 is counted, which is 1 to 5 % faster, that by 4 is not, which is 1 to 7 % faster
  constexpr bool POW2 = (STAGES & (STAGES - 1)) == 0;
  int st = 0;
  for (int t = 0; t + 1 < nk; ++t) {
    if (POW2) st = t % STAGES;
    const int next = POW2 ? (t + 1) % STAGES : (st + 1 == STAGES ? 0 : st + 1), prev = POW2 ? (t - 1 + STAGES) % STAGES : (st == 0 ? STAGES - 1 : st - 1);
    const bool refill = t >= 1 && t - 1 + STAGES < nk;   // k-tile t - 1 + STAGES goes into the buffer k-tile t - 1 left
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks + 1 < KS) {
        DP_DTL_FRAGS(st, ks + 1, (ks + 1) & 1);
      } else {
        wait_lgkmcnt0();
        // copies younger than k-tile t + 1 that may stay in flight: whole k-tiles t + 2 .. t - 2 + STAGES
        // and the parts of k-tile t - 1 + STAGES issued so far (never more than are really there)
        const int avail = nk - 2 - t;
        if (avail >= STAGES - 2) wait_vmcnt<(STAGES - 2) * LOADS - PART_LAST>();
        else static_for<STAGES - 2>([&](auto n) { if (avail == n) wait_vmcnt<n * LOADS>(); });
        barrier_nofence();
        DP_DTL_FRAGS(next, 0, 0);
      }
      if (INTERLEAVE && ks + 1 < KS) {
        // 64-deep k-tiles: the scheduler may place one fragment read behind each MFMA instead of issuing the whole
        // batch first (6-10 % on the N = 640 projections; the 32-deep tiles lose 4 % with it and keep the batch)
        _Pragma("unroll") for (int q_ = 0; q_ < TM * TN; ++q_) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
      } else {
        __builtin_amdgcn_sched_barrier(0);
      }
      DP_DTL_MFMAS(ks & 1);
      __builtin_amdgcn_sched_barrier(0);
      if (refill) DP_DTL_ISSUE_PART(t - 1 + STAGES, prev, ks, KS);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (SEG && --seg_left == 0) close_segment();
    st = next;
  }
  if (POW2) st = (nk - 1) % STAGES;
  {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks + 1 < KS) DP_DTL_FRAGS(st, ks + 1, (ks + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
      DP_DTL_MFMAS(ks & 1);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  }
#undef DP_DTL_FRAGS
#undef DP_DTL_MFMAS
#undef DP_DTL_ISSUE_PART
  if (SEG) {
    if (!RING || seg_left != p.k_tiles_per_split) close_segment();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = total[SEG ? i : 0][SEG ? j : 0];
  }
  __syncthreads();   // every wave is done with the operand tiles before they are reused below

  float* Cw = reinterpret_cast<float*>(smem_raw) + wave * 32 * S::C_LD;
  if constexpr (KIND < 0) {
    wave_epilogue<TM, TN, WN, S::C_LD>(acc, Cw, p.epi, m0 + wm0, n0 + wn0, lane);
  } else {
    const int n = n0 + wn0 + lane % CH * 8;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) Cw[acc_row(r, g) * S::C_LD + j * 32 + l32] = acc[i][j][r];
      asm volatile("" ::: "memory");
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int row = (it * 64 + lane) / CH, m = m0 + wm0 + i * 32 + row;
        float v[8];
        pp_slab_row(&Cw[row * S::C_LD + lane % CH * 8], v);
        if (m < p.epi.M && n < p.epi.N) pp_finish<EPI>(p.epi, m, n, v, in[i][it], bias);
      }
      asm volatile("" ::: "memory");
    }
  }
}

// ------------------------------------------------------------------ bf16 / fp8 MFMA kernel, alternating wave groups
// y = x W^T on contraction-contiguous operands with the main loop of dp_gemm_pp.h.  KTAIL: K is not a multiple of the k-tile;
// chunks of the last k-tile past K are fetched from outside the buffers (zeros) in both operands.
// WALK: a workgroup takes the tiles blockIdx.x, + gridDim.x, ... and issues the first copies of the next tile before the epilogue of the present one, whose
// slabs lie behind the first stage.  A round of tiles spends 1.1 us between one workgroup and the next and 1.7 until the first k-tile is there, beside 10 us of main
// loop and 2.6 of epilogue (8-bit product of 8192 x 4608, K = 1152).  How much of the 2.8 us is gained depends on the clock, which falls as the matrix
// cores idle less.  A pass among others, against the same code with a workgroup per tile, in turn on one card and on another: that product with its
// quantisation 54.3 -> 53.5 and 55.4 -> 53.6 us (60.6 -> 53.4 together with the bias requested ahead in pp_epilogue); seven DiT blocks 32 x 256 x 1152
// 10012 -> 9813 and 10049 -> 9658; two U-Net blocks 8 x 1024 x 640 1628 -> 1622, 8 x 4096 x 320 3256 -> 3240; the convolution of the image encoder
// 10297 -> 10268 (8 x 512 x 512) and 1143 -> 1149 (384 x 328): not taken there.
template <class T> struct PpWalk {
  static constexpr size_t slab(int rows) { return (size_t)T::NW * rows * T::C_LD * 4; }
  static constexpr int RPS = T::W % 32 == 0 ? 16 : 32;
  static constexpr size_t BYTES = T::STAGE + (slab(RPS) > T::STAGE ? slab(RPS) : (size_t)T::STAGE);
  static_assert(BYTES <= 160 * 1024, "tile shape");
};
template <class T, int KIND, bool FP8, bool KTAIL, bool WALK = false>
__device__ __forceinline__ void gemm_pp_body(const GemmBf16Params& p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / T::WGN, wn = wave % T::WGN;
  const int nk = (p.K + T::BK - 1) / T::BK;
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;
  // rows past the edge are fetched from the last valid one: they only feed outputs that are never stored
  uint32_t va[2][T::LA], vb0[T::LB0], vb1[T::LB1];
  int m0, n0, n_kt = nk;      // n_kt: 0 once there is no further tile; its copies then read nothing
  auto piece_b = [&](int h, int j) { return min(wave * (h ? T::LB1 : T::LB0) + j, (h ? T::B1_BYTES : T::B0_BYTES) / 1024 - 1); };
  auto set_tile = [&](int id) {
    int tile_m, tile_n, ln = lane;
    if constexpr (WALK) asm volatile("" : "+v"(ln));      // what follows from the lane alone is formed again for each tile: it would take registers from the loop
    tile_of_block(id, p.tiles_m, p.tiles_n, p.group_m, tile_m, tile_n);
    m0 = tile_m * T::BM; n0 = tile_n * T::BN;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < T::LA; ++j) {
        const int r = pp_piece_row(wave * T::LA + j, ln), c = pp_piece_chunk(r, ln);
        va[h][j] = 2u * ((uint32_t)min(m0 + h * (T::BM / 2) + r, p.M - 1) * p.lda + c * 8);
      }
    auto offset_b = [&](int h, int j) {
      const int r = pp_piece_row(piece_b(h, j), ln), c = pp_piece_chunk(r, ln);
      const int row = KIND == PE_GEGLU1 ? h * p.epi.geglu_inner + min(n0 / 2 + r, p.epi.geglu_inner - 1) : min(n0 + h * T::BN0 + r, p.N - 1);
      return 2u * ((uint32_t)row * p.ldb + c * 8);
    };
#pragma unroll
    for (int j = 0; j < T::LB0; ++j) vb0[j] = offset_b(0, j);
#pragma unroll
    for (int j = 0; j < T::LB1; ++j) vb1[j] = offset_b(1, j);
  };
  const int k_last = p.K - (nk - 1) * T::BK;         // columns of the last k-tile
  auto tail = [&](uint32_t v, int piece, int t) {
    if (!KTAIL || t != nk - 1) return v;
    const int r = pp_piece_row(piece, lane);
    return pp_piece_chunk(r, lane) * 8 < k_last ? v : OUTSIDE;
  };
  // (of a buffer of no size nothing is read, whatever the offset)
  auto k_offset = [&](int t) { return WALK && t >= n_kt ? 0u : (uint32_t)t * (2u * T::BK); };
  auto copy_a = [&](auto hc, int t, unsigned char* dst) {
    constexpr int h = decltype(hc)::value;
    const rsrc_t r = make_rsrc(p.A, t < n_kt ? p.a_bytes : 0u);
    const uint32_t off = k_offset(t);
#pragma unroll
    for (int j = 0; j < T::LA; ++j) async_copy_16B_buf(r, tail(va[h][j], wave * T::LA + j, t), off, dst + (wave * T::LA + j) * 1024);
  };
  auto copy_b = [&](auto hc, int t, unsigned char* dst) {
    constexpr int h = decltype(hc)::value;
    const rsrc_t r = make_rsrc(p.B, t < n_kt ? p.b_bytes : 0u);
    const uint32_t off = k_offset(t);
#pragma unroll
    for (int j = 0; j < (h ? T::LB1 : T::LB0); ++j)
      async_copy_16B_buf(r, tail(h ? vb1[h ? j : 0] : vb0[h ? 0 : j], piece_b(h, j), t), off, dst + piece_b(h, j) * 1024);
  };
  typename T::acc_t acc[2][T::TM][T::TN];
  float csum[2][T::TM];
  set_tile(blockIdx.x);
  if constexpr (!WALK) {
    pp_main_loop<T, FP8, false, false, !FP8 && !(KTAIL && T::BM == 256 && T::BN == 256)>(acc, smem_raw, nk, wm, wn, wave >= 4, lane, copy_a, copy_b, false, csum);
    pp_epilogue<T, KIND, 32>(acc, smem_raw, p.epi, m0, n0, wave, wm, wn, lane, []() {});
  } else {
    const int n_tiles = p.tiles_m * p.tiles_n;
    pp_first_k_tile<T>(smem_raw, copy_a, copy_b);
    for (int id = blockIdx.x;;) {
      pp_main_loop<T, FP8, false, true, false>(acc, smem_raw, nk, wm, wn, wave >= 4, lane, copy_a, copy_b, false, csum);
      id += gridDim.x;
      int le = lane;
      asm volatile("" : "+v"(le));
      // (Without a further tile as copies of nothing: behind a branch, the compiler would have to take the shorter count of what is on its way and
      // wait for the copies before the operands of the epilogue are used.)
      pp_epilogue<T, KIND, PpWalk<T>::RPS>(acc, smem_raw + T::STAGE, p.epi, m0, n0, wave, wm, wn, le, [&]() {
        n_kt = id < n_tiles ? nk : 0;
        set_tile(min(id, n_tiles - 1));
        pp_first_k_tile<T>(smem_raw, copy_a, copy_b);
      });
      if (id >= n_tiles) break;
      lds_barrier();      // the second stage is free again
    }
    wait_vmcnt<0>();      // no copy outlives its LDS
  }
}
template <class T, int KIND, bool FP8, bool KTAIL, bool WALK = false>
__global__ void __launch_bounds__(512, 2) gemm_pp_kernel(const GemmBf16Params p) { gemm_pp_body<T, KIND, FP8, KTAIL, WALK>(p); }
// Several products of one shape, operands and outputs at fixed distances (elements): problem blockIdx.y.
struct GemmStrides { long a, b, out; };
template <class T, int KIND, bool KTAIL>
__global__ void __launch_bounds__(512, 2) gemm_pp_strided_kernel(GemmBf16Params p, const GemmStrides d) {
  const long i = blockIdx.y;
  p.A += i * d.a; p.B += i * d.b;
  if constexpr (KIND == PE_F32) p.epi.out32 += i * d.out;
  else p.epi.out += i * d.out;
  gemm_pp_body<T, KIND, false, KTAIL>(p);
}

// y = x W^T on 64x64 tiles whose NW waves share the contraction instead of the tile: wave w computes the whole tile over the k-tiles
// w, w + NW, ... of the workgroup's range, from a stage of LDS of its own, and the NW partial tiles are added at the end, in wave order.
// Why: of a 64x64 tile split 2x2 among four waves, each reads 2 fragments per MFMA (32 KB read and 16 KB written per k-tile) and waits at a barrier
// a k-tile (0.15 to 0.185 us on the ring, tile64_us); here a k-tile is read once (16 KB, 4 fragments for 4 MFMAs) and no wave ever waits for another before the
// end.  A wave holds one k-tile in registers and one on its way to LDS, two where a CU has a single workgroup of 64x64 (the stages then leave no
// room for another); the other waves of the CU hide the latency.  What a launch of few tiles spends beside that is its beginning and
// end: 77 x 3072, K = 768 took 6.6 us, 1.0 until the copies were issued, 2.1 for three k-tiles, 2.5 to add up 32 rows at a time with every
// epilogue in one kernel.  With a kernel per kind of epilogue, its operands requested ahead and 64 rows at a time: 7.4 -> 6.3 us a launch,
// 1024 x 1152, K = 1152 / 4608: 10.2 -> 9.1 / 20.2 -> 18.9; steps of the text encoder on one sample 525 -> 470 us, of seven DiT blocks
// 4 x 256 x 1152 2287 -> 2163, of a U-Net block 2 x 513 x 1280 (three passes, two micro-batches) 1321 -> 1238.
// What bounds it is fetching operands, about 20 TB/s over all CUs, so the widest tile that still gives one workgroup per CU is taken (kWave).
// Measured (M x N, K; us, 64x64 tiles split 2x2 or 128x128 ones with split-K before): 1026 x 1280, 3840: 27 -> 19, 10240: 66 -> 40;
// 1024 x 1152, 4608: 32 -> 20; 2048 x 1152, 4608: 37 -> 30; 924 x 768, 3072: 21 -> 12.5.
// Outputs of few tiles leave most CUs without one, and a CU fetches about 0.1 KB per ns however many tiles there are: 32 rows with eight waves, which
// have as much on its way to LDS in the first round trip as four of 64x64, on the widest of 32, 64, 96 columns that gives every CU at most one tile
// (us, 64x64 tiles with four waves, split further where it paid -> 32 rows: 80 x 2304, K = 768 6.2 -> 3.9, K = 3072 and 768 columns 10.0 -> 6.6, 160 x 3072, 768
// 6.4 -> 5.0, 312 x 768, 3072 11.9 -> 7.0, 616 x 768, 768 6.3 -> 4.9, 928 x 768, 768 6.4 -> 5.9; with 12 or 16 waves, or two k-tiles each on its way, no
// better).  The text encoder on one sample 423 -> 337 us.
// ST: k-tiles of a wave on their way to LDS.  RP: rows of the tile that are added up at a time.
template <int NW_, int TM_, int TN_, int ST_ = 1>
struct WaveTile {
  static constexpr int NW = NW_, TM = TM_, TN = TN_, ST = ST_, BM = 32 * TM, BN = 32 * TN, LD = BN + 4, A_BYTES = BM * 128, REGION = (BM + BN) * 128;
  static constexpr int RP = TM == 1 || (TN == 3 && TM == 2) ? 32 : 64, GROUPS = RP * BN / 8, ITEMS = (GROUPS + NW * 64 - 1) / (NW * 64);      // groups of eight columns of a pass, and per thread
  static constexpr size_t SLAB = (size_t)NW * RP * LD * 4, STAGES = (size_t)NW * ST * REGION, BYTES = STAGES > SLAB ? STAGES : SLAB;
  static_assert(BM % RP == 0 && BYTES <= 160 * 1024, "tile shape");
};
// B_MC: dx = dy W with the weights as they are stored, [contraction][columns]; their tile is read with the transposing LDS load.  Against
// a transposed copy (us): on average over 64 to 8192 rows none more on 128x128 tiles, 2 % on 64x64, 4 % on 128x96, 32x32 and 32x64, 8 to 10 % on 64x96 and 32x96, whose rows of 192 bytes begin inside cache lines (1024 x 1152, K = 4608 19.5
// and 20.8; 1026 x 1280, K = 3840 18.1 and 19.9), which is less than the copy costs (4 N K bytes at 6.3 TB/s: 3.4 and 3.1) but for a few (1026 x 1024, K = 8192 31.0 and 39.3
// beside 5.3; 2560 x 512, K = 4096 17.6 and 20.3 beside 1.3): a U-Net block 2 x 513 x 1280, two micro-batches of
// three passes 1279 -> 1256, seven DiT blocks 4 x 256 x 1152 2163 -> 2150.
// NORM (32 rows, contractions up to 1024): the rows operand is the LayerNorm of fp32 rows, formed here instead of by a launch of its own, which on few rows is a
// chain of two memory round trips and the gap between two launches.  Every wave normalises four rows while its first k-tile of weights is on its way; the rows lie
// in LDS k-tile by k-tile, the waves' stages hold weights alone.  Every workgroup of a row of tiles does so again: 98 KB of rows from the L2 for 24 to 72 of them.
template <class T, int KIND, bool B_MC = false, bool NORM = false>
__global__ void __launch_bounds__(T::NW * 64, T::TM * T::TN == 1 ? 4 : (T::TM * T::TN <= 6 ? 2 : 1)) gemm_wave_kernel(const GemmBf16Params p) {
  constexpr int NW = T::NW, TM = T::TM, TN = T::TN, LD = T::LD, ST = T::ST, COPIES = 4 * ((NORM ? 0 : TM) + TN), REGION = NORM ? T::BN * 128 : T::REGION, OFF_B = NORM ? 0 : T::A_BYTES;
  static_assert(!NORM || (TM == 1 && !B_MC && ST == 1 && NW == 8), "normalised rows");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, l32 = lane & 31;
  int tile_m, tile_n;
  tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tile_m, tile_n);
  const int m0 = tile_m * T::BM, n0 = tile_n * T::BN;
  const int kt_begin = blockIdx.z * p.k_tiles_per_split, kt_end = min(p.K / 64, kt_begin + p.k_tiles_per_split);
  uint32_t va[4 * TM], vb[4 * TN];
#pragma unroll
  for (int j = 0; j < 4 * TM; ++j) {
    const int r = 8 * j + (lane >> 3), c = (lane & 7) ^ kc_key<64>(r);
    va[j] = 2u * ((uint32_t)min(m0 + r, p.M - 1) * p.lda + c * 8);
  }
#pragma unroll
  for (int j = 0; j < 4 * TN; ++j) {
    if constexpr (B_MC) {
      constexpr int CHUNKS = T::BN / 8;
      const int o = 64 * j + lane, k = o / CHUNKS, c = pp_mc_swz<T::BN>(o % CHUNKS, k);
      vb[j] = 2u * ((uint32_t)k * p.ldb + min(n0 + c * 8, p.N - 8));
    } else {
      const int r = 8 * j + (lane >> 3), c = (lane & 7) ^ kc_key<64>(r);
      vb[j] = 2u * ((uint32_t)min(n0 + r, p.N - 1) * p.ldb + c * 8);
    }
  }
  uint32_t ob[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) ob[j] = B_MC ? pp_mc_offset<T::BN>(32 * j, lane) : 0;
  unsigned char* own = smem_raw + (NORM ? p.K * (2 * T::BM) : 0) + wave * (ST * REGION);
  // copies of k-tile t (past the last one: issued all the same, since the waits count them, from outside the buffers)
  auto issue = [&](int t, int stage) {
    const bool in = t < kt_end;
    const rsrc_t ra = make_rsrc(p.A, in ? p.a_bytes : 0u), rb = make_rsrc(p.B, in ? p.b_bytes : 0u);
    const uint32_t off = in ? (uint32_t)t * 128u : 0u, off_b = B_MC ? off * (uint32_t)p.ldb : off;
    unsigned char* dst = own + stage * REGION;
#pragma unroll
    for (int j = 0; j < (NORM ? 0 : 4 * TM); ++j) async_copy_16B_buf(ra, va[j], off, dst + j * 1024);
#pragma unroll
    for (int j = 0; j < 4 * TN; ++j) async_copy_16B_buf(rb, vb[j], off_b, dst + OFF_B + j * 1024);
  };
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  auto k_tile = [&](int t, int stage) {
    bf16x8 fa[4][TM], fb[4][TN];
    u32x2 raw[4][TN][2];
    wait_vmcnt<(ST - 1) * COPIES>();
    const unsigned char* src = own + stage * REGION;
    const unsigned char* rows = NORM ? smem_raw + t * (T::BM * 128) : src;
    if constexpr (B_MC) {
      static_for<4>([&](auto ks) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const uint32_t at = lds_address(src) + OFF_B + ob[j];
          lds_read_tr_raw<ks * 32 * T::BN>(raw[ks][j][0], at);
          lds_read_tr_raw<(ks * 16 + 4) * 2 * T::BN>(raw[ks][j][1], at);
        }
      });
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int r = 32 * i + l32;
        fa[ks][i] = *reinterpret_cast<const bf16x8*>(rows + r * 128 + ((2 * ks + g) ^ kc_key<64>(r)) * 16);
      }
#pragma unroll
      for (int j = 0; j < (B_MC ? 0 : TN); ++j) {
        const int r = 32 * j + l32;
        fb[ks][j] = *reinterpret_cast<const bf16x8*>(src + OFF_B + r * 128 + ((2 * ks + g) ^ kc_key<64>(r)) * 16);
      }
    }
    wait_lgkmcnt0();
    if constexpr (B_MC) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          lds_arrived(raw[ks][j][0]); lds_arrived(raw[ks][j][1]);
          fb[ks][j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(raw[ks][j][0], raw[ks][j][1], 0, 1, 2, 3));
        }
    }
    if (ST > 1 || t + NW < kt_end) issue(t + ST * NW, stage);
    __builtin_amdgcn_sched_barrier(0);      // (all copies before the products: they are what the next k-tile waits for)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma32(fb[ks][j], fa[ks][i], acc[i][j]);      // transposed: a lane gets four neighbouring columns of a row
  };
  int t = kt_begin + wave;
  if constexpr (NORM) {
    constexpr int ROWS = T::BM / NW;
    auto normalise = [&](auto ncc) {
      constexpr int NC = decltype(ncc)::value;      // chunks of four columns a lane: K = 256 NC
      f32x4 x[ROWS][NC];
      bf16x4 ga[NC], be[NC];
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        const float* row = p.norm_x + (size_t)min(m0 + wave * ROWS + i, p.M - 1) * (256 * NC) + 4 * lane;
#pragma unroll
        for (int c = 0; c < NC; ++c) x[i][c] = *reinterpret_cast<const f32x4*>(row + 256 * c);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) { ga[c] = *reinterpret_cast<const bf16x4*>(p.norm_gamma + 256 * c + 4 * lane); be[c] = *reinterpret_cast<const bf16x4*>(p.norm_beta + 256 * c + 4 * lane); }
      __builtin_amdgcn_sched_barrier(0);      // (the rows first: what is issued behind them need not be waited for with them)
      issue(t, 0);
      __builtin_amdgcn_sched_barrier(0);
      // the arithmetic of ln_fwd_kernel, which has 64 lanes a row for these widths in the encoder: the same bits
      float mu[ROWS], rs[ROWS];
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        mu[i] = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int u = 0; u < 4; ++u) mu[i] += x[i][c][u];
      }
#pragma unroll
      for (int i = 0; i < ROWS; ++i) mu[i] = wave_sum(mu[i]) / (256 * NC);
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        rs[i] = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            x[i][c][u] -= mu[i];
            rs[i] = fmaf(x[i][c][u], x[i][c][u], rs[i]);
          }
      }
#pragma unroll
      for (int i = 0; i < ROWS; ++i) rs[i] = rsqrtf(wave_sum(rs[i]) / (256 * NC) + p.norm_eps);
      const int k_tile = lane / 16, chunk = lane % 16 / 2;      // of the first chunk; the next one lies four k-tiles on
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        const int r = wave * ROWS + i;
        unsigned char* dst = smem_raw + k_tile * (T::BM * 128) + r * 128 + (chunk ^ kc_key<64>(r)) * 16 + lane % 2 * 8;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          bf16x4 o;
#pragma unroll
          for (int u = 0; u < 4; ++u) o[u] = (bf16)fmaf(x[i][c][u] * rs[i], (float)ga[c][u], (float)be[c][u]);
          *reinterpret_cast<bf16x4*>(dst + c * (4 * T::BM * 128)) = o;
        }
      }
    };
    switch (p.K / 256) {
      case 1: normalise(std::integral_constant<int, 1>()); break;
      case 2: normalise(std::integral_constant<int, 2>()); break;
      case 3: normalise(std::integral_constant<int, 3>()); break;
      default: normalise(std::integral_constant<int, 4>());
    }
    lds_barrier();
  } else {
#pragma unroll
    for (int i = 0; i < ST; ++i) issue(t + i * NW, i);
  }
#pragma unroll 1
  for (; t < kt_end; t += ST * NW) {
#pragma unroll
    for (int i = 0; i < ST; ++i)
      if (i == 0 || t + i * NW < kt_end) k_tile(t + i * NW, i);
  }
  // The partial tiles meet in LDS, RP rows at a time; what the epilogue reads beside them is requested before.
  float* slab = reinterpret_cast<float*>(smem_raw);
  constexpr int CH = T::BN / 8;
#pragma unroll
  for (int pass = 0; pass < T::BM / T::RP; ++pass) {
    PpIn<KIND> in[T::ITEMS];
    bf16x8 bias[T::ITEMS];
#pragma unroll
    for (int it = 0; it < T::ITEMS; ++it) {
      const int x = min(it * NW * 64 + tid, T::GROUPS - 1), m = m0 + pass * T::RP + x / CH, n = n0 + x % CH * 8;
      pp_load<KIND>(p.epi, m, n, in[it]);
      bias[it] = KIND != PE_F32 && p.epi.bias ? *reinterpret_cast<const bf16x8*>(p.epi.bias + min(n, p.epi.N - 8)) : zero8();
    }
    if (pass == 0) wait_vmcnt<0>();      // (copies from outside the buffers may still be under way to where the slab will be)
    __syncthreads();
#pragma unroll
    for (int i = 0; i < T::RP / 32; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4 v;
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = acc[pass * (T::RP / 32) + i][j][4 * q + u];
          *reinterpret_cast<f32x4*>(slab + (wave * T::RP + 32 * i + l32) * LD + 32 * j + 8 * q + 4 * g) = v;
        }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < T::ITEMS; ++it) {
      const int x = it * NW * 64 + tid, row = x / CH, c = x % CH * 8, m = m0 + pass * T::RP + row, n = n0 + c;
      if (T::GROUPS % (NW * 64) != 0 && x >= T::GROUPS) continue;
      float v[8], bv[8];
      const float* src = slab + row * LD + c;
      *reinterpret_cast<f32x4*>(&v[0]) = *reinterpret_cast<const f32x4*>(src);
      *reinterpret_cast<f32x4*>(&v[4]) = *reinterpret_cast<const f32x4*>(src + 4);
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        const f32x4 y0 = *reinterpret_cast<const f32x4*>(src + w * T::RP * LD), y1 = *reinterpret_cast<const f32x4*>(src + w * T::RP * LD + 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) { v[u] += y0[u]; v[4 + u] += y1[u]; }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) bv[u] = (float)bias[it][u];
      if (m < p.epi.M && n < p.epi.N) pp_finish<KIND>(p.epi, m, n, v, in[it], bv);
    }
  }
}

// Second pass of a split-K GEMM with a storage-dtype output: sums the fp32 partial tiles in ascending
// split order (fixed order, run-to-run identical) and applies the GEMM's epilogue to the sums.  One thread
// per 8 consecutive columns of a row.
__global__ void __launch_bounds__(256) reduce_epilogue_kernel(EpiParams<bf16> e, const float* __restrict__ partial, int splits) {
  const int per_row = e.N / 8;
  const size_t idx = blockIdx.x * (size_t)256 + threadIdx.x;
  if (idx >= (size_t)e.M * per_row) return;
  const int m = (int)(idx / per_row), n = (int)(idx % per_row) * 8;
  const float* p = partial + (size_t)m * e.N + n;
  const size_t plane = (size_t)e.M * e.N;
  float v[8];
  *reinterpret_cast<f32x4*>(&v[0]) = *reinterpret_cast<const f32x4*>(p);
  *reinterpret_cast<f32x4*>(&v[4]) = *reinterpret_cast<const f32x4*>(p + 4);
  for (int z = 1; z < splits; ++z) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(p + z * plane), b = *reinterpret_cast<const f32x4*>(p + z * plane + 4);
#pragma unroll
    for (int t = 0; t < 4; ++t) { v[t] += a[t]; v[4 + t] += b[t]; }
  }
  epi_vec8(e, m, n, v);
}

// ------------------------------------------------------------------ host side
template <typename T>
static EpiParams<T> make_epi(const GemmArgs& a) {
  EpiParams<T> e;
  e.M = a.M; e.N = a.N;
  e.out = (T*)a.out; e.ldo = a.ldo;
  e.out32 = a.out_f32; e.ldo32 = a.ldo32; e.accumulate = a.accumulate;
  e.partial = nullptr;
  e.bias = (const T*)a.bias;
  e.pre_out = (T*)a.pre_out; e.ld_pre = a.ld_pre;
  e.act = a.act;
  e.dact_pre = (const T*)a.dact_pre; e.ld_dact = a.ld_dact; e.dact_kind = a.dact_kind;
  e.gate = (const T*)a.gate; e.gate_ld = a.gate_ld; e.rows_per_batch = a.rows_per_batch > 0 ? a.rows_per_batch : 1;
  e.residual = a.residual; e.ld_res = a.ld_res; e.residual_f32 = a.residual_f32; e.out_fused_f32 = a.out_fused_f32;
  e.geglu = a.geglu; e.geglu_inner = a.geglu_inner; e.geglu_u = (const T*)a.geglu_u; e.ld_geglu = a.ld_geglu;
  e.out_scale = 1.0f;
  return e;
}

// Bytes a bf16 GEMM launch has to move once: both operands, the result in its output type, and every
// tensor its fused epilogue reads or writes beside it (fp32 residual in and out, the saved projection next
// to a GeGLU output, the saved pre-activation of a backward).  Split-K partial sums are not counted.
static double gemm_tensor_bytes(const GemmArgs& a) {
  const double mn = (double)a.M * a.N;
  double b = 2.0 * ((double)a.M * a.K + (double)a.N * a.K);
  if (a.out_f32) return b + 4.0 * mn * (a.accumulate ? 2.0 : 1.0);
  if (a.geglu == 1) return b + 2.0 * (double)a.M * a.geglu_inner + (a.pre_out ? 2.0 * mn : 0.0);
  if (a.geglu == 2) return b + 2.0 * 2.0 * (double)a.M * 2.0 * a.geglu_inner;      // u read, du written: [M, 2 inner] each
  b += mn * (a.out_fused_f32 ? 4.0 : 2.0);
  if (a.pre_out) b += 2.0 * mn;
  if (a.dact_pre) b += 2.0 * mn;
  if (a.residual) b += mn * (a.residual_f32 ? 4.0 : 2.0);
  return b;
}

// Group height of the workgroup-to-tile map.  An XCD's contiguous share of the tiles spans 1 / k of a group
// when k XCDs share one: the row operand's panels of that group are then fetched by k L2s and each L2 fetches
// 1 / k of the column operand, k * (row operand bytes) + (8 / k) * (column operand bytes) in total, least at
// k = sqrt(8 * cols / rows).  Narrow outputs (N <= ~0.25 M: the N = 640 and 1152 projections) want k = 1, whole
// tile-rows per XCD, which halves the fetches of their large row operand against the fixed 8 tile-rows used
// before; wide ones (N = 5120) keep two XCDs per group.  Measured on cfg2 (L2 fetch bytes per launch, rocprofv3
// FETCH_SIZE): 256x128x64 projections 65 -> 47 MB, weight-gradient GEMMs 119 -> 94 MB; step time -0.3 to -1 %.
static int choose_group_m(const GemmArgs& a, int tiles_m, int tiles_n) {
  const double rows = a.M, cols = a.N;
  const double ks = std::sqrt(8.0 * cols / rows);
  const int k = ks < 1.41 ? 1 : (ks < 2.83 ? 2 : (ks < 5.66 ? 4 : 8));
  const long n = (long)tiles_m * tiles_n, ppx = (n + 7) / 8;
  const long g = (k * ppx + tiles_n / 2) / tiles_n;
  return (int)std::max<long>(1, std::min<long>(g, tiles_m));
}

static int pp_kind(const GemmArgs& a);

// Tile configurations of the bf16 kernel.
struct TileCfg { int bm, bn, bk, waves; };
static const TileCfg kCfgs[] = {
    {128, 128, 64, 4},   // 0: two workgroups per CU; small or ragged problems
    {256, 128, 64, 8},   // 1
    {256, 256, 64, 8},   // 2: least LDS and L2 traffic per FLOP; large problems
    {128, 256, 64, 8},   // 3
    {256, 128, 32, 8},   // 4: shallower k-tile, two workgroups per CU
    {128, 128, 32, 4},   // 5
};
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);
constexpr int kCUs = 256;

// Split-K factor of the fp32-output (weight-gradient) GEMMs: the largest power of two that keeps every
// workgroup of the launch resident at once (`slots` = CUs x workgroups per CU of the configuration), with
// at least 8 64-deep k-tiles per split and at most 32 partial sums to reduce.  A launch that spills into a
// second round loses what the extra splits gained (90 tiles of 256x256, one per CU: 2 splits run 10 %
// faster than 4).  (A stage's weight gradients go through gemm_dw.hip, whose plan covers a whole block.)
static int choose_splits(long tiles, int kt, int slots) {
  const long cap = std::min<long>(std::min<long>(slots / std::max<long>(tiles, 1), kt / 8), 32);
  int s = 1;
  while (2 * s <= cap) s *= 2;
  return s;
}

// Split-K factor of a GEMM with a storage-dtype output (second pass: reduce_epilogue_kernel).  It pays
// where a few tiles would each walk the contraction alone while most CUs idle: the frozen encoder's
// projections on a partial batch (6 to 72 tiles of 128x128, K = 768 or 3072).  Measured on MI355X, encoder
// forward in samples/s without and with it: 1074 -> 1450 (slices of 1 sample), 4118 -> 5224 (4), 15881 ->
// 18057 (16).  The second pass costs a launch and the partial sums' traffic, so a short contraction
// (K < 2048) is split only up to 48 tiles (at 54 and 72 tiles it lost 9 %), a long one up to 96 (at 120
// tiles, 64 samples, the gain is cancelled).  At least 6 64-deep k-tiles per split; 3 or 12 measured no better.
static int choose_splits_epi(long tiles, int kt) {
  if (kt < 12 || tiles > (kt >= 32 ? 96 : 48)) return 1;
  const long cap = std::min<long>(std::min<long>(kCUs / std::max<long>(tiles, 1), kt / 6), 16);
  int s = 1;
  while (2 * s <= cap) s *= 2;
  return s;
}

// 64x64 tiles, up to 512 on the ring of four buffers (us, K = 768 / 4608: 48 tiles 5.3 / 14.5, 256 5.9 / 16.1, 288 7.6 / 26.3).  One a CU has 64 KB on its way, half of what
// the waves that share a contraction have, and takes 0.185 us a k-tile and not 0.15 where the weights come from memory, as a frozen layer's do (two parts of 308 x 1024, K = 4096
// 11.6 us in the text encoder, 8.9 by themselves).  More of them: 0.5 us a k-tile per 512 (32768 of them with two k-tiles each: 165 us; 256x256 tiles 90).
static float tile64_many_us(long tiles, int kt) { return 0.2f + (float)tiles / 512.0f * (1.57f + 0.5f * (float)kt); }
static float tile64_us(long tiles, int kt, int z) {
  tiles *= z; kt = (kt + z - 1) / z;
  if (tiles <= 256) return 3.4f + 0.002f * (float)tiles + (float)kt * (0.185f + 0.00008f * (float)tiles);
  const float some = 3.9f + (float)kt * (0.26f + 0.0002f * (float)tiles);
  return tiles <= 512 ? some : std::max(some, tile64_many_us(tiles, kt));
}
// The same where the tile decides in which order an output's products are added: the times of the loop before the ring.  With the ring's own times some products go
// from waves that share the contraction to 64x64 tiles (616 x 1280, 616 x 2304, 308 x 3072, K = 768; 1232 x 1280, K = 1024), which moves everything behind them by
// bf16 rounding.  What that order costs, us, these times and the ring's: U-Net blocks 8 x 1024 x 640 1612 / 1610, 8 x 256 x 1280 1280 / 1279; text encoder, weights from memory, of
// width 768 on 4 / 6 / 8 samples 466 / 571 / 574 and 462 / 575 / 588, of width 512 on 6 / 8 384 / 439 and 377 / 424, of width 1024 on 4 / 6 / 8 564 / 644 / 772 and 561 / 640 / 774;
// slice after slice of a batch, of width 768 on 4 / 8 414 / 510 and 397 / 508, of width 512 on 8 / 16 431 / 511 and 412 / 507, of width 1024 on 4 / 8 553 / 754 and 552 / 757.
static float tile64_choice_us(long tiles, int kt, int z) {
  tiles *= z; kt = (kt + z - 1) / z;
  const float some = 4.0f + (float)kt * (tiles <= 128 ? 0.31f : 0.39f);
  return tiles <= 512 ? some : std::max(some, tile64_many_us(tiles, kt));
}
// 128x128 tiles, eight waves.  heavy: an epilogue with an activation, which nothing overlaps.
static float tile128_us(long tiles, int kt, bool heavy) {
  return (float)((tiles + kCUs - 1) / kCUs) * ((heavy ? 5.5f : 4.0f) + (float)kt * (0.40f + 0.0004f * (float)std::min<long>(tiles, kCUs)));
}
// The pass that adds z partial results; ln: and does the LayerNorm that would otherwise be a launch of its own.
static float reduce_us(int rows, int N, int z, bool ln) { return (ln ? 0.5f : 5.0f) + (float)(z + 2) * (float)rows * (float)N * 1.5e-6f; }

static bool heavy_epilogue(const GemmArgs& a) { return a.act || a.dact_pre || a.geglu; }

// Split-K factor of a storage-dtype GEMM on 128x128 tiles (configuration 13) and its estimated time in us: rounds of 256
// workgroups plus, where it is split, a second launch and the partial sums' traffic.  A stage on a small local batch (1024 rows,
// 72 tiles, contractions of 3456 or 4608) spends 28-36 us in one of these projections unsplit, 22-27 us split by 3.  ln: the
// second launch also does the LayerNorm that would otherwise be one of its own.
static int splits_128(int rows, int N, int K, bool ln, bool heavy, float* us) {
  const long tiles = (long)((rows + 127) / 128) * ((N + 127) / 128);
  const int kt = K / 64;
  int best = 1;
  for (int s = 1; s <= 8 && (s == 1 || kt / s >= 6); ++s) {
    const float t = tile128_us(tiles * s, (kt + s - 1) / s, heavy && s == 1) + (s > 1 ? reduce_us(rows, N, s, ln) : 0.0f);
    if (s == 1 || t < *us) { best = s; *us = t; }
  }
  return best;
}


// Tiles whose waves share the contraction (gemm_wave_kernel): fixed part of a tile, which grows a little with the number of tiles, and the time
// of a k-tile of the workgroup, one wave's divided by the waves, each of which waits for memory; two: the same for 257 to 512 tiles, which 64x64, 64x96 and 32x32 run two a CU side by
// side, 32x64 and 32x96, whose buffers fill a CU, one after the other.  us,
// fitted on MI355X over 77..4928 rows, 640..10240 columns, contractions of 640..10240 (within 8 %; two_per_kt, which grows with the contraction, on the dear side);
// 32 rows over 80..1232 rows, 512..4096 columns, contractions of 512..4096.
struct WaveCost { int bm, bn; float fixed, per_tile, per_kt, per_kt_tile, two_fixed, two_per_kt; };
static const WaveCost kWave[] = {{64, 64, 3.6f, 0.005f, 0.173f, 0.f, 4.1f, 0.36f}, {64, 96, 3.7f, 0.0075f, 0.212f, 0.f, 5.6f, 0.50f},
                                 {128, 96, 6.8f, 0.005f, 0.255f, 0.0003f, 0.f, 0.f}, {128, 128, 8.0f, 0.015f, 0.325f, 0.0002f, 0.f, 0.f},
                                 {32, 32, 2.6f, 0.0013f, 0.083f, 0.f, 3.1f, 0.166f}, {32, 64, 3.1f, 0.0013f, 0.1245f, 0.f, 5.0f, 0.25f}, {32, 96, 3.3f, 0.0017f, 0.171f, 0.f, 5.5f, 0.34f}};
// Estimated time; splits: parts the contraction is cut into beyond the waves of a workgroup, where few tiles would each walk a long one.
static float wave_us(const WaveCost& c, int rows, int N, int K, bool may_split, bool ln, int* splits) {
  const int kt = K / 64;
  const int tiles_n = (N + c.bn - 1) / c.bn;
  const int tiles = (int)std::min<long>((long)((rows + c.bm - 1) / c.bm) * tiles_n, 1 << 24);
  auto time = [&](int z) {
    const int n = tiles * z, part = (kt + z - 1) / z;
    if (c.bm == 32 && n > 2 * kCUs) return 1e9f;      // a third round, of which the terms know nothing; 64 rows are as good or better (8300 x 104, K = 4096: 32.2 us, 64x64 24.3, 128x128 20.2)
    const float reduce = z > 1 ? reduce_us(rows, N, z, ln) : 0.f;
    if (n > kCUs && c.two_fixed > 0.f) return std::max(1.0f, (float)n / 512.0f) * (c.two_fixed + (float)part * c.two_per_kt) + (n > 2 * kCUs ? 1.0f : 0.f) + reduce;
    const float live = (float)std::min(n, kCUs);
    return (float)((n + kCUs - 1) / kCUs) * (c.fixed + c.per_tile * live + (float)part * (c.per_kt + c.per_kt_tile * live)) + reduce;
  };
  float best = 0.f;
  *splits = 1;
  for (int z = 1; z <= 8 && (z == 1 || (may_split && kt / z >= 4 && tiles * z <= kCUs)); ++z) {
    const float t = time(z);
    if (z == 1 || t < best) { best = t; *splits = z; }
  }
  return best;
}
// The same when the choice is made for `choice_rows` rows (GemmArgs::choice_rows) but M rows are computed.
size_t gemm_epi_splitk_ws_bytes_for(int M, int N, int K, int choice_rows) {
  float us;
  int sp = 1;
  for (const bool ln : {false, true})
    for (const bool heavy : {false, true}) sp = std::max(sp, splits_128(choice_rows, N, K, ln, heavy, &us));
  for (const WaveCost& c : kWave)
    for (const bool ln : {false, true}) {
      int w;
      wave_us(c, choice_rows, N, K, true, ln, &w);
      sp = std::max(sp, w);
    }
  const int shapes[][2] = {{64, 64}, {128, 128}, {256, 128}, {256, 256}};
  for (const auto& t : shapes) {
    const long tiles = (long)((choice_rows + t[0] - 1) / t[0]) * ((N + t[1] - 1) / t[1]);
    sp = std::max(sp, choose_splits_epi(tiles, K / 64));
  }
  return sp > 1 ? (size_t)sp * M * N * sizeof(float) : 0;
}

size_t gemm_epi_splitk_ws_bytes(int M, int N, int K) { return gemm_epi_splitk_ws_bytes_for(M, N, K, M); }
// Waves and choose_splits_epi split up to a number of tiles; splits_128 while the reduction of two parts costs less than the most a split can
// save, one round of tiles.
int gemm_epi_split_rows(int N, int K) {
  const int kt = K / 64;
  long rows = 0;
  auto tiles = [&](int most, int bm, int bn) { rows = std::max(rows, (long)(most / ((N + bn - 1) / bn)) * bm); };
  if (kt >= 8) for (const WaveCost& c : kWave) tiles(kCUs / 2, c.bm, c.bn);
  if (kt >= 12) {
    tiles(96, 64, 64); tiles(96, 128, 128); tiles(96, 256, 128); tiles(96, 256, 256);
    rows = std::max(rows, (long)(tile128_us(kCUs, kt, true) / (reduce_us(1000, N, 2, true) - 0.5f) * 1000.f) + 1);
  }
  return (int)std::min<long>(rows, 1L << 30);
}

// Picks the tile configuration (indices as in launch_gemm's switch), from sweeps of all GEMM shapes of
// the five workloads on MI355X:
//  - y = x W^T (both operands K-contiguous; also dx = dy W on transposed weight copies): the tile with the least
//    estimated time, among alternating wave groups, waves that share the contraction and the plain direct-to-LDS ones;
//  - dx = dy W with W as stored: waves that share the contraction where the transposed copy's product would run on them
//    (gemm_takes_stored_weight); else 256x256 direct-to-LDS tiles when they fill the CUs, or the register-staged kernel;
//  - dW = dy^T x (both operands read through the transposing LDS load): register-staged 128x128 tiles,
//    two workgroups per CU; 256x256 direct-to-LDS tiles for large M and N.
static int choose_cfg(int M, int N, int K, bool a_mc, bool b_mc, bool dtl_ok, bool pp_ok, bool allow16 = true, bool may_split = false, bool ln = false, bool wave_ok = false, bool heavy = false, bool geglu_fwd = false, bool onto_f32 = false) {
  const long t256x256 = (long)((M + 255) / 256) * ((N + 255) / 256);
  const long t256x128 = (long)((M + 255) / 256) * ((N + 127) / 128);
  const bool dtl32 = dtl_ok && K % 32 == 0, dtl64 = dtl_ok && K % 64 == 0;
  pp_ok = pp_ok && dtl_ok;
  if (a_mc) return (dtl32 && b_mc && t256x256 >= 80) ? 6 : 0;
  if (!b_mc) {
    // y = x W^T on contraction-contiguous operands.
    // A few hundred rows and a short contraction (the frozen encoder's projections on a partial batch): 64x64 tiles give
    // 4x the workgroups of 128x128 ones, each with a quarter of the work per k-tile, and no split-K pass is needed.
    // Measured on the text encoder (samples/s at slices of 1 / 4 / 16): 1538 / 5617 / 19148 -> 1733 / 6490 / 20040; with more
    // 128x128 tiles than the limits below the larger tiles win again (16 samples, K = 3072: -6 % with 64x64 tiles).
    if (dtl64 && !allow16 && !geglu_fwd && (long)((M + 127) / 128) * ((N + 127) / 128) <= (K <= 1024 ? 100 : 24)) return 15;
    // Otherwise the tile with the least estimated time: rounds over the 256 CUs x (fixed part of a tile + k-tiles x time of
    // one), both in us, fitted on MI355X over projections of 1024..32768 rows, 320..5120 columns, contractions of
    // 320..5120.  The alternating-group tiles hold one workgroup per CU; which of their widths wins is mostly a matter of how
    // full the last round is (8192 x 4608: 576 tiles of 256x256 are 2.25 rounds, 768 of 256x192 exactly 3 shorter ones).
    // (The times are those of one k-tile a round of the loop; with two, up to 256 tiles of 256x128 take 0.61 us a k-tile.  The choice has not been fitted to that.)
    // The fused GeGLU forward is chosen among the tiles that have it (100 x 9216 on 128x128 tiles of eight waves instead of four 19.4 -> 15.7 us,
    // 2052 x 7680 on 256x128 ones instead of 256x256 62.0 -> 59.5, 4050 x 6144 the same way 58.6 -> 60).
    struct Cand { int idx, bm, bn; float fixed, per_kt; bool pp, need64; };
    static const Cand cands[] = {{17, 256, 256, 5.0f, 1.30f, true, false}, {19, 256, 192, 5.0f, 1.05f, true, false}, {20, 256, 160, 5.5f, 0.99f, true, false},
                                 {18, 256, 128, 5.0f, 0.72f, true, false}, {13, 128, 128, 0.f, 0.f, false, true}, {8, 128, 128, 5.0f, 0.75f, false, false},
                                 {6, 256, 256, 5.0f, 1.70f, false, false}, {9, 256, 128, 5.0f, 0.85f, false, true}};
    // A product that is added to an fp32 tensor reads and writes 8 bytes an output.  Tiles of 128 rows do so when all of them are at their ends together, the
    // 256-row ones in their rounds, the waves that share a contraction request what they read ahead (4928 x 768 in the text encoder, us: 128x128, K = 768 / 3072
    // 10.7 -> 16.5 / 31 -> 38; 256x128, K = 768 13.5 -> 17.5; 128x128 of such waves, K = 3072 30.7 -> 31.8).  Text encoder of
    // width 768 on 48 / 56 / 64 / 66 / 72 samples: 1336 / 1576 / 1672 / 1700 / 1883 us without these terms, 1307 / 1472 / 1566 / 1592 / 1887 with them.
    const float outputs = onto_f32 ? (float)M * (float)N * 1e-6f : 0.f;
    int best = -1;
    float best_cost = 0.f;
    auto consider = [&](int idx, float cost) { if (best < 0 || cost < best_cost) { best = idx; best_cost = cost; } };
    for (const Cand& c : cands) {
      if (c.pp ? !pp_ok : (c.need64 ? !dtl64 : !dtl32)) continue;
      if (geglu_fwd && (c.idx == 19 || c.idx == 20)) continue;      // its column permutation wants equal column halves, and the direct-to-LDS loaders
      if (c.idx == 20 && !allow16) continue;       // the 16x16x32 instruction sums a k-step of 32 at once: other bits than the 32x32x16 tiles
      const long tiles = (long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
      float cost = (float)((tiles + kCUs - 1) / kCUs) * (c.fixed + (float)((K + 63) / 64) * c.per_kt) + 0.9f * outputs;
      if (c.idx == 13) {
        int z = 1;
        cost = tile128_us(tiles, K / 64, heavy);
        if (may_split) z = splits_128(M, N, K, ln, heavy, &cost);
        if (z == 1) cost += 1.4f * outputs;
      }
      consider(c.idx, cost);
    }
    if (dtl64 && !geglu_fwd) {
      const long tiles = (long)((M + 63) / 64) * ((N + 63) / 64);
      const int z = may_split ? choose_splits_epi(tiles, K / 64) : 1;
      consider(15, tile64_choice_us(tiles, K / 64, z) + (z > 1 ? reduce_us(M, N, z, ln) : outputs));
    }
    if (dtl64 && wave_ok)
      for (int i = 0; i < (int)(sizeof(kWave) / sizeof(kWave[0])); ++i) {
        int splits;
        const float us = wave_us(kWave[i], M, N, K, may_split, ln, &splits);
        consider(25 + i, us + (splits > 1 ? 0.f : (kWave[i].bm <= 64 ? 0.8f : 0.3f) * outputs));
      }
    if (best >= 0) return best;
    return t256x128 >= 128 ? 1 : 0;
  }
  if (dtl32 && t256x256 >= 128) return 6;
  if (dtl32 && K <= 1024) return 8;
  if (K >= 2 * N && t256x256 >= 128) return 2;
  return t256x128 >= 128 ? 1 : 0;
}

size_t gemm_splitk_ws_bytes(int M, int N, int K) {
  size_t worst = 0;
  for (int c = 0; c < kNumCfgs; ++c) {
    const long tiles = (long)((M + kCfgs[c].bm - 1) / kCfgs[c].bm) * ((N + kCfgs[c].bn - 1) / kCfgs[c].bn);
    const int s = choose_splits(tiles, (K + kCfgs[c].bk - 1) / kCfgs[c].bk, 2 * kCUs);
    if (s > 1) worst = std::max(worst, (size_t)s * ((size_t)M * N + M) * sizeof(float));   // + the column sums of A per split
  }
  return worst;
}

template <int BM, int BN, int BK, int WGM, int WGN, bool A_MC, bool B_MC>
static int launch_bf16_cfg(const GemmArgs& a, hipStream_t s) {
  using S = GemmSmem<BM, BN, BK, WGM, WGN, A_MC, B_MC>;
  GemmBf16Params p;
  p.A = (const bf16*)a.A; p.B = (const bf16*)a.B;
  p.M = a.M; p.N = a.N; p.K = a.K; p.lda = a.lda; p.ldb = a.ldb; p.split_major = 0;
  p.epi = make_epi<bf16>(a);
  p.tiles_m = (a.M + BM - 1) / BM; p.tiles_n = (a.N + BN - 1) / BN;
  p.group_m = choose_group_m(a, p.tiles_m, p.tiles_n);
  const int kt = (a.K + BK - 1) / BK;
  int splits = 1;
  if (a.out_f32) {
    splits = choose_splits((long)p.tiles_m * p.tiles_n, kt, S::BYTES <= 80 * 1024 ? 2 * kCUs : kCUs);
    if (splits > 1) {
      const size_t need = (size_t)splits * ((size_t)a.M * a.N + (a.colsum_out ? a.M : 0)) * sizeof(float);
      if (!a.splitk_ws || a.splitk_ws_bytes < need) splits = 1;
    }
  }
  p.k_tiles_per_split = (kt + splits - 1) / splits;
  splits = (kt + p.k_tiles_per_split - 1) / p.k_tiles_per_split;
  if (splits > 1) p.epi.partial = a.splitk_ws;
  float* colsum_ws = nullptr;
  p.colsum = nullptr; p.colsum_stride = 0; p.colsum_acc = 0;
  if (A_MC && a.colsum_out) {
    if (!a.out_f32) return set_error(DP_EUNSUPPORTED, "gemm: column sums come with an fp32 output only");
    if (splits > 1) { colsum_ws = a.splitk_ws + (size_t)splits * a.M * a.N; p.colsum = colsum_ws; p.colsum_stride = a.M; }
    else { p.colsum = a.colsum_out; p.colsum_acc = a.accumulate; }
  }
  dim3 grid(p.tiles_m * p.tiles_n, 1, splits);
  p.split_major = 0;
  if (splits > 1) { p.split_major = splits; grid = dim3(p.tiles_m * p.tiles_n * splits, 1, 1); }
  const size_t smem = S::BYTES;
  auto kern = gemm_bf16_kernel<BM, BN, BK, WGM, WGN, A_MC, B_MC>;
  static std::atomic<bool> attr_set{false};   // setting it twice is harmless; the flag only saves the call
  if (!attr_set.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess)
      return set_error(DP_EHIP, "hipFuncSetAttribute(gemm) failed");
    attr_set.store(true, std::memory_order_release);
  }
  {
    // the timing scope brackets the GEMM kernel alone (the split-K reduction is its own class)
    KScope ks(a.a_mc ? KK_GEMM_TN : (a.b_mc ? KK_GEMM_NN : KK_GEMM_NT), 2.0 * a.M * a.N * a.K,
              gemm_tensor_bytes(a), s, a.M, a.N, a.K);
    hipLaunchKernelGGL(kern, grid, dim3(WGM * WGN * 64), smem, s, p);
  }
  if (hipGetLastError() != hipSuccess) return set_error(DP_EHIP, "gemm launch failed");
  if (splits > 1) {
    KScope ks(KK_REDUCE, 0.0, 4.0 * (splits + 1.0) * a.M * a.N, s, a.M, a.N, splits);
    return launch_reduce_partials2(a.splitk_ws, splits, (size_t)a.M * a.N, a.out_f32, colsum_ws, colsum_ws ? (size_t)a.M : 0,
                                   a.colsum_out, a.accumulate, s);
  }
  return DP_OK;
}

static int set_lds_limit(const void* kern, size_t bytes, std::atomic<bool>& done) {
  if (done.load(std::memory_order_acquire)) return DP_OK;     // setting it twice is harmless; the flag only saves the call
  if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return set_error(DP_EHIP, "hipFuncSetAttribute(gemm) failed");
  done.store(true, std::memory_order_release);
  return DP_OK;
}

static bool reduction_does_ln(const GemmArgs& a) {
  return !a.out_f32 && a.ln_out && a.ln_applied && a.ln_gamma && a.ln_beta && a.residual && a.residual_f32 && a.out_fused_f32 &&
         a.out == a.residual && a.ldo == a.N && a.ld_res == a.N && !a.act && !a.dact_pre && !a.gate && !a.pre_out && !a.geglu && a.N <= 2048;
}

// A kernel of `kt` k-tiles per output tile with its contraction cut into `splits` parts (1: none), and the pass that adds them.
template <class Kern>
static int launch_split(const GemmArgs& a, GemmBf16Params& p, Kern kern, int threads, size_t smem, std::atomic<bool>& attr_set, int kt, int splits, hipStream_t s) {
  if (splits > 1) {
    const size_t need = (size_t)splits * a.M * a.N * sizeof(float);
    if (!a.splitk_ws || a.splitk_ws_bytes < need) {
      // with choice_rows the split is part of what the caller asked for: running unsplit would silently change the sums
      if (a.choice_rows > 0) return set_error(DP_EWORKSPACE, "gemm: split-K workspace too small for the split chosen from choice_rows");
      splits = 1;
    }
  }
  p.k_tiles_per_split = (kt + splits - 1) / splits;
  splits = (kt + p.k_tiles_per_split - 1) / p.k_tiles_per_split;
  if (splits > 1) p.epi.partial = a.splitk_ws;
  DP_TRY(set_lds_limit((const void*)kern, smem, attr_set));
  {
    // the timing scope brackets the GEMM kernel alone (the split-K reduction is its own class)
    KScope ks(a.a_mc ? KK_GEMM_TN : (a.b_mc ? KK_GEMM_NN : KK_GEMM_NT), 2.0 * a.M * a.N * a.K,
              gemm_tensor_bytes(a), s, a.M, a.N, a.K);
    hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n, 1, splits), dim3(threads), smem, s, p);
  }
  if (hipGetLastError() != hipSuccess) return set_error(DP_EHIP, "gemm launch failed");
  if (a.ln_applied) *a.ln_applied = 0;
  if (splits > 1 && reduction_does_ln(a)) {
    // the reduction pass also normalises the rows it completes (one launch less per projection onto the residual stream)
    *a.ln_applied = 1;
    return launch_reduce_residual_ln(a.splitk_ws, splits, a.M, a.N, a.bias, (float*)a.out, a.ln_out, a.ln_gamma, a.ln_beta, a.ln_eps, s);
  }
  if (splits > 1 && !a.out_f32) {
    KScope ks(KK_REDUCE, 0.0, 4.0 * splits * a.M * a.N + 2.0 * a.M * a.N, s, a.M, a.N, splits);
    const size_t groups = (size_t)a.M * (a.N / 8);
    hipLaunchKernelGGL(reduce_epilogue_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, s, make_epi<bf16>(a), a.splitk_ws, splits);
    return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm split-K epilogue launch failed");
  }
  if (splits > 1) {
    KScope ks(KK_REDUCE, 0.0, 4.0 * (splits + 1.0) * a.M * a.N, s, a.M, a.N, splits);
    return launch_reduce_partials(a.splitk_ws, splits, (size_t)a.M * a.N, a.out_f32, a.accumulate, s);
  }
  return DP_OK;
}

template <int BM, int BN, bool A_MC, bool B_MC>
static int dtl_params(const GemmArgs& a, GemmBf16Params& p) {
  p.A = (const bf16*)a.A; p.B = (const bf16*)a.B;
  p.M = a.M; p.N = a.N; p.K = a.K; p.lda = a.lda; p.ldb = a.ldb; p.split_major = 0;
  p.epi = make_epi<bf16>(a);
  p.tiles_m = (a.M + BM - 1) / BM; p.tiles_n = (a.N + BN - 1) / BN;
  p.group_m = choose_group_m(a, p.tiles_m, p.tiles_n);
  if (!dtl_addressable(a)) return set_error(DP_EUNSUPPORTED, "gemm: operand too large for the forced direct-to-LDS configuration");
  p.a_bytes = (uint32_t)(A_MC ? operand_extent_bytes(a.K, a.M, a.lda) : operand_extent_bytes(a.M, a.K, a.lda));
  p.b_bytes = (uint32_t)(B_MC ? operand_extent_bytes(a.K, a.N, a.ldb) : operand_extent_bytes(a.N, a.K, a.ldb));
  return DP_OK;
}

// Parts that the contraction is cut into on BM x BN tiles, `slots` of which the chip holds.
template <int BM, int BN, int BK>
static int dtl_splits(const GemmArgs& a, int slots) {
  const long tiles_n = (a.N + BN - 1) / BN;
  const int kt = a.K / BK;
  if (a.out_f32) return choose_splits((a.M + BM - 1) / BM * tiles_n, kt * BK / 64, slots);
  if (!a.splitk_ws || a.geglu == 1 || a.choice_rows < 0) return 1;
  const long rows = a.choice_rows > 0 ? a.choice_rows : a.M;
  float us;
  const int splits = BM == 128 && BN == 128 && BK == 64 ? splits_128((int)rows, a.N, a.K, a.ln_out != nullptr, heavy_epilogue(a), &us) : choose_splits_epi((rows + BM - 1) / BM * tiles_n, kt * BK / 64);
  return a.choice_rows > 0 || a.splitk_ws_bytes >= (size_t)splits * a.M * a.N * sizeof(float) ? splits : 1;
}

template <int BM, int BN, int BK, int STAGES, int WGM, int WGN, bool A_MC, bool B_MC>
static int launch_dtl_cfg(const GemmArgs& a, hipStream_t s) {
  using S = DtlSmem<BM, BN, BK, STAGES, WGM, WGN>;
  GemmBf16Params p;
  DP_TRY((dtl_params<BM, BN, A_MC, B_MC>(a, p)));
  const int kt = a.K / BK, splits = dtl_splits<BM, BN, BK>(a, S::BYTES <= 80 * 1024 ? 2 * kCUs : kCUs);
  if constexpr (!A_MC && !B_MC && BK == 64 && ((BM == 64 && BN == 64) || (BM == 128 && BN == 128 && WGM == 4))) {
    const int kind = a.out_f32 || splits > 1 ? PE_F32 : pp_kind(a);
    switch (kind) {
#define DP_DTL_CASE(k_) case k_: { \
        static std::atomic<bool> set{false}; \
        return launch_split(a, p, gemm_bf16_dtl_kernel<BM, BN, BK, STAGES, WGM, WGN, A_MC, B_MC, false, false, k_>, WGM * WGN * 64, S::BYTES, set, kt, splits, s); }
      DP_DTL_CASE(PE_PLAIN) DP_DTL_CASE(PE_F32) DP_DTL_CASE(PE_RES) DP_DTL_CASE(PE_RESH) DP_DTL_CASE(PE_GATE) DP_DTL_CASE(PE_ACT1) DP_DTL_CASE(PE_ACT2)
      DP_DTL_CASE(PE_ACT3) DP_DTL_CASE(PE_DACT1) DP_DTL_CASE(PE_DACT2) DP_DTL_CASE(PE_GEGLU2)
#undef DP_DTL_CASE
      default: break;      // the fused GeGLU forward, and combinations no kind has
    }
  }
  static std::atomic<bool> attr_set{false};
  return launch_split(a, p, gemm_bf16_dtl_kernel<BM, BN, BK, STAGES, WGM, WGN, A_MC, B_MC>, WGM * WGN * 64, S::BYTES, attr_set, kt, splits, s);
}

// The additions of a launch with its contraction cut into `splits` parts, in one workgroup per output tile.
template <int BM, int BN, int BK, int STAGES, int WGM, int WGN>
static int launch_segments(const GemmArgs& a, int splits, hipStream_t s) {
  using S = DtlSmem<BM, BN, BK, STAGES, WGM, WGN>;
  GemmBf16Params p;
  DP_TRY((dtl_params<BM, BN, false, false>(a, p)));
  p.k_tiles_per_split = (a.K / BK + splits - 1) / splits;
  const bool ln = reduction_does_ln(a);
  if (ln && (!a.splitk_ws || a.splitk_ws_bytes < (size_t)a.M * a.N * sizeof(float))) return set_error(DP_EWORKSPACE, "gemm: split-K workspace too small for the split chosen from choice_rows");
  if (ln) p.epi.partial = a.splitk_ws;      // the sums, for the pass that adds bias and residual and normalises (the same one as after a split launch)
  auto launch = [&](auto kind) {
    auto kern = gemm_bf16_dtl_kernel<BM, BN, BK, STAGES, WGM, WGN, false, false, false, true, kind>;
    static std::atomic<bool> attr_set{false};
    DP_TRY(set_lds_limit((const void*)kern, S::BYTES, attr_set));
    KScope ks(KK_GEMM_NT, 2.0 * a.M * a.N * a.K, gemm_tensor_bytes(a), s, a.M, a.N, a.K);
    hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n), dim3(WGM * WGN * 64), S::BYTES, s, p);
    return (int)DP_OK;
  };
  // (the kinds that the encoder's projections have)
  switch (ln ? PE_F32 : pp_kind(a)) {
    case PE_F32: DP_TRY(launch(std::integral_constant<int, PE_F32>())); break;
    case PE_PLAIN: DP_TRY(launch(std::integral_constant<int, PE_PLAIN>())); break;
    case PE_RES: DP_TRY(launch(std::integral_constant<int, PE_RES>())); break;
    case PE_ACT3: DP_TRY(launch(std::integral_constant<int, PE_ACT3>())); break;
    default: DP_TRY(launch(std::integral_constant<int, -1>())); break;
  }
  if (hipGetLastError() != hipSuccess) return set_error(DP_EHIP, "gemm launch failed");
  if (a.ln_applied) *a.ln_applied = ln;
  return ln ? launch_reduce_residual_ln(a.splitk_ws, 1, a.M, a.N, a.bias, (float*)a.out, a.ln_out, a.ln_gamma, a.ln_beta, a.ln_eps, s) : DP_OK;
}

template <class T, int KIND, bool FP8, bool KTAIL>
static int launch_pp_kernel(const GemmBf16Params& p, hipStream_t s) {
  // up to one tile per CU there is nothing to walk to, and a part of a k-tile is rare
  if constexpr (!KTAIL) {
    if (p.tiles_m * p.tiles_n > kCUs) {
      auto kern = gemm_pp_kernel<T, KIND, FP8, KTAIL, true>;
      static std::atomic<bool> walk_set{false};
      DP_TRY(set_lds_limit((const void*)kern, PpWalk<T>::BYTES, walk_set));
      hipLaunchKernelGGL(kern, dim3(kCUs), dim3(512), PpWalk<T>::BYTES, s, p);
      return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm launch failed");
    }
  }
  auto kern = gemm_pp_kernel<T, KIND, FP8, KTAIL>;
  static std::atomic<bool> attr_set{false};
  DP_TRY(set_lds_limit((const void*)kern, T::BYTES, attr_set));
  hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n), dim3(512), T::BYTES, s, p);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm launch failed");
}
// C = out_scale * (A_q B_q^T) (+ bias) for OCP E4M3 operands A_q [M, K], B_q [N, K] (bytes, contraction contiguous), storage-dtype
// (bf16) output.  The kernel sees the operands as two-byte elements: K / 2 of them per row.
static GemmBf16Params fp8_params(const Fp8GemmArgs& a, int bm, int bn) {
  GemmBf16Params p;
  memset(&p, 0, sizeof(p));
  p.A = (const bf16*)a.A; p.B = (const bf16*)a.B;
  p.M = a.M; p.N = a.N; p.K = a.K / 2; p.lda = a.lda / 2; p.ldb = a.ldb / 2;
  EpiParams<bf16>& e = p.epi;
  e.M = a.M; e.N = a.N; e.out = (bf16*)a.out; e.ldo = a.ldo; e.bias = (const bf16*)a.bias; e.rows_per_batch = 1; e.out_scale = a.out_scale;
  p.tiles_m = (a.M + bm - 1) / bm; p.tiles_n = (a.N + bn - 1) / bn;
  GemmArgs shape; memset(&shape, 0, sizeof(shape)); shape.M = a.M; shape.N = a.N;
  p.group_m = choose_group_m(shape, p.tiles_m, p.tiles_n);
  p.a_bytes = (uint32_t)((size_t)(a.M - 1) * a.lda + a.K);
  p.b_bytes = (uint32_t)((size_t)(a.N - 1) * a.ldb + a.K);
  return p;
}
template <int BM, int BN, int WGM, int WGN>
static int launch_fp8_cfg(const Fp8GemmArgs& a, hipStream_t s) {
  constexpr int BK = 64, STAGES = 3;
  using S = DtlSmem<BM, BN, BK, STAGES, WGM, WGN>;
  GemmBf16Params p = fp8_params(a, BM, BN);
  p.k_tiles_per_split = p.K / BK;
  auto kern = gemm_bf16_dtl_kernel<BM, BN, BK, STAGES, WGM, WGN, false, false, true, false, PE_PLAIN>;
  static std::atomic<bool> attr_set{false};
  DP_TRY(set_lds_limit((const void*)kern, S::BYTES, attr_set));
  KScope ks(KK_GEMM_FP8, 2.0 * a.M * a.N * a.K, (double)a.M * a.K + (double)a.N * a.K + 2.0 * a.M * a.N, s, a.M, a.N, a.K);
  hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n, 1, 1), dim3(WGM * WGN * 64), S::BYTES, s, p);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm fp8 launch failed");
}
template <class T>
static int launch_fp8_pp(const Fp8GemmArgs& a, hipStream_t s) {
  KScope ks(KK_GEMM_FP8, 2.0 * a.M * a.N * a.K, (double)a.M * a.K + (double)a.N * a.K + 2.0 * a.M * a.N, s, a.M, a.N, a.K);
  return launch_pp_kernel<T, PE_PLAIN, true, false>(fp8_params(a, T::BM, T::BN), s);
}

int launch_gemm_fp8(const Fp8GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return set_error(DP_EINVAL, "gemm fp8: non-positive size");
  if (!a.A || !a.B || !a.out) return set_error(DP_EINVAL, "gemm fp8: null operand");
  if (a.K % 128) return set_error(DP_EUNSUPPORTED, "gemm fp8: K must be a multiple of 128");
  if (a.lda % 16 || a.ldb % 16 || a.lda < a.K || a.ldb < a.K) return set_error(DP_EUNSUPPORTED, "gemm fp8: leading dims must be multiples of 16 bytes and at least K");
  if (a.N % 8 || a.ldo % 8 || a.ldo < a.N) return set_error(DP_EUNSUPPORTED, "gemm fp8: N and ldc must be multiples of 8, ldc >= N");
  if (!(a.out_scale > 0.f)) return set_error(DP_EINVAL, "gemm fp8: the output scale must be positive");
  const void* ps[] = {a.A, a.B, a.out, a.bias};
  for (const void* q : ps) if ((uintptr_t)q % 16) return set_error(DP_EALIGN, "gemm fp8: operands must be 16-byte aligned");
  if ((size_t)(a.M - 1) * a.lda + a.K >= (1ull << 32) || (size_t)(a.N - 1) * a.ldb + a.K >= (1ull << 32))
    return set_error(DP_EUNSUPPORTED, "gemm fp8: operand larger than 4 GiB");
  // the tile with the least estimated time, as in choose_cfg: a k-tile of 128 8-bit values costs what one of 64 bf16 values costs
  // (same bytes, twice the products at twice the rate)
  const struct { int bm, bn; float fixed, per_kt; } tiles[] = {{256, 256, 6.0f, 1.40f}, {256, 192, 6.0f, 1.10f}, {256, 128, 5.0f, 0.75f}, {128, 128, 4.0f, 0.45f}};
  int best = 0;
  float best_us = 0.f;
  for (int i = 0; i < 4; ++i) {
    const long n = (long)((a.M + tiles[i].bm - 1) / tiles[i].bm) * ((a.N + tiles[i].bn - 1) / tiles[i].bn);
    const float us = (float)((n + kCUs - 1) / kCUs) * (tiles[i].fixed + (float)(a.K / 128) * tiles[i].per_kt);
    if (i == 0 || us < best_us) { best = i; best_us = us; }
  }
  switch (best) {
    case 0: return launch_fp8_pp<PpTile<256, 128, 128, 4, 2>>(a, s);
    case 1: return launch_fp8_pp<PpTile<256, 128, 64, 4, 2>>(a, s);
    case 2: return launch_fp8_pp<PpTile<256, 64, 64, 4, 2>>(a, s);
    default: return launch_fp8_cfg<128, 128, 4, 2>(a, s);
  }
}

// Epilogue kind of a problem for the kernels with one epilogue per kind, or -1 if it combines what no kind combines.
static int pp_kind(const GemmArgs& a) {
  if (a.geglu) return a.geglu == 1 ? PE_GEGLU1 : PE_GEGLU2;
  if (a.residual) {
    if (a.act || a.dact_pre || (a.pre_out && !a.gate)) return -1;
    if (!a.residual_f32) return a.gate || a.out_fused_f32 ? -1 : PE_RESH;
    return a.gate ? PE_GATE : PE_RES;
  }
  if (a.gate || a.out_fused_f32) return -1;
  if (a.act) return a.dact_pre || a.act > 3 ? -1 : PE_ACT1 + a.act - 1;
  if (a.pre_out) return -1;
  if (a.dact_pre) return a.dact_kind == ACT_GELU_ERF ? PE_DACT1 : (a.dact_kind == ACT_GELU_TANH ? PE_DACT2 : -1);
  return PE_PLAIN;
}

// Which instruction.  With all CUs busy the clock is set by the power that the matrix cores draw: a loop of v_mfma_f32_16x16x32 on normally distributed
// operands runs at 2.09 GHz (2.06 PFLOP/s) where the same products by 32x32x16 hold 1.81 (1.81).  256x256 and 256x192 tiles, which come nearest to that:
// 8192^3 781 -> 755 and 899 -> 854 us on one card; steps of two U-Net blocks 8 x 4096 x 320, seven DiT blocks 32 x 256 x 1152 and the text encoder on 64 samples
// 3397 -> 3360, 10073 -> 9940 and 1549 -> 1487 us there, on a card whose clock falls less 3236 -> 3230, 9672 -> 9585 and 1477 -> 1469.  Tiles of
// 128 columns wait for their operands (8192 x 5120, K = 640: 75 us either way) and keep the larger instruction, as do calls that have to agree bit for bit with
// other tiles (choice_rows, and the fused GeGLU forward, whose bits are those of the separate kernels): the smaller one adds up 32 products at a time.  While
// CUs idle the clock is high and the larger one ahead, on 256x256 tiles the more so the longer they walk (PP_IDLE_KT; us, 32x32x16 and 16x16x32, by tiles and contraction;
// 96 and 128 tiles of K = 1152 27.0 and 28.6, 26.6 and 28.2):
//   K =  640: 160 tiles 19.7 and 20.1, 192 21.9 and 21.5, 256 25.2 and 24.7, 288 37.5 and 37.9, 384 40.6 and 40.6, 512 51.2 and 46.8
//   K = 1152: 160 28.6 and 29.5, 192 30.3 and 30.7, 224 33.5 and 33.2, 256 37.1 and 35.9, 288 55.8 and 56.9, 384 60.4 and 60.2, 512 72.8 and 68.5
//   K = 2304: 160 47.6 and 49.6, 208 54.5 and 57.4, 240 59.5 and 59.2, 256 63.1 and 61.0, 264 98.3 and 100.4, 480 117.3 and 117.0
//   K = 4608: 160 89.4 and 96.1, 192 94.9 and 102.8, 240 109.4 and 111.0, 256 115.4 and 112.6, 288 185 and 188, 448 209 and 211
// On 256x192 tiles the smaller one is ahead from 160 on, whatever the contraction (64 to 4608) and the last round: 160 tiles of K = 320 / 1152 / 4608 12.8 -> 12.5, 23.2 -> 22.6,
// 67.8 -> 67.7, 224 12.7 -> 12.4, 25.5 -> 24.4, 82.4 -> 76.9, 264 21.0 -> 20.4, 44.7 -> 43.4, 149 -> 144, 512 22.2 -> 21.5, 52.6 -> 50.5, 178 -> 173.
constexpr int PP_IDLE_KT = 3;
template <class T>
static bool pp_on_16(long tiles, int K) {
  if (T::BN < 192 || tiles < 160) return false;
  const long slots = (tiles + kCUs - 1) / kCUs * kCUs;
  return T::BN == 192 || (slots - tiles) * (K / 64) <= PP_IDLE_KT * slots;      // k-tiles that a CU idles through in a round, on average
}
template <class T, int KIND>
static int launch_pp_kind(const GemmBf16Params& p, bool any_order, hipStream_t s) {
  if (p.K % T::BK) return launch_pp_kernel<T, KIND, false, true>(p, s);
  if constexpr (T::BN >= 192 && KIND != PE_GEGLU1) {
    if (any_order && pp_on_16<T>((long)p.tiles_m * p.tiles_n, p.K)) return launch_pp_kernel<typename T::On16, KIND, false, false>(p, s);
  }
  return launch_pp_kernel<T, KIND, false, false>(p, s);
}

template <class T>
static GemmBf16Params pp_params(const GemmArgs& a) {
  GemmBf16Params p;
  p.A = (const bf16*)a.A; p.B = (const bf16*)a.B;
  p.M = a.M; p.N = a.N; p.K = a.K; p.lda = a.lda; p.ldb = a.ldb; p.split_major = 0;
  p.epi = make_epi<bf16>(a);
  p.tiles_m = (a.M + T::BM - 1) / T::BM; p.tiles_n = (a.N + T::BN - 1) / T::BN;
  p.group_m = choose_group_m(a, p.tiles_m, p.tiles_n);
  p.a_bytes = (uint32_t)operand_extent_bytes(a.M, a.K, a.lda);
  p.b_bytes = (uint32_t)operand_extent_bytes(a.N, a.K, a.ldb);
  return p;
}

template <class T, int KIND, bool KTAIL>
static int launch_pp_strided(const GemmArgs& a, int count, const GemmStrides& d, hipStream_t s) {
  const GemmBf16Params p = pp_params<T>(a);
  auto kern = gemm_pp_strided_kernel<T, KIND, KTAIL>;
  static std::atomic<bool> attr_set{false};
  DP_TRY(set_lds_limit((const void*)kern, T::BYTES, attr_set));
  KScope ks(KK_GEMM_NT, 2.0 * a.M * a.N * a.K * count, gemm_tensor_bytes(a) * count, s, a.M * count, a.N, a.K);
  hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n, count), dim3(512), T::BYTES, s, p, d);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm launch failed");
}
template <class T>
static int launch_pp_strided_kind(const GemmArgs& a, int count, const GemmStrides& d, hipStream_t s) {
  const bool tail = a.K % T::BK != 0;
  if (a.out_f32) return tail ? launch_pp_strided<T, PE_F32, true>(a, count, d, s) : launch_pp_strided<T, PE_F32, false>(a, count, d, s);
  return tail ? launch_pp_strided<T, PE_PLAIN, true>(a, count, d, s) : launch_pp_strided<T, PE_PLAIN, false>(a, count, d, s);
}
// `count` products y = x W^T (+ bias), operands and outputs at fixed distances.  The attention block of the image encoder makes them per
// sample; one at a time, its probabilities x values (4096 x 512, K = 4096) are 32 tiles of 256x256 for 256 CUs and its scores wait for each
// other's last round.  One launch for all of them when 256x128 tiles occupy at least half of the CUs, else one by one.  The additions are in the
// same order either way.
int launch_gemm_strided(const GemmArgs& a, int count, long stride_a, long stride_b, long stride_out, hipStream_t s) {
  if (a.dtype != BF16 || count <= 0 || a.a_mc || a.b_mc || a.accumulate || (!a.out_f32 && pp_kind(a) != PE_PLAIN) || a.choice_rows >= 0 || stride_a % 8 || stride_b % 8 || stride_out % 8)
    return set_error(DP_EUNSUPPORTED, "gemm: operands or epilogue of a strided batch");
  const long n256 = (long)((a.M + 255) / 256) * ((a.N + 255) / 256) * count, n128 = (long)((a.M + 255) / 256) * ((a.N + 127) / 128) * count;
  if (n128 >= kCUs / 2 && dtl_addressable(a) && count <= 65535) {
    const float kt = (float)((a.K + 63) / 64), t256 = (float)((n256 + kCUs - 1) / kCUs) * (5.0f + 1.30f * kt), t128 = (float)((n128 + kCUs - 1) / kCUs) * (5.0f + 0.72f * kt);
    const GemmStrides d{stride_a, stride_b, stride_out};
    return t256 <= t128 ? launch_pp_strided_kind<PpTile<256, 128, 128, 4, 2>>(a, count, d, s) : launch_pp_strided_kind<PpTile<256, 64, 64, 4, 2>>(a, count, d, s);
  }
  for (int i = 0; i < count; ++i) {
    GemmArgs g = a;
    g.A = (const bf16*)a.A + i * stride_a; g.B = (const bf16*)a.B + i * stride_b;
    if (a.out_f32) g.out_f32 = a.out_f32 + i * stride_out;
    else g.out = (bf16*)a.out + i * stride_out;
    DP_TRY(launch_gemm(g, s));
  }
  return DP_OK;
}

template <class T>
static int launch_pp(const GemmArgs& a, hipStream_t s) {
  if (a.a_mc || a.b_mc || a.out_f32) return set_error(DP_EUNSUPPORTED, "gemm: the forced configuration needs contraction-contiguous operands and a storage-dtype output");
  if (!dtl_addressable(a)) return set_error(DP_EUNSUPPORTED, "gemm: operand too large for the forced direct-to-LDS configuration");
  const int kind = pp_kind(a);
  if (kind < 0) return set_error(DP_EUNSUPPORTED, "gemm: the forced configuration does not have this epilogue");
  const GemmBf16Params p = pp_params<T>(a);
  const bool any_order = a.choice_rows == 0;
  KScope ks(KK_GEMM_NT, 2.0 * a.M * a.N * a.K, gemm_tensor_bytes(a), s, a.M, a.N, a.K);
  switch (kind) {
#define DP_PP_CASE(k_) case k_: return launch_pp_kind<T, k_>(p, any_order, s)
    DP_PP_CASE(PE_PLAIN); DP_PP_CASE(PE_RES); DP_PP_CASE(PE_RESH); DP_PP_CASE(PE_GATE); DP_PP_CASE(PE_ACT1); DP_PP_CASE(PE_ACT2);
    DP_PP_CASE(PE_ACT3); DP_PP_CASE(PE_DACT1); DP_PP_CASE(PE_DACT2); DP_PP_CASE(PE_GEGLU2);
#undef DP_PP_CASE
    case PE_GEGLU1:
      if constexpr (T::SN0 == T::SN1) return launch_pp_kind<T, PE_GEGLU1>(p, any_order, s);
    default: return set_error(DP_EUNSUPPORTED, "gemm: epilogue kind");
  }
}

template <class T, int KIND, bool B_MC = false>
static int launch_wave_kind(const GemmArgs& a, GemmBf16Params& p, int splits, hipStream_t s) {
  static std::atomic<bool> attr_set{false};
  return launch_split(a, p, gemm_wave_kernel<T, KIND, B_MC>, T::NW * 64, T::BYTES, attr_set, a.K / 64, splits, s);
}
// The rows operand normalised on the way in: 32-row tiles, unsplit.
template <class T, int KIND>
static int launch_wave_norm_kind(const GemmArgs& a, hipStream_t s) {
  GemmBf16Params p = pp_params<T>(a);
  p.norm_x = a.norm_x; p.norm_gamma = (const bf16*)a.norm_gamma; p.norm_beta = (const bf16*)a.norm_beta; p.norm_eps = a.norm_eps;
  const size_t bytes = std::max((size_t)a.K * 2 * T::BM + (size_t)T::NW * T::BN * 128, (size_t)T::SLAB);
  static std::atomic<bool> attr_set{false};
  auto kern = gemm_wave_kernel<T, KIND, false, true>;
  DP_TRY(set_lds_limit((const void*)kern, 160 * 1024, attr_set));
  p.k_tiles_per_split = a.K / 64;
  KScope ks(KK_GEMM_NT, 2.0 * a.M * a.N * a.K, gemm_tensor_bytes(a) + 2.0 * a.M * a.K, s, a.M, a.N, a.K);
  hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n), dim3(T::NW * 64), bytes, s, p);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm launch failed");
}
template <class T>
static int launch_wave_norm(const GemmArgs& a, hipStream_t s) {
  return a.act ? launch_wave_norm_kind<T, PE_ACT3>(a, s) : launch_wave_norm_kind<T, PE_PLAIN>(a, s);
}
// The kinds of a backward pass, which the tiles above have for weights as they are stored.
static bool wave_stored_kind(int kind) { return kind == PE_PLAIN || kind == PE_DACT1 || kind == PE_DACT2 || kind == PE_GEGLU2; }
template <class T>
static int launch_wave_tile(const GemmArgs& a, int splits, hipStream_t s) {
  GemmBf16Params p = pp_params<T>(a);
  if (a.b_mc) {
    p.b_bytes = (uint32_t)operand_extent_bytes(a.K, a.N, a.ldb);
    if (splits > 1) return launch_wave_kind<T, PE_F32, true>(a, p, splits, s);
    switch (pp_kind(a)) {
      case PE_PLAIN: return launch_wave_kind<T, PE_PLAIN, true>(a, p, 1, s);
      case PE_DACT1: return launch_wave_kind<T, PE_DACT1, true>(a, p, 1, s);
      case PE_DACT2: return launch_wave_kind<T, PE_DACT2, true>(a, p, 1, s);
      case PE_GEGLU2: return launch_wave_kind<T, PE_GEGLU2, true>(a, p, 1, s);
      default: return set_error(DP_EUNSUPPORTED, "gemm: the forced configuration does not have this epilogue for weights as they are stored");
    }
  }
  if (splits > 1) return launch_wave_kind<T, PE_F32>(a, p, splits, s);
  switch (pp_kind(a)) {
#define DP_WAVE_CASE(k_) case k_: return launch_wave_kind<T, k_>(a, p, 1, s)
    DP_WAVE_CASE(PE_PLAIN); DP_WAVE_CASE(PE_RES); DP_WAVE_CASE(PE_RESH); DP_WAVE_CASE(PE_GATE); DP_WAVE_CASE(PE_ACT1); DP_WAVE_CASE(PE_ACT2);
    DP_WAVE_CASE(PE_ACT3); DP_WAVE_CASE(PE_DACT1); DP_WAVE_CASE(PE_DACT2); DP_WAVE_CASE(PE_GEGLU2);
#undef DP_WAVE_CASE
    default: return set_error(DP_EUNSUPPORTED, "gemm: the forced configuration does not have this epilogue");
  }
}
// T1: the same tile with one k-tile less on its way, two workgroups of which fit a CU.
template <class T, class T1>
static int launch_wave(const GemmArgs& a, const WaveCost& c, hipStream_t s) {
  if (a.a_mc || a.out_f32 || a.geglu == 1 || a.K % 64 || !dtl_addressable(a)) return set_error(DP_EUNSUPPORTED, "gemm: the forced configuration needs a contraction-contiguous row operand, K % 64 == 0 and a storage-dtype output");
  int splits = 1;
  if (a.splitk_ws && a.choice_rows == 0) wave_us(c, a.M, a.N, a.K, true, a.ln_out != nullptr, &splits);
  if (splits > 1 && a.splitk_ws_bytes < (size_t)splits * a.M * a.N * sizeof(float)) splits = 1;
  const int kps = (a.K / 64 + splits - 1) / splits;
  splits = (a.K / 64 + kps - 1) / kps;
  const long tiles = (long)((a.M + T::BM - 1) / T::BM) * ((a.N + T::BN - 1) / T::BN) * splits;
  return std::is_same<T, T1>::value || tiles <= kCUs ? launch_wave_tile<T>(a, splits, s) : launch_wave_tile<T1>(a, splits, s);
}

template <int BM, int BN, int BK, int STAGES, int WGM, int WGN>
static int launch_dtl_layout(const GemmArgs& a, hipStream_t s) {
  if (a.K % BK) return set_error(DP_EUNSUPPORTED, "gemm: K is not a multiple of the k-tile of the forced configuration");
  if (!a.a_mc && !a.b_mc) return launch_dtl_cfg<BM, BN, BK, STAGES, WGM, WGN, false, false>(a, s);
  if (!a.a_mc && a.b_mc) return launch_dtl_cfg<BM, BN, BK, STAGES, WGM, WGN, false, true>(a, s);
  if (a.a_mc && a.b_mc) return launch_dtl_cfg<BM, BN, BK, STAGES, WGM, WGN, true, true>(a, s);
  return launch_dtl_cfg<BM, BN, BK, STAGES, WGM, WGN, true, false>(a, s);
}

template <int BM, int BN, int BK, int WGM, int WGN>
static int launch_bf16_layout(const GemmArgs& a, hipStream_t s) {
  if (!a.a_mc && !a.b_mc) return launch_bf16_cfg<BM, BN, BK, WGM, WGN, false, false>(a, s);
  if (!a.a_mc && a.b_mc) return launch_bf16_cfg<BM, BN, BK, WGM, WGN, false, true>(a, s);
  if (a.a_mc && a.b_mc) return launch_bf16_cfg<BM, BN, BK, WGM, WGN, true, true>(a, s);
  return launch_bf16_cfg<BM, BN, BK, WGM, WGN, true, false>(a, s);
}

// The bias gradient can ride in a weight-gradient GEMM when that GEMM runs on the register-staged kernel, or in fp32.
bool gemm_colsum_supported(const GemmArgs& a) {
  if (a.dtype == F32) return a.a_mc && a.out_f32;
  if (a.dtype != BF16 || !a.a_mc || !a.b_mc || !a.out_f32 || a.M % 8) return false;
  const int cfg = (a.force_cfg > 0) ? a.force_cfg - 1 : choose_cfg(a.M, a.N, a.K, true, true, dtl_addressable(a), false);
  return cfg >= 0 && cfg <= 5;
}

bool gemm_geglu_fwd_supported(const GemmArgs& a) {
  return a.dtype == BF16 && !a.a_mc && !a.b_mc && a.K % 32 == 0 && a.geglu_inner > 0 && a.geglu_inner % 32 == 0 &&
         a.N == 2 * a.geglu_inner && a.ldo >= a.geglu_inner && (!a.pre_out || a.ld_pre >= a.N) && dtl_addressable(a);
}

// The tile choice for a problem of `rows` rows.  Its estimates cost the host about a microsecond, so each thread remembers the last choices, by
// everything they depend on.
static int chosen_cfg(const GemmArgs& a, int rows, bool may_split) {
  struct Entry { int rows, n, k, flags, cfg; };
  constexpr int ENTRIES = 64;
  static thread_local Entry table[ENTRIES] = {};        // n = 0: empty
  const bool pp = !a.out_f32 && pp_kind(a) >= 0, any_order = a.choice_rows == 0, wave = any_order && pp && a.geglu != 1, dtl = dtl_addressable(a), heavy = heavy_epilogue(a), geglu_fwd = a.geglu == 1;
  const bool onto_f32 = any_order && a.residual && a.residual_f32;
  const int flags = onto_f32 << 10 | geglu_fwd << 9 | heavy << 8 | (a.a_mc != 0) | (a.b_mc != 0) << 1 | dtl << 2 | pp << 3 | any_order << 4 | may_split << 5 | (a.ln_out != nullptr) << 6 | wave << 7;
  Entry& e = table[((unsigned)rows * 0x9E3779B1u ^ (unsigned)a.N * 0x85EBCA77u ^ (unsigned)a.K * 0xC2B2AE3Du ^ (unsigned)flags * 0x27D4EB2Fu) >> 26];
  if (e.n == a.N && e.rows == rows && e.k == a.K && e.flags == flags) return e.cfg;
  e = Entry{rows, a.N, a.K, flags, choose_cfg(rows, a.N, a.K, a.a_mc != 0, a.b_mc != 0, dtl, pp, any_order, may_split, a.ln_out != nullptr, wave, heavy, geglu_fwd, onto_f32)};
  return e.cfg;
}

// choice_rows > 0: the parts the contraction is cut into depend on the shape of the problem with choice_rows rows alone, and so do the sums; the
// tile and whether the parts run as workgroups of their own (few tiles) or one after the other in a workgroup (many: no partial tiles through
// memory) may depend on the rows there are, since they change no bit.  Encoder of 12 layers of width 768, calls of 24 / 48 / 96 samples of 77 rows: 1.27 / 2.26 / 4.10 ms with the
// tiles of one sample's shape as well, 1.05 / 1.51 / 2.73 ms.
static int launch_invariant(const GemmArgs& a, bool may_split, hipStream_t s) {
  const int cfg = chosen_cfg(a, a.choice_rows, may_split), kt = a.K / 64;
  GemmArgs g = a;
  int z = 1;
  if (may_split && (cfg == 13 || cfg == 15)) {
    float us;
    z = cfg == 13 ? splits_128(a.choice_rows, a.N, a.K, a.ln_out != nullptr, heavy_epilogue(a), &us) : choose_splits_epi((long)((a.choice_rows + 63) / 64) * ((a.N + 63) / 64), kt);
  } else if (may_split && cfg >= 6 && cfg <= 16) {
    g.force_cfg = cfg + 1;       // another kind of tile with a split of its own
    return launch_gemm(g, s);
  }
  if (z == 1) {
    g.choice_rows = -1;
    return launch_gemm(g, s);
  }
  const long t64 = (long)((a.M + 63) / 64) * ((a.N + 63) / 64), t128 = (long)((a.M + 127) / 128) * ((a.N + 127) / 128);
  const bool ln = reduction_does_ln(a);
  // (the partial tiles of a launch this size stay in the caches: 0.6 us per million of them)
  auto pass = [&](int planes) { return (ln ? 1.0f : 5.0f) + (float)(planes + 2) * (float)a.M * (float)a.N * 0.6e-6f; };
  const float parts = (cfg == 15 ? tile64_us(t64, kt, z) : tile128_us(t128 * z, (kt + z - 1) / z, false)) + pass(z);
  const float seg64 = tile64_us(t64, kt, 1) + (ln ? pass(1) : 0.f), seg128 = tile128_us(t128, kt, !ln && a.act) + (ln ? pass(1) : 0.f);
  if (parts <= seg64 && parts <= seg128) {
    g.force_cfg = cfg + 1;
    return launch_gemm(g, s);
  }
  if (seg64 <= seg128) return t64 <= 2 * kCUs ? launch_segments<64, 64, 64, 4, 2, 2>(a, z, s) : launch_segments<64, 64, 64, 3, 2, 2>(a, z, s);
  return launch_segments<128, 128, 64, 4, 4, 2>(a, z, s);
}

// Whether dx = dy W is as fast on the weights as they are stored as on a transposed copy: where the copy's product would run on tiles whose waves share the
// contraction.
bool gemm_takes_stored_weight(const GemmArgs& a) {
  if (a.dtype != BF16 || a.a_mc || a.out_f32 || a.choice_rows || a.K % 64 || a.N % 8 || !wave_stored_kind(pp_kind(a))) return false;
  GemmArgs g = a;
  g.b_mc = 0; g.ldb = a.K;
  if (!dtl_addressable(g)) return false;
  g.b_mc = 1; g.ldb = a.N;
  if (!dtl_addressable(g)) return false;
  g.b_mc = 0; g.ldb = a.K;
  const int cfg = chosen_cfg(g, a.M, a.splitk_ws != nullptr);
  return cfg >= 25 && cfg <= 31;
}

// Where the product runs on 32-row tiles, one a CU at most, whose launch and LayerNorm's are both mostly their beginning and end, and the rows fit LDS beside the
// weights.  The rows cost a workgroup 2 us (vector instructions and their way through LDS), a LayerNorm launch 4 with the gap before the next: text encoder of 12 layers, one sample
// of width 768 / 1024 / 512 340 -> 331 / 429 -> 414 / 330 -> 286 us; with two tiles a CU, 4 samples of width 1024, 558 -> 576.
bool gemm_norm_supported(const GemmArgs& a) {
  if (a.dtype != BF16 || a.a_mc || a.b_mc || a.out_f32 || a.choice_rows || a.force_cfg || a.K % 256 || a.K > 1024 || a.lda != a.K || a.N % 8 || !dtl_addressable(a)) return false;
  const int kind = pp_kind(a);
  if (kind != PE_PLAIN && kind != PE_ACT3) return false;
  const int cfg = chosen_cfg(a, a.M, false), bn = 32 * (cfg - 28);
  return cfg >= 29 && cfg <= 31 && (long)((a.M + 31) / 32) * ((a.N + bn - 1) / bn) <= kCUs;
}

int launch_gemm(const GemmArgs& a, hipStream_t s) {
  if (a.ln_applied) *a.ln_applied = 0;
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return set_error(DP_EINVAL, "gemm: non-positive size");
  if (!a.A || !a.B || (!a.out && !a.out_f32)) return set_error(DP_EINVAL, "gemm: null operand");
  if (a.out_f32 && a.ldo32 < a.N) return set_error(DP_EINVAL, "gemm: ldo32 < N");
  if (a.out_f32 && a.ldo32 != a.N) return set_error(DP_EUNSUPPORTED, "gemm: fp32 output must be dense");
  if (a.colsum_out && !gemm_colsum_supported(a)) return set_error(DP_EUNSUPPORTED, "gemm: column sums are not available for this problem");
  if (a.dtype == BF16) {
    // 16-byte vector loads: every row start and the contiguous extent must be multiples of 8 elements
    const int a_inner = a.a_mc ? a.M : a.K, b_inner = a.b_mc ? a.N : a.K;
    if ((a.lda % 8) || (a.ldb % 8) || (a_inner % 8) || (b_inner % 8))
      return set_error(DP_EUNSUPPORTED, "gemm(bf16): leading dims and contiguous extents must be multiples of 8");
    if (((uintptr_t)a.A % 16) || ((uintptr_t)a.B % 16)) return set_error(DP_EALIGN, "gemm(bf16): operands must be 16-byte aligned");
    if (a.lda < a_inner || a.ldb < b_inner) return set_error(DP_EINVAL, "gemm: leading dim too small");
    if (a.N % 8) return set_error(DP_EUNSUPPORTED, "gemm(bf16): N must be a multiple of 8");
    if (a_inner < 8 || b_inner < 8) return set_error(DP_EUNSUPPORTED, "gemm(bf16): contiguous extents must be at least 8");
    const int elds[] = {a.out ? a.ldo : 8, a.pre_out ? a.ld_pre : 8, a.dact_pre ? a.ld_dact : 8, a.gate ? a.gate_ld : 8, a.residual ? a.ld_res : 8};
    for (int x : elds) if (x % 8 || x < 8) return set_error(DP_EUNSUPPORTED, "gemm(bf16): epilogue leading dims must be multiples of 8");
    const void* eps[] = {a.out, a.out_f32, a.bias, a.pre_out, a.dact_pre, a.gate, a.residual, a.splitk_ws};
    for (const void* x : eps) if ((uintptr_t)x % 16) return set_error(DP_EALIGN, "gemm(bf16): epilogue operands must be 16-byte aligned");
    if (a.geglu) {
      if (a.geglu != 1 && a.geglu != 2) return set_error(DP_EINVAL, "gemm: bad geglu mode");
      if (!a.out || a.out_f32 || a.act || a.dact_pre || a.gate || a.residual || a.out_fused_f32)
        return set_error(DP_EUNSUPPORTED, "gemm: a GeGLU epilogue combines with a bias only");
      if (a.geglu == 1 && !gemm_geglu_fwd_supported(a)) return set_error(DP_EUNSUPPORTED, "gemm: fused GeGLU forward not available for this problem");
      if (a.geglu == 2) {
        if (a.N != a.geglu_inner || a.geglu_inner % 8 || !a.geglu_u || a.ld_geglu % 8 || a.ld_geglu < 2 * a.geglu_inner ||
            a.ldo < 2 * a.geglu_inner || a.pre_out || ((uintptr_t)a.geglu_u % 16))
          return set_error(DP_EINVAL, "gemm: bad fused GeGLU backward arguments");
      }
    }
    if (a.norm_x) {
      if (!gemm_norm_supported(a)) return set_error(DP_EUNSUPPORTED, "gemm: the rows of this problem cannot be normalised inside it");
      if ((uintptr_t)a.norm_x % 16 || (uintptr_t)a.norm_gamma % 8 || (uintptr_t)a.norm_beta % 8) return set_error(DP_EALIGN, "gemm: misaligned LayerNorm operands");
      switch (chosen_cfg(a, a.M, false)) {
        case 29: return launch_wave_norm<WaveTile<8, 1, 1>>(a, s);
        case 30: return launch_wave_norm<WaveTile<8, 1, 2>>(a, s);
        default: return launch_wave_norm<WaveTile<8, 1, 3>>(a, s);
      }
    }
    const bool may_split = !a.out_f32 && a.splitk_ws && a.geglu != 1 && a.choice_rows >= 0;
    const bool forced = a.force_cfg > 0 && a.force_cfg <= kNumCfgs + 26;
    if (a.choice_rows > 0 && !forced && !a.a_mc && !a.b_mc) return launch_invariant(a, may_split, s);
    int cfg = forced ? a.force_cfg - 1 : chosen_cfg(a, a.M, may_split);
    if (!forced && a.b_mc && a.ldb == a.N && gemm_takes_stored_weight(a)) {
      GemmArgs g = a;
      g.b_mc = 0; g.ldb = a.K;
      cfg = chosen_cfg(g, a.M, may_split);
    }
    if (a.geglu == 1 && (cfg < 6 || cfg == 11 || cfg == 15 || cfg == 16 || cfg > 18)) return set_error(DP_EUNSUPPORTED, "gemm: the forced configuration does not have the fused GeGLU forward");
    // (11 and 12 name tiles that are there under 20 and 7 as well: callers may force them)
    switch (cfg) {
      case 1: return launch_bf16_layout<256, 128, 64, 4, 2>(a, s);
      case 2: return launch_bf16_layout<256, 256, 64, 2, 4>(a, s);
      case 3: return launch_bf16_layout<128, 256, 64, 2, 4>(a, s);
      case 4: return launch_bf16_layout<256, 128, 32, 4, 2>(a, s);
      case 5: return launch_bf16_layout<128, 128, 32, 2, 2>(a, s);
      case 6: return launch_dtl_layout<256, 256, 32, 4, 2, 4>(a, s);
      case 7: case 12: return launch_dtl_layout<256, 128, 32, 4, 4, 2>(a, s);
      case 8: return launch_dtl_layout<128, 128, 32, 4, 2, 2>(a, s);
      case 9: return launch_dtl_layout<256, 128, 64, 3, 4, 2>(a, s);
      case 10: return launch_dtl_layout<128, 128, 64, 3, 2, 2>(a, s);
      case 13: return launch_dtl_layout<128, 128, 64, 4, 4, 2>(a, s);   // eight waves on a 128x128 tile; three buffers instead of four, one workgroup a CU either way: 4 to 8 % more
      case 14: return launch_dtl_layout<128, 128, 32, 4, 4, 2>(a, s);
      // small tiles: many workgroups for problems of a few hundred rows (contraction-contiguous operands only: the chunk
      // permutation of a contraction-strided tile needs at least 128 columns)
      // Four buffers of 64x64 take the ring's loop, three leave a CU room for a third workgroup (us, contraction 3072 / 4608, four and three: 192 tiles 11.2 / 15.8 and
      // 15.2 / 28.8, 480 20.7 / 29.0 and 22.4 / 31.5, 540 28.7 / 40.9 and 27.4 / 38.5, 768 30.6 / 44.5 and 30.4 / 42.6, two full rounds of 512 41.4 / 59.8 and 46.2 / 66.7).
      case 15:
      case 16:
        if (a.a_mc || a.b_mc || a.K % 64) return set_error(DP_EUNSUPPORTED, "gemm: the forced 64-row configurations need contraction-contiguous operands and K % 64 == 0");
        if (cfg == 15) {
          const long tiles = (long)((a.M + 63) / 64) * ((a.N + 63) / 64) * dtl_splits<64, 64, 64>(a, 2 * kCUs);
          return tiles <= 2 * kCUs ? launch_dtl_cfg<64, 64, 64, 4, 2, 2, false, false>(a, s) : launch_dtl_cfg<64, 64, 64, 3, 2, 2, false, false>(a, s);
        }
        return launch_dtl_cfg<64, 128, 64, 3, 2, 2, false, false>(a, s);
      case 17: return launch_pp<PpTile<256, 128, 128, 4, 2>>(a, s);
      case 18: return launch_pp<PpTile<256, 64, 64, 4, 2>>(a, s);
      case 19: return launch_pp<PpTile<256, 128, 64, 4, 2>>(a, s);
      case 21: case 22: case 23: case 24:
        return launch_gemm_dw_group(&a, 1, gemm_dw_group_plan(&a, 1, cfg - 20, a.splitk_ws ? a.splitk_ws_bytes : 0), s);
      case 11: case 20:
        if (cfg == 11 && a.K % 64) return set_error(DP_EUNSUPPORTED, "gemm: the forced 256x160 configuration needs K % 64 == 0");
        return launch_pp<PpTile<256, 96, 64, 4, 2, 16>>(a, s);
      case 25: return launch_wave<WaveTile<4, 2, 2, 2>, WaveTile<4, 2, 2>>(a, kWave[0], s);
      case 26: return launch_wave<WaveTile<4, 2, 3>, WaveTile<4, 2, 3>>(a, kWave[1], s);
      case 27: return launch_wave<WaveTile<4, 4, 3>, WaveTile<4, 4, 3>>(a, kWave[2], s);
      case 28: return launch_wave<WaveTile<4, 4, 4>, WaveTile<4, 4, 4>>(a, kWave[3], s);
      case 29: return launch_wave<WaveTile<8, 1, 1>, WaveTile<8, 1, 1>>(a, kWave[4], s);
      case 30: return launch_wave<WaveTile<8, 1, 2>, WaveTile<8, 1, 2>>(a, kWave[5], s);
      case 31: return launch_wave<WaveTile<8, 1, 3>, WaveTile<8, 1, 3>>(a, kWave[6], s);
      default: break;
    }
    return launch_bf16_layout<128, 128, 64, 2, 2>(a, s);
  }
  return launch_gemm_f32(a, s);
}

}  // namespace dp
