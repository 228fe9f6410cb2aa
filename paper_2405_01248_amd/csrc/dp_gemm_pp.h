// Main loop and epilogue of the 256-row MFMA tiles whose eight waves work in two alternating groups.
//
// A SIMD of a CDNA4 compute unit holds two of the workgroup's eight waves.  In a loop that keeps all waves in step both
// of them fetch fragments at the same time and multiply at the same time, so LDS and matrix pipe take turns: the
// 256x256x32 tile with one barrier per k-tile runs at 1.19 PFLOP/s on 8192^3.  Here waves 4-7 run one barrier behind waves
// 0-3: while one wave of a SIMD issues the MFMAs of a quarter of its tile, the other one fetches the fragments of
// its next quarter and issues the global -> LDS copies.  Every quarter of a k-tile is two slots, separated by barriers:
//   fetch slot:    LDS reads of one operand half, copies of one half two k-tiles ahead, one counted wait
//   compute slot:  the MFMAs of one (row half, column half) combination at raised wave priority
// The tile is cut into two row halves and two column halves (which may differ in width); a wave owns an equal share of
// each.  Order of a k-tile t (rows x columns): A0 B0, A0 B1, A1 B0, A1 B1, fetching
// A0(t), B1(t), A1(t), B0(t + 1) ahead of them, so each fetch slot reads one half and each half is read once.
//
// LDS: two stages of [A0 A1 B0 B1], 64-deep k-tiles (128-byte rows, 16-byte chunk c of row r at c ^ ((r >> 1) & 7)).  The
// stage of k-tile t receives k-tile t + 2 half by half once both groups are past their reads of a half: with S the slot in which
// the leading group fetches A0(t), a half fetched in slot s by the leading group is fetched in s + 1 and has arrived in s + 2
// for the trailing one, and it is overwritten from slot s + 4 on.  Each half is copied six quarters ahead of its fetch
// and waited for one quarter ahead of it (by then five younger halves are in flight), so that the barriers between publish it.
#pragma once
#include "dp_gemm_epilogue.h"
#include <type_traits>

namespace dp {

typedef __attribute__((ext_vector_type(8))) int i32x8;

// BN0, BN1: columns of the two column halves.  FR: rows and columns of the MFMA (32: 32x32x16, 16: 16x16x32; the latter allows
// halves that are multiples of 16 per wave, e.g. 96 + 64).
template <int BM_, int BN0_, int BN1_, int WGM_, int WGN_, int FR_ = 32>
struct PpTile {
  static constexpr int BM = BM_, BN0 = BN0_, BN1 = BN1_, BN = BN0_ + BN1_, BK = 64, WGM = WGM_, WGN = WGN_, NW = WGM * WGN, FR = FR_;
  typedef PpTile<BM_, BN0_, BN1_, WGM_, WGN_, 16> On16;                              // the same tile on the smaller instruction
  static constexpr int SM = BM / 2 / WGM, SN0 = BN0 / WGN, SN1 = BN1 / WGN;         // a wave's share of a row half and of the column halves
  static constexpr int TM = SM / FR, TN0 = SN0 / FR, TN1 = SN1 / FR, TN = TN0 + TN1, TNM = TN0 > TN1 ? TN0 : TN1;
  static constexpr int A_HALF = BM / 2 * 128, B0_BYTES = BN0 * 128, B1_BYTES = BN1 * 128, STAGE = 2 * A_HALF + B0_BYTES + B1_BYTES;
  static constexpr int OB0 = 2 * A_HALF, OB1 = OB0 + B0_BYTES;                        // stage: A0 A1 B0 B1
  // copies per wave of one half; where the pieces of a half do not divide evenly the surplus slots repeat the last piece
  static constexpr int LA = A_HALF / 1024 / NW, LB0 = (B0_BYTES / 1024 + NW - 1) / NW, LB1 = (B1_BYTES / 1024 + NW - 1) / NW;
  static constexpr int W = SN0 + SN1, C_LD = W + (FR == 16 ? 4 : 8);                 // epilogue slab of a wave: 32 rows x W columns
  static constexpr size_t EPI_BYTES = (size_t)NW * 32 * C_LD * 4;
  static constexpr size_t BYTES = 2 * (size_t)STAGE > EPI_BYTES ? 2 * (size_t)STAGE : EPI_BYTES;
  typedef typename std::conditional<FR == 32, f32x16, f32x4>::type acc_t;
  static constexpr int ACC_REGS = FR == 32 ? 16 : 4;
  static_assert(NW == 8 && SM % FR == 0 && SN0 % FR == 0 && SN1 % FR == 0 && SM % 32 == 0 && W % 16 == 0, "tile shape");
  static_assert(A_HALF % (1024 * NW) == 0 && BYTES <= 160 * 1024, "tile shape");
};

// ---- operands with the contraction contiguous: rows of 128 bytes
__device__ __forceinline__ int pp_key(int r) { return (r >> 1) & 7; }
// Row inside a half and the source chunk behind piece `piece` (1 KB: 8 rows of 128 bytes) for this lane.
__device__ __forceinline__ int pp_piece_row(int piece, int lane) { return piece * 8 + (lane >> 3); }
__device__ __forceinline__ int pp_piece_chunk(int row, int lane) { return (lane & 7) ^ pp_key(row); }
// ---- operands with the contraction strided (dW = dy^T x): 64 k-rows of COLS columns, read with the transposing LDS load.
// The four k-rows that 32 lanes of that load touch have to lie in four different 64-byte bank groups: chunk c of k-row k sits
// at c ^ 4 (k & 3), in rows of only 128 bytes (which alternate between the two halves of the banks by themselves) at c ^ 4 ((k >> 1) & 1); rows of 192 bytes
// begin in four different groups as they are, and rows of 64 bytes are those groups.
template <int COLS> __device__ __forceinline__ int pp_mc_swz(int c, int k) {
  static_assert(COLS % 64 == 0 || COLS == 96 || COLS == 32, "row length");
  return COLS % 128 == 0 ? c ^ (4 * (k & 3)) : (COLS % 64 == 0 ? c ^ (4 * ((k >> 1) & 1)) : c);
}
template <int COLS> __device__ __forceinline__ int pp_mc_piece_k(int piece, int lane) { return piece * (512 / COLS) + lane / (COLS / 8); }
template <int COLS> __device__ __forceinline__ int pp_mc_piece_chunk(int k, int lane) { return pp_mc_swz<COLS>(lane % (COLS / 8), k); }
// Byte offset inside a half of this lane's part of the fragment with first column col0 and first k-row 0; the other
// k-rows are constant distances away: k0 * COLS * 2 bytes, and the second half of a fragment 4 * COLS * 2 (k + 4 has the same permutation).
template <int COLS>
__device__ __forceinline__ uint32_t pp_mc_offset(int col0, int lane) {
  const int b = lane >> 4, j = lane & 15, k = 8 * (b >> 1) + (j >> 2), c = col0 / 8 + 2 * (b & 1) + ((j & 3) >> 1);
  return (uint32_t)(k * COLS + pp_mc_swz<COLS>(c, k) * 8 + 4 * (j & 1)) * 2u;
}
// The copies of k-tile 0, which may be issued before the loop's own (AHEAD).
template <class T, class CopyA, class CopyB>
__device__ __forceinline__ void pp_first_k_tile(unsigned char* smem, CopyA copy_a, CopyB copy_b) {
  copy_b(std::integral_constant<int, 0>(), 0, smem + T::OB0); copy_a(std::integral_constant<int, 0>(), 0, smem);
  copy_b(std::integral_constant<int, 1>(), 0, smem + T::OB1); copy_a(std::integral_constant<int, 1>(), 0, smem + T::A_HALF);
}
// copy_a(half, t, dst) / copy_b(half, t, dst): issue this wave's LA / LB0, LB1 copies of a half of k-tile t to dst (the
// half's first byte in LDS).  t may be nk or nk + 1: then the copies have to be issued all the same (the waits count them), from
// outside the buffers, so that they move nothing (or from anywhere inside them: what they bring is not multiplied).
// MC: both operands have the contraction strided.  colsum (MC only): a wave-uniform flag; csum[half][i] then receives
// the sum over the contraction of row i of the wave's part of A (this lane's k-slots; lanes l and l + 32 hold the two halves).
// AHEAD: the copies of k-tile 0 (pp_first_k_tile) are on their way already.
// PAIRS: two k-tiles a round of the loop, so that the stages' addresses are constants.  What a fetch slot issues beside its reads and copies counts: a
// wave issues an instruction every four cycles or so, and with 44 to 64 scalar and 15 to 23 vector ones a k-tile the slots of a 256x128 tile took longer
// than the 128 cycles of matrix work beside them; 26 to 35 and 0 to 6 are left.  bf16 products of one tile a CU: 8192 x 640, K = 640 / 5120 12.3 -> 11.3 / 57.3
// -> 54.3 us, 8192 x 1152, K = 1152 / 4608 24.4 -> 23.1 / 78.3 -> 73.2.  Not where workgroups walk over tiles (32768 x 1280, K = 320 40.7 -> 43.0 us, 8192^3 739 -> 721) nor
// for FP8 (8192 x 4608, K = 1152 48.7 -> 52.2), whose scalar registers run out, and not where the second set of addresses spills: the 512x128 convolution, and 256x256 tiles
// of a contraction that is no multiple of 64, whose last k-tile is masked lane by lane (4096 x 4096, K = 72 / 432 / 1080 / 4104, us: 12.7 / 21.2 / 37.4 / 111.2, with
// two k-tiles a round and 8 to 16 bytes of scratch a lane 13.0 / 21.6 / 37.7 / 110.4; fewer tiles than CUs, K = 1080: 25.7 and 24.5, where 256x128 tiles take 16.9).
template <class T, bool FP8, bool MC, bool AHEAD = false, bool PAIRS = true, class CopyA, class CopyB>
__device__ __forceinline__ void pp_main_loop(typename T::acc_t (&acc)[2][T::TM][T::TN], unsigned char* smem, int nk, int wm, int wn, bool trailing,
                                             int lane, CopyA copy_a, CopyB copy_b, bool colsum, float (&csum)[2][T::TM]) {
  constexpr int TM = T::TM, TN0 = T::TN0, LA = T::LA, LB0 = T::LB0, LB1 = T::LB1, FR = T::FR;
  constexpr int KS = FP8 ? 2 : (FR == 32 ? 4 : 2);
  static_assert(!(MC || FP8) || FR == 32, "fp8 and contraction-strided operands use the 32x32 instructions");
  const int lr = lane % FR, q = lane / FR;
  bf16x8 fa[FP8 ? 1 : TM][KS], fb[2][FP8 ? 1 : T::TNM][KS];
  i32x8 qa[FP8 ? TM : 1][2], qb[2][FP8 ? T::TNM : 1][2];
  u32x2 ra[MC ? TM : 1][4][2], rb[2][MC ? T::TNM : 1][4][2];         // transposed fragments, 8 bytes each, as they arrive
  uint32_t oa[2][TM], ob0[2][T::TN0], ob1[2][T::TN1];      // by stage: the second one is out of reach of an instruction's offset
  if constexpr (MC) {
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const uint32_t base = lds_address(smem) + (uint32_t)(st * T::STAGE);
#pragma unroll
      for (int i = 0; i < TM; ++i) oa[st][i] = base + pp_mc_offset<T::BM / 2>(wm * T::SM + i * 32, lane);
#pragma unroll
      for (int j = 0; j < TN0; ++j) ob0[st][j] = base + T::OB0 + pp_mc_offset<T::BN0>(wn * T::SN0 + j * 32, lane);
#pragma unroll
      for (int j = 0; j < T::TN1; ++j) ob1[st][j] = base + T::OB1 + pp_mc_offset<T::BN1>(wn * T::SN1 + j * 32, lane);
    }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      csum[a][i] = 0.f;
#pragma unroll
      for (int j = 0; j < T::TN; ++j)
#pragma unroll
        for (int r = 0; r < T::ACC_REGS; ++r) acc[a][i][j][r] = 0.f;
    }

  auto chunk16 = [&](const unsigned char* half, int row, int chunk) {
    return *reinterpret_cast<const u32x4*>(half + row * 128 + ((chunk ^ pp_key(row)) * 16));
  };
  auto fetch8 = [&](const unsigned char* p, int r, int ks) {
    const u32x4 lo = chunk16(p, r, 4 * ks + 2 * q), hi = chunk16(p, r, 4 * ks + 2 * q + 1);
    return __builtin_bit_cast(i32x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto fetch_a = [&](auto stage, auto hc) {
    constexpr int h = decltype(hc)::value;
    const unsigned char* p = smem + stage * T::STAGE + h * T::A_HALF;
    if constexpr (MC) {
      constexpr int ROW = T::BM / 2 * 2, HALF = h * T::A_HALF;
#pragma unroll
      for (int i = 0; i < TM; ++i)
        static_for<4>([&](auto ks) { lds_read_tr_raw<HALF + ks * 16 * ROW>(ra[i][ks][0], oa[stage][i]); lds_read_tr_raw<HALF + (ks * 16 + 4) * ROW>(ra[i][ks][1], oa[stage][i]); });
      return;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int r = wm * T::SM + i * FR + lr;
        if constexpr (FP8) qa[i][ks] = fetch8(p, r, ks);
        else fa[i][ks] = __builtin_bit_cast(bf16x8, chunk16(p, r, (64 / FR) * ks + q));
      }
  };
  auto fetch_b = [&](auto stage, auto hc) {
    constexpr int h = decltype(hc)::value;
    const unsigned char* p = smem + stage * T::STAGE + (h ? T::OB1 : T::OB0);
    if constexpr (MC) {
      constexpr int ROW = (h ? T::BN1 : T::BN0) * 2;
#pragma unroll
      for (int j = 0; j < (h ? T::TN1 : TN0); ++j) {
        const uint32_t at = h ? ob1[stage][h ? j : 0] : ob0[stage][h ? 0 : j];
        static_for<4>([&](auto ks) { lds_read_tr_raw<ks * 16 * ROW>(rb[h][j][ks][0], at); lds_read_tr_raw<(ks * 16 + 4) * ROW>(rb[h][j][ks][1], at); });
      }
      return;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int j = 0; j < (h ? T::TN1 : TN0); ++j) {
        const int r = wn * (h ? T::SN1 : T::SN0) + j * FR + lr;
        if constexpr (FP8) qb[h][j][ks] = fetch8(p, r, ks);
        else fb[h][j][ks] = __builtin_bit_cast(bf16x8, chunk16(p, r, (64 / FR) * ks + q));
      }
  };
  // MC: fragments from what the transposing loads delivered
  auto join = [](u32x2& lo, u32x2& hi) {
    lds_arrived(lo); lds_arrived(hi);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3));
  };
  auto arrived_a = [&]() {
    if constexpr (MC) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) fa[i][ks] = join(ra[i][ks][0], ra[i][ks][1]);
    }
  };
  auto arrived_b = [&](auto hc) {
    constexpr int h = decltype(hc)::value;
    if constexpr (MC) {
#pragma unroll
      for (int j = 0; j < (h ? T::TN1 : TN0); ++j)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) fb[h][j][ks] = join(rb[h][j][ks][0], rb[h][j][ks][1]);
    }
  };
  // new_a / new_b: whether the row / column half is multiplied for the first time since it was fetched
  auto multiply = [&](int ha, auto hc, bool new_a, bool new_b) {
    constexpr int h = decltype(hc)::value;
    wait_lgkmcnt0();
    if (new_a) arrived_a();
    if (new_b) arrived_b(hc);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < (h ? T::TN1 : TN0); ++j) {
          auto& c = acc[ha][i][(h ? TN0 : 0) + j];
          if constexpr (FP8) c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(qa[i][ks], qb[h][j][ks], c, 0, 0, 0, 127, 0, 127);
          else if constexpr (FR == 32) c = mfma32(fa[i][ks], fb[h][j][ks], c);
          else c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[h][j][ks], fa[i][ks], c, 0, 0, 0);      // transposed: see pp_acc_to_slab
        }
    if constexpr (MC && h == 0) {
      // the bias gradient beside a weight gradient: vector work of a few workgroups under their matrix work
      if (colsum) {
        const bf16x2 one = {(bf16)1.f, (bf16)1.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const bf16x8 v = fa[i][ks];
            csum[ha][i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 0, 1), one, csum[ha][i], false);
            csum[ha][i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 2, 3), one, csum[ha][i], false);
            csum[ha][i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 4, 5), one, csum[ha][i], false);
            csum[ha][i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 6, 7), one, csum[ha][i], false);
          }
      }
    }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    barrier_nofence();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto slot_end = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    barrier_nofence();
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr std::integral_constant<int, 0> H0{};
  constexpr std::integral_constant<int, 1> H1{};
  auto k_tile = [&](auto stage, auto other, int t) {
    unsigned char* here = smem + stage * T::STAGE;
    fetch_a(stage, H0);
    copy_a(H1, t + 1, smem + other * T::STAGE + T::A_HALF);
    wait_vmcnt<3 * LA + LB0 + LB1>();
    slot_end();
    multiply(0, H0, true, true);
    fetch_b(stage, H1);
    copy_b(H0, t + 2, here + T::OB0);
    wait_vmcnt<2 * LA + 2 * LB0 + LB1>();
    slot_end();
    multiply(0, H1, false, true);
    fetch_a(stage, H1);
    copy_a(H0, t + 2, here);
    wait_vmcnt<3 * LA + LB0 + LB1>();
    slot_end();
    multiply(1, H0, true, false);
    fetch_b(other, H0);                 // past the last k-tile: not used
    copy_b(H1, t + 2, here + T::OB1);
    wait_vmcnt<2 * LA + LB0 + 2 * LB1>();
    slot_end();
    multiply(1, H1, false, false);
  };

  if constexpr (!AHEAD) pp_first_k_tile<T>(smem, copy_a, copy_b);
  copy_b(H0, 1, smem + T::STAGE + T::OB0); copy_a(H0, 1, smem + T::STAGE); copy_b(H1, 1, smem + T::STAGE + T::OB1);
  wait_vmcnt<2 * LA + LB0 + 2 * LB1>();        // the first B0 and A0 are there
  barrier_nofence();
  fetch_b(H0, H0);
  if constexpr (MC) {
    // the transposing loads are not in the compiler's books: a register it copies on the way into the loop has to hold its value by then
    wait_lgkmcnt0();
#pragma unroll
    for (int j = 0; j < TN0; ++j)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) { lds_arrived(rb[0][j][ks][0]); lds_arrived(rb[0][j][ks][1]); }
  }
  if (trailing) barrier_nofence();
  if constexpr (PAIRS) {
    for (int t = 0;; t += 2) {
      k_tile(H0, H1, t);
      if (t + 1 >= nk) break;
      k_tile(H1, H0, t + 1);
      if (t + 2 >= nk) break;
    }
  } else {
    for (int t = 0; t < nk; ++t) k_tile(t & 1, ~t & 1, t);
  }
  if (!trailing) barrier_nofence();
  wait_vmcnt<0>();                      // the epilogue reuses the stages
  __syncthreads();
}

// ------------------------------------------------------------------ epilogue
// One kernel per kind: what a kind does not use is not compiled into it, so the loops can be unrolled and all
// global operands of a 32-row slab (residual, saved pre-activation, gate) are requested before the first of them is
// needed; in the rolled, all-purpose epilogue each 8-column group waits for its own operands in turn.
enum PpEpi { PE_PLAIN = 0, PE_F32, PE_RES, PE_RESH, PE_GATE, PE_ACT1, PE_ACT2, PE_ACT3, PE_DACT1, PE_DACT2, PE_GEGLU1, PE_GEGLU2 };

// What a forward pass saves for the backward is read again after hundreds of megabytes of other tensors: it passes the caches by instead of
// taking the place of what the next kernel reads (a step of 1 U-Net block 8 x 4096 x 320: 1648 -> 1630 us, 8 x 1024 x 640: 838 -> 834,
// 2 DiT blocks 32 x 256 x 1152: 2249 -> 2237).  Likewise the last read of it; for the derivative of an activation, which is read
// while the product's own operands are few, that measured no difference.
__device__ __forceinline__ void store_later(bf16* p, bf16x8 v) { __builtin_nontemporal_store(v, reinterpret_cast<bf16x8*>(p)); }
__device__ __forceinline__ bf16x8 load_last(const bf16* p) { return __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(p)); }

template <int KIND> struct PpIn { f32x4 r0, r1; bf16x8 a, b; };

template <int KIND>
__device__ __forceinline__ void pp_load(const EpiParams<bf16>& e, int m, int n, PpIn<KIND>& in) {
  m = min(m, e.M - 1); n = min(n, e.N - 8);
  if constexpr (KIND == PE_F32) {
    if (!e.partial && e.accumulate) {
      const float* o = e.out32 + (size_t)m * e.ldo32 + n;
      in.r0 = *reinterpret_cast<const f32x4*>(o); in.r1 = *reinterpret_cast<const f32x4*>(o + 4);
    }
  }
  if constexpr (KIND == PE_RES || KIND == PE_GATE) {
    const float* rp = (const float*)e.residual + (size_t)m * e.ld_res + n;
    in.r0 = *reinterpret_cast<const f32x4*>(rp); in.r1 = *reinterpret_cast<const f32x4*>(rp + 4);
  }
  if constexpr (KIND == PE_RESH) in.a = *reinterpret_cast<const bf16x8*>((const bf16*)e.residual + (size_t)m * e.ld_res + n);
  if constexpr (KIND == PE_GATE) in.a = *reinterpret_cast<const bf16x8*>(e.gate + (size_t)(m / e.rows_per_batch) * e.gate_ld + n);
  if constexpr (KIND == PE_DACT1 || KIND == PE_DACT2) in.a = *reinterpret_cast<const bf16x8*>(e.dact_pre + (size_t)m * e.ld_dact + n);
  if constexpr (KIND == PE_GEGLU2) {
    const bf16* up = e.geglu_u + (size_t)m * e.ld_geglu + n;
    in.a = load_last(up); in.b = load_last(up + e.geglu_inner);
  }
}

// Takes delivery of the operands ahead of the branch around their use.  Behind the branch alone, the compiler would have to count them as on their way still
// when their registers are used again, which in a kernel that walks over tiles is inside the main loop: a wait on each k-tile.
template <int KIND>
__device__ __forceinline__ void pp_arrived(PpIn<KIND>& in) {
  if constexpr (KIND == PE_F32 || KIND == PE_RES || KIND == PE_GATE) asm volatile("" : "+v"(in.r0), "+v"(in.r1));
  if constexpr (KIND == PE_RESH || KIND == PE_GATE || KIND == PE_DACT1 || KIND == PE_DACT2 || KIND == PE_GEGLU2) asm volatile("" : "+v"(in.a));
  if constexpr (KIND == PE_GEGLU2) asm volatile("" : "+v"(in.b));
}
template <int KIND>
__device__ __forceinline__ void pp_finish(const EpiParams<bf16>& e, int m, int n, float (&v)[8], const PpIn<KIND>& in, const float (&bias)[8]) {
  if constexpr (KIND == PE_F32) {
    float* o = e.partial ? e.partial + ((size_t)blockIdx.z * e.M + m) * e.N + n : e.out32 + (size_t)m * e.ldo32 + n;
    if (!e.partial && e.accumulate) {
#pragma unroll
      for (int t = 0; t < 4; ++t) { v[t] += in.r0[t]; v[4 + t] += in.r1[t]; }
    }
    *reinterpret_cast<f32x4*>(o) = *reinterpret_cast<const f32x4*>(&v[0]);
    *reinterpret_cast<f32x4*>(o + 4) = *reinterpret_cast<const f32x4*>(&v[4]);
    return;
  }
  if constexpr (KIND == PE_PLAIN) {
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] *= e.out_scale;
  }
#pragma unroll
  for (int t = 0; t < 8; ++t) v[t] += bias[t];
  bf16x8 o, o1;
  if constexpr (KIND == PE_GEGLU2) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float gt = (float)in.b[t];
      o[t] = (bf16)(v[t] * gelu_erf_f(gt));
      o1[t] = (bf16)(v[t] * (float)in.a[t] * gelu_erf_grad_f(gt));
    }
    bf16* op = e.out + (size_t)m * e.ldo + n;
    *reinterpret_cast<bf16x8*>(op) = o;
    *reinterpret_cast<bf16x8*>(op + e.geglu_inner) = o1;
    return;
  }
  if constexpr (KIND == PE_ACT1 || KIND == PE_ACT2 || KIND == PE_ACT3 || KIND == PE_GATE) {
    if (e.pre_out) {
#pragma unroll
      for (int t = 0; t < 8; ++t) o[t] = (bf16)v[t];
      store_later(e.pre_out + (size_t)m * e.ld_pre + n, o);
    }
  }
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    if constexpr (KIND == PE_ACT1) v[t] = gelu_erf_f(v[t]);
    if constexpr (KIND == PE_ACT2) v[t] = gelu_tanh_f(v[t]);
    if constexpr (KIND == PE_ACT3) v[t] = quick_gelu_f(v[t]);
    if constexpr (KIND == PE_DACT1) v[t] *= gelu_erf_grad_f((float)in.a[t]);
    if constexpr (KIND == PE_DACT2) v[t] *= gelu_tanh_grad_f((float)in.a[t]);
    if constexpr (KIND == PE_GATE) v[t] *= (float)in.a[t];
    if constexpr (KIND == PE_RESH) v[t] += (float)in.a[t];
    if constexpr (KIND == PE_RES || KIND == PE_GATE) v[t] += t < 4 ? in.r0[t & 3] : in.r1[t & 3];
  }
  if constexpr (KIND == PE_RES || KIND == PE_GATE) {
    if (e.out_fused_f32) {
      float* op = reinterpret_cast<float*>(e.out) + (size_t)m * e.ldo + n;
      *reinterpret_cast<f32x4*>(op) = *reinterpret_cast<const f32x4*>(&v[0]);
      *reinterpret_cast<f32x4*>(op + 4) = *reinterpret_cast<const f32x4*>(&v[4]);
      return;
    }
  }
#pragma unroll
  for (int t = 0; t < 8; ++t) o[t] = (bf16)v[t];
  *reinterpret_cast<bf16x8*>(e.out + (size_t)m * e.ldo + n) = o;
}

__device__ __forceinline__ void pp_bias(const bf16* bias, int n, float (&b)[8]) {
#pragma unroll
  for (int t = 0; t < 8; ++t) b[t] = 0.f;
  if (bias) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(bias + n);
#pragma unroll
    for (int t = 0; t < 8; ++t) b[t] = (float)v[t];
  }
}
__device__ __forceinline__ void pp_slab_row(const float* p, float (&v)[8]) {
  *reinterpret_cast<f32x4*>(&v[0]) = *reinterpret_cast<const f32x4*>(p);
  *reinterpret_cast<f32x4*>(&v[4]) = *reinterpret_cast<const f32x4*>(p + 4);
}

// Rows part * RPS .. + RPS - 1 of the 32 rows i32 of a wave's row half, on their way from its accumulators to its slab.  On the 16x16x32 instruction
// the products are formed transposed (weights as the row operand), so that a lane has one row and four neighbouring columns: one write of 16 bytes where
// it took four of 4.  8192 x 1920, K = 640 on 256x256 tiles 25.0 -> 24.1 us, 8192 x 5120 on 256x192 73.7 -> 71.3.  A lane of the 32x32x16 one would have
// rows of both slabs of 16, half of the lanes writing at a time: 8192 x 5120 on 256x128 75.0 -> 77.8 us, the 8-bit product of 8192 x 4608 47.5 -> 50.
template <class T, int RPS>
__device__ __forceinline__ void pp_acc_to_slab(float* Cw, const typename T::acc_t (&acc)[T::TM][T::TN], int i32, int part, int lane) {
  if constexpr (T::FR == 16) {
#pragma unroll
    for (int i = RPS == 32 ? 0 : part; i < (RPS == 32 ? 2 : part + 1); ++i)
#pragma unroll
      for (int j = 0; j < T::TN; ++j) *reinterpret_cast<f32x4*>(Cw + (i * 16 + lane % 16 - part * RPS) * T::C_LD + j * 16 + 4 * (lane / 16)) = acc[2 * i32 + i][j];
  } else {
#pragma unroll
    for (int j = 0; j < T::TN; ++j)
#pragma unroll
      for (int r = part * (RPS / 2); r < (part + 1) * (RPS / 2); ++r) Cw[(acc_row(r, lane >> 5) - part * RPS) * T::C_LD + j * 32 + lane % 32] = acc[i32][j][r];
  }
}

// A wave turns its accumulators through LDS, 32 rows x W columns at a time, into 8 consecutive columns per lane.  Its two
// column parts lie in different halves of the tile; the fused GeGLU forward has the values of an output in the first and
// their gates in the second half (the B loader sees to that).  RPS: rows per slab.  ahead(): called once the operands of the first slab are requested.
template <class T, int KIND, int RPS = 32, class Ahead>
__device__ __forceinline__ void pp_epilogue(const typename T::acc_t (&acc)[2][T::TM][T::TN], unsigned char* smem, const EpiParams<bf16>& e, int m0, int n0,
                                            int wave, int wm, int wn, int lane, Ahead ahead) {
  float* Cw = reinterpret_cast<float*>(smem) + wave * RPS * T::C_LD;
  constexpr bool GG1 = KIND == PE_GEGLU1;
  static_assert(!GG1 || T::SN0 == T::SN1, "the fused GeGLU needs equal column halves");
  constexpr int CH = (GG1 ? T::SN0 : T::W) / 8, NIT = (RPS * CH + 63) / 64, PARTS = 32 / RPS;
  static_assert(RPS == 32 || (RPS == 16 && RPS * CH % 64 == 0), "slab");
  constexpr bool FIXED = 64 % CH == 0;              // a lane keeps its columns over the rows of a slab
  const int n_end = GG1 ? e.geglu_inner : e.N;
  auto column = [&](int lc) { return GG1 ? n0 / 2 + wn * T::SN0 + lc : n0 + (lc < T::SN0 ? wn * T::SN0 + lc : T::BN0 + wn * T::SN1 + lc - T::SN0); };
  float bias[8], bias_g[8];
  // Otherwise the bias of every pass is requested here.  Beside its use, each request stands behind the stores of the pass before, and memory operations
  // are counted in order: the pass waits until those stores are in memory.
  bf16x8 bias_it[FIXED ? 1 : NIT];
  {
    const rsrc_t rb = make_rsrc(e.bias, e.bias ? 2u * (uint32_t)n_end : 0u);      // (no bias: a buffer of no size reads as zeros)
#pragma unroll
    for (int it = 0; it < (FIXED ? 1 : NIT); ++it) bias_it[it] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rb, 2 * column(((it * 64 + lane) % CH) * 8), 0, 0));
  }
  bf16x8 bias_g_it;
  if constexpr (GG1) bias_g_it = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(e.bias ? e.bias + e.geglu_inner : nullptr, e.bias ? 2u * (uint32_t)n_end : 0u), 2 * column((lane % CH) * 8), 0, 0));
#pragma unroll
  for (int s = 0; s < 2 * T::SM / RPS; ++s) {
    const int ha = s / (T::SM / RPS), i32 = s / PARTS % (T::SM / 32), part = s % PARTS;
    const int row0 = m0 + ha * (T::BM / 2) + wm * T::SM + i32 * 32 + part * RPS;
    PpIn<KIND> in[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int id = it * 64 + lane;
      pp_load<KIND>(e, row0 + min(id / CH, RPS - 1), column((id % CH) * 8), in[it]);
    }
    if (s == 0) {
      ahead();
#pragma unroll
      for (int t = 0; t < 8; ++t) { bias[t] = (float)bias_it[0][t]; if constexpr (GG1) bias_g[t] = (float)bias_g_it[t]; }
    }
    pp_acc_to_slab<T, RPS>(Cw, acc[ha], i32, part, lane);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int id = it * 64 + lane, lr = id / CH, lc = (id % CH) * 8, m = row0 + lr, n = column(lc);
      pp_arrived<KIND>(in[it]);
      if (RPS * CH % 64 != 0 && lr >= RPS) continue;
      float v[8];
      pp_slab_row(&Cw[lr * T::C_LD + lc], v);
      if constexpr (GG1) {
        float gt[8];
        pp_slab_row(&Cw[lr * T::C_LD + T::SN0 + lc], gt);
        if (m < e.M && n < n_end) {
          bf16x8 uv, ug, o;
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            uv[t] = (bf16)(v[t] + bias[t]); ug[t] = (bf16)(gt[t] + bias_g[t]);
            o[t] = (bf16)((float)uv[t] * gelu_erf_f((float)ug[t]));
          }
          if (e.pre_out) {
            bf16* up = e.pre_out + (size_t)m * e.ld_pre + n;
            store_later(up, uv);
            store_later(up + e.geglu_inner, ug);
          }
          *reinterpret_cast<bf16x8*>(e.out + (size_t)m * e.ldo + n) = o;
        }
      } else {
        if constexpr (!FIXED) {
#pragma unroll
          for (int t = 0; t < 8; ++t) bias[t] = (float)bias_it[it][t];
        }
        if (m < e.M && n < n_end) pp_finish<KIND>(e, m, n, v, in[it], bias);
      }
    }
    asm volatile("" ::: "memory");
  }
}

}  // namespace dp
