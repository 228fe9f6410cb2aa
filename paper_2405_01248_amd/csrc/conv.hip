// 3x3 convolution (zero padding 1, stride 1 or 2) of a channels-last bf16 tensor as an implicit GEMM
// on the MFMA pipeline: out[(b, i, j), o] = sum over (tap, c) of x[b, i * stride + u - 1, j * stride + v - 1, c] *
// w[o, tap * C_in + c], tap = 3u + v.  Rows of the product are output pixels, its contraction runs over the
// nine taps times the input channels; the A operand is never materialised: every thread gathers its 16-byte
// pieces of the input (8 channels of one pixel, which lie inside one tap because C_in is a multiple of 8)
// straight from the tensor, with zeros where the tap falls into the padding.  The kernel that takes every shape stages
// its tiles through registers into padded LDS tiles (double buffered); the layers of an encoder run on the ones further
// down, which copy to LDS directly.  v_mfma_f32_32x32x16_bf16 throughout; the
// epilogue is the GEMM kernels' (bias, optional residual in the storage dtype).  This is the layer class of
// the frozen image encoder (Sec. 2.1, Sec. 2.3: the non-trainable layers that take tens to hundreds of
// milliseconds and are cut into partial batches, Sec. 5).
#include "dp_device.h"
#include "dp_kernels.h"
#include "dp_errors.h"
#include "dp_ktime.h"
#include "dp_gemm_pp.h"
#include "dp_gemm_ring.h"

#include <algorithm>
#include <atomic>

namespace dp {

// Quotient by a divisor known at launch, for numerators below 2^31: three instructions instead of the thirty of a division.  The method is that of Granlund and
// Montgomery (Division by Invariant Integers using Multiplication, 1994): with 2^shift the power of two not below d and mul = floor(2^32 (2^shift - d) / d) + 1, the
// quotient is (floor(mul n / 2^32) + n) / 2^shift, whose sum stays below 2^32.
struct FastDiv { uint32_t mul, shift; };
static FastDiv make_fast_div(int d) {
  FastDiv f;
  f.shift = 0;
  while ((1ull << f.shift) < (unsigned)d) ++f.shift;
  f.mul = (uint32_t)((((1ull << f.shift) - (unsigned)d) << 32) / (unsigned)d + 1);
  return f;
}
__device__ __forceinline__ int fast_div(int n, FastDiv f) { return (int)((__umulhi((uint32_t)n, f.mul) + (uint32_t)n) >> f.shift); }

struct ConvParams {
  const bf16* x; const bf16* w;
  int H, W, Cin, Ho, Wo, stride;
  FastDiv by_px, by_wo;          // Ho * Wo, Wo
  int M, N, K;                   // output pixels, output channels, 9 * C_in
  int tiles_m, tiles_n, group_m;
  int taps_uniform;              // C_in % 64 == 0: a 64-deep k-tile lies inside one filter tap
  float* gn_partial; int gn_block;   // per (block of gn_block pixels, channel): sum and sum of squares of the output, or nullptr
  EpiParams<bf16> epi;
};

template <int BM, int BN, int WGM, int WGN>
struct ConvSmem {
  static constexpr int BK = 64, LD = BK + 8;
  static constexpr int WN = BN / WGN, C_LD = WN + 4;
  static constexpr size_t TILE_BYTES = 2 * (size_t)(BM + BN) * LD * 2;
  static constexpr size_t EPI_BYTES = (size_t)WGM * WGN * 32 * C_LD * 4;
  static constexpr size_t BYTES = TILE_BYTES > EPI_BYTES ? TILE_BYTES : EPI_BYTES;
};

template <int BM, int BN, int WGM, int WGN>
__global__ void __launch_bounds__(WGM * WGN * 64) conv3x3_bf16_kernel(const ConvParams p) {
  using S = ConvSmem<BM, BN, WGM, WGN>;
  constexpr int BK = S::BK, LD = S::LD, NT = WGM * WGN * 64;
  constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
  constexpr int A_PER = BM * BK / 8 / NT, B_PER = BN * BK / 8 / NT, ROWS_PER_PASS = NT / 8;
  static_assert((BM * BK / 8) % NT == 0 && (BN * BK / 8) % NT == 0 && NT % 8 == 0, "tile/threads mismatch");

  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16* As = reinterpret_cast<bf16*>(smem_raw);
  bf16* Bs = As + 2 * BM * LD;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 5, l32 = lane & 31;
  const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;
  int tile_m, tile_n;
  tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  // A thread stages chunk c8 (8 contraction values) of rows tid / 8 + i * ROWS_PER_PASS of both tiles.  The
  // output pixel behind an A row does not change along the contraction: decode it once.
  const int c8 = tid & 7, r0 = tid >> 3;
  int pix_b[A_PER], pix_h[A_PER], pix_w[A_PER];
  unsigned row_ok = 0;
#pragma unroll
  for (int i = 0; i < A_PER; ++i) {
    const int gm = m0 + r0 + i * ROWS_PER_PASS;
    row_ok |= (unsigned)(gm < p.M) << i;
    const int q = min(gm, p.M - 1);
    const int b = q / (p.Ho * p.Wo), rem = q - b * (p.Ho * p.Wo), ho = rem / p.Wo, wo = rem - ho * p.Wo;
    pix_b[i] = b; pix_h[i] = ho * p.stride - 1; pix_w[i] = wo * p.stride - 1;
  }

  bf16x8 ra[A_PER], rb[B_PER];
  unsigned oka = 0, okb = 0;
  auto load_global = [&](int kt) {
    const int k0 = kt * BK, gk = k0 + c8 * 8;
    int tap, ci;
    if (p.taps_uniform) { tap = k0 / p.Cin; ci = k0 - tap * p.Cin + c8 * 8; }      // tap: one scalar division per k-tile
    else { tap = gk / p.Cin; ci = gk - tap * p.Cin; }
    const bool kok = gk < p.K;
    tap = min(tap, 8); ci = min(ci, p.Cin - 8);
    const int u = tap / 3, v = tap - 3 * u;
    oka = 0; okb = 0;
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
      const int hi = pix_h[i] + u, wi = pix_w[i] + v;
      const bool ok = ((row_ok >> i) & 1) && kok && (unsigned)hi < (unsigned)p.H && (unsigned)wi < (unsigned)p.W;
      const int hc = min(max(hi, 0), p.H - 1), wc = min(max(wi, 0), p.W - 1);      // a valid address in any case
      ra[i] = *reinterpret_cast<const bf16x8*>(p.x + (((size_t)pix_b[i] * p.H + hc) * p.W + wc) * p.Cin + ci);
      oka |= (unsigned)ok << i;
    }
#pragma unroll
    for (int i = 0; i < B_PER; ++i) {
      const int gn = n0 + r0 + i * ROWS_PER_PASS;
      rb[i] = *reinterpret_cast<const bf16x8*>(p.w + (size_t)min(gn, p.N - 1) * p.K + min(gk, p.K - 8));
      okb |= (unsigned)(gn < p.N && kok) << i;
    }
  };
  auto store_lds = [&](int buf) {
    bf16* as = As + buf * BM * LD;
    bf16* bs = Bs + buf * BN * LD;
#pragma unroll
    for (int i = 0; i < A_PER; ++i)
      *reinterpret_cast<bf16x8*>(as + (r0 + i * ROWS_PER_PASS) * LD + c8 * 8) = ((oka >> i) & 1) ? ra[i] : zero8();
#pragma unroll
    for (int i = 0; i < B_PER; ++i)
      *reinterpret_cast<bf16x8*>(bs + (r0 + i * ROWS_PER_PASS) * LD + c8 * 8) = ((okb >> i) & 1) ? rb[i] : zero8();
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nkt = (p.K + BK - 1) / BK;
  load_global(0);
  store_lds(0);
  __syncthreads();
  for (int kt = 0; kt < nkt; ++kt) {
    const int buf = kt & 1;
    const bool more = kt + 1 < nkt;
    if (more) load_global(kt + 1);
    const bf16* as = As + buf * BM * LD;
    const bf16* bs = Bs + buf * BN * LD;
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(as + (wm0 + i * 32 + l32) * LD + ks * 16 + 8 * g);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(bs + (wn0 + j * 32 + l32) * LD + ks * 16 + 8 * g);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma32(fa[i], fb[j], acc[i][j]);
    }
    if (more) store_lds(buf ^ 1);
    __syncthreads();
  }
  // the operand tiles are dead past the last barrier: each wave reuses its slice of LDS for the epilogue
  float* Cw = reinterpret_cast<float*>(smem_raw) + wave * 32 * S::C_LD;
  wave_epilogue<TM, TN, WN, S::C_LD>(acc, Cw, p.epi, m0 + wm0, n0 + wn0, lane);
}


// ------------------------------------------------------------------ alternating wave groups
// The same product with the main loop of dp_gemm_pp.h.  Tiles travel global -> LDS without passing through registers
// (buffer_load ... lds, 16 bytes per lane, every lane with an address of its own, so the gather of the input pixels costs
// nothing extra).  A 64-deep k-tile lies inside one filter tap (C_in a multiple of 64): its source address is the
// output pixel's base address plus an offset that is the same for the whole wave, and a lane whose tap falls into the
// padding aims its copy past the end of the buffer, which the hardware answers with zeros.
// Measured on the 256 -> 256 channel layers at 256 x 256 pixels, 8 samples: see launch_conv3x3.
//
// Epilogue: bias, optional residual, bf16 store and, if asked, the first pass of a GroupNorm over the output: per channel the
// sum and the sum of squares of the stored (rounded) values over a block of pixels (ConvParams::gn_block).  They are formed in an order that no tile shape
// changes: in a band of 32 rows, the rows with equal r % 8 in ascending order, these eight sums pairwise by the bits of
// r from the highest down, then the block's bands in ascending order.
// Byte offset of the input pixel at the tap centre of output pixel m0 + row, plus this lane's 16-byte chunk of the tile row `row`, and
// the 9-bit set of taps that fall inside the image for that pixel (empty for rows past M).
__device__ __forceinline__ void conv_pixel(const ConvParams& p, int m0, int row, int lane, int& base, unsigned& taps) {
  const int gm = m0 + row, q = min(gm, p.M - 1), c = pp_piece_chunk(row, lane);
  const int b = fast_div(q, p.by_px), rem = q - b * (p.Ho * p.Wo), ho = fast_div(rem, p.by_wo), wo = rem - ho * p.Wo;
  const int hc = ho * p.stride, wc = wo * p.stride;
  base = (int)(2u * ((uint32_t)((b * p.H + hc) * p.W + wc) * (uint32_t)p.Cin + (uint32_t)c * 8u));
  const unsigned cols = (wc > 0 ? 1u : 0u) | 2u | (wc + 1 < p.W ? 4u : 0u);      // (the centre tap is always inside)
  const unsigned m = (hc > 0 ? cols : 0u) | cols << 3 | (hc + 1 < p.H ? cols << 6 : 0u);
  taps = gm < p.M ? m : 0u;
}

// Reduction over lanes of two values at once, by v_permlane*_swap: the lower half of the wave (16-lane row of each pair) gets a's sum of both
// halves, the upper one b's.  One swap and one add for two values, no LDS: through ds_bpermute the sums below took 64 LDS operations per band.
__device__ __forceinline__ float fold_halves32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
  const uint32_t lo = r[0], hi = r[1];
  return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}
__device__ __forceinline__ float fold_halves16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
  const uint32_t lo = r[0], hi = r[1];
  return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}
template <int N> __device__ __forceinline__ float row_rotate(float v) {      // lane i of a row of 16 gets lane (i - N) mod 16
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xF, 0xF, true));
}
// Sums over the 64 / CH rows of a pass (lane = row * CH + chunk) of v[0..7] and v[8..15], by the bits of the row from the highest down; stores the
// sums of v[0..7] at dst[0..7], those of v[8..15] at dst[ld + 0..7].  CH 4: bit 5 of the lane is summed already.
template <int CH>
__device__ __forceinline__ void conv_reduce_rows(float (&v)[16], int lane, float* dst, int ld) {
  const int b5 = lane >> 5, b4 = lane >> 4 & 1, b3 = lane >> 3 & 1, b2 = lane >> 2 & 1;
#pragma unroll
  for (int t = 0; t < 8; ++t) v[t] = CH == 4 ? (b5 ? v[t + 8] : v[t]) : fold_halves32(v[t], v[t + 8]);
#pragma unroll
  for (int t = 0; t < 4; ++t) v[t] = fold_halves16(v[t], v[t + 4]);
  float* d = dst + b5 * ld + 4 * b4;
  if constexpr (CH == 16) {
#pragma unroll
    for (int t = 0; t < 4; ++t) d[t] = v[t];
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] += row_rotate<8>(v[t]);
    if constexpr (CH == 4) {
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] += row_rotate<4>(v[t]);
    }
    const float v0 = b3 ? v[2] : v[0], v1 = b3 ? v[3] : v[1];
    d += 2 * b3;
    if constexpr (CH == 8) { d[0] = v0; d[1] = v1; }
    else d[b2] = b2 ? v1 : v0;
  }
}

// Epilogue of one band: the 32 rows x W columns of fp32 values at Cw.  row0, col0: output row and column of the band; column(lc): the
// output column of slab column lc, relative to col0 (and to stat).  stat: where the band's sums go, the sums of squares ld later.
template <int W> struct ConvBand {      // lanes by chunk of eight channels and row; rows per pass over the band and passes
  static constexpr int CH = W / 8, RPI = 64 / CH, NIT = 32 / RPI;
};
// The band's residual.  A wave requests that of both its bands before it begins with the first: one after the other, each waited for memory:
// 10.4 -> 8.7 us an epilogue of a 512x128 tile (5.4 without a residual), 9.6 -> 8.6 of a 256x256 one (5.2).
template <int W, class Column>
__device__ __forceinline__ void conv_band_request(const ConvParams& p, int row0, int col0, int lane, bf16x8 (&o)[ConvBand<W>::NIT], Column column) {
  using B = ConvBand<W>;
  const EpiParams<bf16>& e = p.epi;
  const int n = min(col0 + column((lane % B::CH) * 8), e.N - 8), r = row0 + lane / B::CH;
#pragma unroll
  for (int it = 0; it < B::NIT; ++it) o[it] = *reinterpret_cast<const bf16x8*>((const bf16*)e.residual + (size_t)min(r + it * B::RPI, e.M - 1) * e.ld_res + n);
}
template <int W, bool RES, class Column>
__device__ __forceinline__ void conv_band_epilogue(const ConvParams& p, const float* Cw, int c_ld, int row0, int col0, int lane, float* stat, int ld,
                                                   bf16x8 (&o)[ConvBand<W>::NIT], Column column) {
  constexpr int CH = ConvBand<W>::CH, RPI = ConvBand<W>::RPI, NIT = ConvBand<W>::NIT;
  static_assert(RPI == 4 || RPI == 8 || RPI == 16, "band shape");
  const EpiParams<bf16>& e = p.epi;
  const int lc = (lane % CH) * 8, lr = lane / CH, nt = column(lc), n = col0 + nt;
  float bias[8];
  pp_bias(e.bias, min(n, e.N - 8), bias);
  bf16* out = e.out + (size_t)(row0 + lr) * e.ldo + n;
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    float v[8];
    pp_slab_row(&Cw[(it * RPI + lr) * c_ld + lc], v);
#pragma unroll
    for (int t = 0; t < 8; ++t) o[it][t] = (bf16)(RES ? (v[t] + bias[t]) + (float)o[it][t] : v[t] + bias[t]);
    if (row0 + it * RPI + lr < e.M && n < e.N) *reinterpret_cast<bf16x8*>(out + (size_t)(it * RPI) * e.ldo) = o[it];
  }
  if (!p.gn_partial) return;      // otherwise every row exists
  // sums over the rows with equal r % 8: r and r + 8 in one instruction, onto them r + 16 and r + 24; then pairwise over the bits of r % 8
  constexpr int PAR = RPI == 4 ? 2 : 1;
  float v[PAR][16];
#pragma unroll
  for (int t = 0; t < 16; ++t)
#pragma unroll
    for (int a = 0; a < PAR; ++a) v[a][t] = 0.f;
  const bf16x2 one = {(bf16)1.f, (bf16)1.f};
#pragma unroll
  for (int a = 0; a < PAR; ++a)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int i0 = RPI == 4 ? 4 * half + a : (RPI == 8 ? 2 * half : half), i1 = RPI == 4 ? i0 + 2 : i0 + 1;
      u32x4 x = __builtin_bit_cast(u32x4, o[i0]), y = x;
      if constexpr (RPI == 16) {      // rows lr and lr + 8 of this pass lie in the two halves of the wave
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const auto r = __builtin_amdgcn_permlane32_swap(x[j], x[j], false, false);
          const uint32_t lo = r[0], hi = r[1];
          x[j] = lo; y[j] = hi;
        }
      } else {
        y = __builtin_bit_cast(u32x4, o[i1 < NIT ? i1 : 0]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bf16x2 c0 = __builtin_bit_cast(bf16x2, __builtin_amdgcn_perm(y[j], x[j], 0x05040100u)), c1 = __builtin_bit_cast(bf16x2, __builtin_amdgcn_perm(y[j], x[j], 0x07060302u));
        v[a][2 * j] = __builtin_amdgcn_fdot2_f32_bf16(c0, one, v[a][2 * j], false);
        v[a][2 * j + 1] = __builtin_amdgcn_fdot2_f32_bf16(c1, one, v[a][2 * j + 1], false);
        v[a][8 + 2 * j] = __builtin_amdgcn_fdot2_f32_bf16(c0, c0, v[a][8 + 2 * j], false);
        v[a][9 + 2 * j] = __builtin_amdgcn_fdot2_f32_bf16(c1, c1, v[a][9 + 2 * j], false);
      }
    }
  if constexpr (PAR == 2) {
#pragma unroll
    for (int t = 0; t < 16; ++t) v[0][t] += v[1][t];
  }
  conv_reduce_rows<CH>(v[0], lane, stat + nt, ld);
}
// The tile's statistics: bands of a statistics block added in ascending order.
template <int BM, int BN>
__device__ __forceinline__ void conv_store_stats(const ConvParams& p, const float* stat, int tile_m, int n0, int m0, int tid, int threads) {
  const int bands = p.gn_block / 32, blocks = BM / p.gn_block;
  for (int i = tid; i < blocks * 2 * BN; i += threads) {
    const int blk = i / (2 * BN), which = i / BN % 2, c = i % BN;
    float sum = 0.f;
    for (int band = 0; band < bands; ++band) sum += stat[((size_t)(blk * bands + band) * 2 + which) * BN + c];
    if (n0 + c < p.epi.N && m0 + blk * p.gn_block < p.epi.M) p.gn_partial[((size_t)(tile_m * blocks + blk) * p.epi.N + n0 + c) * 2 + which] = sum;
  }
}

template <class T, bool RES>
__global__ void __launch_bounds__(512, 2) conv3x3_pp_kernel(const ConvParams p, uint32_t x_bytes, uint32_t w_bytes) {
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;          // an offset past any buffer this kernel accepts: the copy delivers zeros
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::WGN, wn = wave % T::WGN;
  int tile_m, tile_n;
  tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tile_m, tile_n);
  const int m0 = tile_m * T::BM, n0 = tile_n * T::BN, nk = p.K / T::BK;

  // per A piece of this wave: byte offset of the output pixel's own input pixel (tap centre) plus this lane's
  // chunk, and the 9-bit set of taps that fall inside the image for that pixel (empty for rows past M)
  int a_base[2][T::LA];
  unsigned a_taps[2][(T::LA + 1) / 2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < T::LA; ++j) {
      unsigned m;
      conv_pixel(p, m0 + h * (T::BM / 2), pp_piece_row(wave * T::LA + j, lane), lane, a_base[h][j], m);
      a_taps[h][j / 2] = j % 2 ? a_taps[h][j / 2] | m << 16 : m;
    }
  auto piece_b = [&](int h, int j) { return min(wave * (h ? T::LB1 : T::LB0) + j, (h ? T::B1_BYTES : T::B0_BYTES) / 1024 - 1); };
  auto offset_b = [&](int h, int j) {
    const int r = pp_piece_row(piece_b(h, j), lane), c = pp_piece_chunk(r, lane);
    return 2u * ((uint32_t)min(n0 + h * T::BN0 + r, p.N - 1) * (uint32_t)p.K + (uint32_t)c * 8u);
  };
  uint32_t vb0[T::LB0], vb1[T::LB1];
#pragma unroll
  for (int j = 0; j < T::LB0; ++j) vb0[j] = offset_b(0, j);
#pragma unroll
  for (int j = 0; j < T::LB1; ++j) vb1[j] = offset_b(1, j);
  // per row half, the k-tile whose copies come next (each half is copied tile by tile in order): its tap and the bytes of its first channel, and
  // the lanes' source offsets for that tap, which are formed once per tap.  No pixel has a tenth tap, so that what is copied past the last k-tile reads
  // nothing.  (Tap and channel counted apart, with a check against the last k-tile a copy: the class took 8.30 ms on 8 samples of 512x512, now 8.03.)
  const int tap_bytes = 2 * p.Cin;
  int it_tap[2] = {-1, -1}, it_off[2] = {tap_bytes, tap_bytes};
  uint32_t va[2][T::LA];
  const rsrc_t rx = make_rsrc(p.x, x_bytes);
  typename T::acc_t acc[2][T::TM][T::TN];
  float csum[2][T::TM];
  pp_main_loop<T, false, false, false, T::BM == 256>(acc, smem_raw, nk, wm, wn, wave >= 4, lane,
      [&](auto hc, int, unsigned char* dst) {
        constexpr int h = decltype(hc)::value;
        if (it_off[h] == tap_bytes) {
          it_off[h] = 0;
          const int tap = ++it_tap[h], u = (tap * 11) >> 5, v = tap - 3 * u;          // tap / 3, tap % 3
          const int off = 2 * ((u - 1) * p.W + (v - 1)) * p.Cin;
#pragma unroll
          for (int j = 0; j < T::LA; ++j) va[h][j] = (a_taps[h][j / 2] >> (tap + 16 * (j % 2))) & 1u ? (uint32_t)(a_base[h][j] + off) : OUTSIDE;
        }
#pragma unroll
        for (int j = 0; j < T::LA; ++j) async_copy_16B_buf(rx, va[h][j], (uint32_t)it_off[h], dst + (wave * T::LA + j) * 1024);
        it_off[h] += 2 * T::BK;
      },
      [&](auto hc, int t, unsigned char* dst) {
        constexpr int h = decltype(hc)::value;
        const rsrc_t r = make_rsrc(p.w, t < nk ? w_bytes : 0u);
        const uint32_t off = (uint32_t)t * (2u * T::BK);
#pragma unroll
        for (int j = 0; j < (h ? T::LB1 : T::LB0); ++j) async_copy_16B_buf(r, h ? vb1[h ? j : 0] : vb0[h ? 0 : j], off, dst + piece_b(h, j) * 1024);
      }, false, csum);

  static_assert(T::SM == 32 && T::WGM * 2 * 32 == T::BM, "epilogue shape");
  float* Cw = reinterpret_cast<float*>(smem_raw) + wave * 32 * T::C_LD;
  float* stat = reinterpret_cast<float*>(smem_raw + T::EPI_BYTES);      // [band][sum | sum of squares][BN], past the slabs
  auto column = [&](int lc) { return lc < T::SN0 ? wn * T::SN0 + lc : T::BN0 + wn * T::SN1 + lc - T::SN0; };
  bf16x8 o[2][ConvBand<T::W>::NIT];
  if constexpr (RES) {
#pragma unroll
    for (int ha = 0; ha < 2; ++ha) conv_band_request<T::W>(p, m0 + ha * (T::BM / 2) + wm * 32, n0, lane, o[ha], column);
  }
#pragma unroll
  for (int ha = 0; ha < 2; ++ha) {
#pragma unroll
    for (int j = 0; j < T::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) Cw[acc_row(r, lane >> 5) * T::C_LD + j * 32 + (lane & 31)] = acc[ha][0][j][r];
    asm volatile("" ::: "memory");
    conv_band_epilogue<T::W, RES>(p, Cw, T::C_LD, m0 + ha * (T::BM / 2) + wm * 32, n0, lane, stat + (size_t)(ha * T::WGM + wm) * 2 * T::BN, T::BN, o[ha], column);
    asm volatile("" ::: "memory");
  }
  if (!p.gn_partial) return;
  __syncthreads();
  conv_store_stats<T::BM, T::BN>(p, stat, tile_m, n0, m0, tid, 512);
}

// ------------------------------------------------------------------ small tiles
// 64x64 and 128x128 tiles for layers with few output pixels (a partial batch of one sample in the deep layers: 32 tiles of 256x128 for 256
// CUs, each walking all 72 k-tiles of a 4608-deep contraction, 61 us).  The ring of dp_gemm_ring.h.  The order of the additions is that of the large tiles, so
// the tile shape, which depends on the number of samples, changes no bit: same k order, same 32-row statistics bands.
// Measured (512 -> 512 channels): 48 x 41 pixels 61 -> 20 us (64x64; 24 with the fragments read right before their use), 96 x 82 65 -> 43 us (128x128); 512 -> 8 head at 48 x 41 71 -> 20 us.
// With ring_main_loop's constant stages and the tap looked at when it changes 21.5 -> 17.9 and 36.9 -> 32.3 us.  (A fourth buffer of 128x128 changes nothing.)
template <int BM_, int BN_, int WGM_, int WGN_, int STAGES_>
struct ConvSmallTile {
  static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, STAGES = STAGES_, NW = WGM * WGN, WM = BM / WGM, WN = BN / WGN, TN = WN / 32;
  static constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, STAGE = A_BYTES + B_BYTES, LA = A_BYTES / 1024 / NW, LB = B_BYTES / 1024 / NW;
  static constexpr int C_LD = WN + 8;
  static constexpr size_t EPI_BYTES = (size_t)NW * 32 * C_LD * 4, STAT_BYTES = (size_t)BM / 32 * 2 * BN * 4;
  static constexpr size_t BYTES = (size_t)STAGES * STAGE > EPI_BYTES + STAT_BYTES ? (size_t)STAGES * STAGE : EPI_BYTES + STAT_BYTES;
  static_assert(WM == 32 && WN % 32 == 0 && A_BYTES % (1024 * NW) == 0 && B_BYTES % (1024 * NW) == 0, "tile shape");
};

template <class T, bool RES>
__global__ void __launch_bounds__(T::NW * 64) conv3x3_small_kernel(const ConvParams p, uint32_t x_bytes, uint32_t w_bytes) {
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;
  constexpr int LA = T::LA, LB = T::LB;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, l32 = lane & 31;
  const int wm = wave / T::WGN, wn = wave % T::WGN;
  int tile_m, tile_n;
  tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, p.group_m, tile_m, tile_n);
  const int m0 = tile_m * T::BM, n0 = tile_n * T::BN, nk = p.K / 64;
  int a_base[LA];
  unsigned a_taps[LA];
#pragma unroll
  for (int j = 0; j < LA; ++j) conv_pixel(p, m0, pp_piece_row(wave * LA + j, lane), lane, a_base[j], a_taps[j]);
  uint32_t va[LA], vb[LB];
#pragma unroll
  for (int j = 0; j < LB; ++j) {
    const int r = pp_piece_row(wave * LB + j, lane), c = pp_piece_chunk(r, lane);
    vb[j] = 2u * ((uint32_t)min(n0 + r, p.N - 1) * (uint32_t)p.K + (uint32_t)c * 8u);
  }
  const int tap_bytes = 2 * p.Cin;
  int it_tap = -1, it_off = tap_bytes;      // (no pixel has a tenth tap: past the last k-tile nothing is read)
  const rsrc_t rx = make_rsrc(p.x, x_bytes);
  f32x16 acc[T::TN];
#pragma unroll
  for (int j = 0; j < T::TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  ring_main_loop<T::STAGES, T::STAGE, T::A_BYTES, LA + LB>(acc, smem_raw, nk, wm * 32, wn * T::WN, lane,
      [&](int t, unsigned char* st) {
        if (it_off == tap_bytes) {
          it_off = 0; ++it_tap;
          const int u = (it_tap * 11) >> 5, v = it_tap - 3 * u, off = 2 * ((u - 1) * p.W + (v - 1)) * p.Cin;
#pragma unroll
          for (int j = 0; j < LA; ++j) va[j] = (a_taps[j] >> it_tap) & 1u ? (uint32_t)(a_base[j] + off) : OUTSIDE;
        }
        const rsrc_t rw = make_rsrc(p.w, t < nk ? w_bytes : 0u);
#pragma unroll
        for (int j = 0; j < LA; ++j) async_copy_16B_buf(rx, va[j], (uint32_t)it_off, st + (wave * LA + j) * 1024);
#pragma unroll
        for (int j = 0; j < LB; ++j) async_copy_16B_buf(rw, vb[j], (uint32_t)t * 128u, st + T::A_BYTES + (wave * LB + j) * 1024);
        it_off += 128;
      }, []() {});
  __syncthreads();
  float* Cw = reinterpret_cast<float*>(smem_raw) + wave * 32 * T::C_LD;
  float* stat = reinterpret_cast<float*>(smem_raw + T::EPI_BYTES);      // [band][sum | sum of squares][BN], past the slabs
  auto column = [](int lc) { return lc; };
  bf16x8 o[ConvBand<T::WN>::NIT];
  if constexpr (RES) conv_band_request<T::WN>(p, m0 + wm * 32, n0 + wn * T::WN, lane, o, column);
#pragma unroll
  for (int j = 0; j < T::TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) Cw[acc_row(r, g) * T::C_LD + j * 32 + l32] = acc[j][r];
  asm volatile("" ::: "memory");
  conv_band_epilogue<T::WN, RES>(p, Cw, T::C_LD, m0 + wm * 32, n0 + wn * T::WN, lane, stat + (size_t)wm * 2 * T::BN + wn * T::WN, T::BN, o, column);
  if (!p.gn_partial) return;
  __syncthreads();
  conv_store_stats<T::BM, T::BN>(p, stat, tile_m, n0, m0, tid, T::NW * 64);
}

// ------------------------------------------------------------------ eight input channels
// The encoder's first layer (an image padded to eight channels): 9 taps x 8 channels, bound by writing the output.  A tap's 8 channels are the
// 16 bytes a lane contributes to an MFMA step of 16, so a pixel's neighbourhood goes from memory straight into the operand: five
// steps of two taps; the tenth slot holds a one against the bias.  The weights are the row operand, dealt to its
// rows so that a lane's 16 accumulators are 16 consecutive channels of one pixel: two 16-byte LDS writes turn them into whole
// lines of the output.  A workgroup walks over tiles of 256 pixels, 64 per wave; GroupNorm sums are kept in lanes over a wave's
// 64 rows and reduced with lane swaps, each step halving the values a lane holds.
// 8 samples of 512 x 512 -> 128 channels (537 MB out): 288 us + 73 us for the sums in a pass of their own through the staged kernel; now 138 us (4.1 TB/s), sums included.
template <int TN>
struct ConvIn8 {
  static constexpr int BN = 32 * TN, KP = 80;
  static constexpr int W_BYTES = BN * KP * 2, SLAB_BYTES = 4 * 32 * 64 * 2, STAT_BYTES = 4 * 2 * BN * 4, BYTES = W_BYTES + SLAB_BYTES + STAT_BYTES;
};
template <int TN>
__global__ void __launch_bounds__(256, 4) conv3x3_in8_kernel(const ConvParams p, uint32_t x_bytes) {
  using T = ConvIn8<TN>;
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, l32 = lane & 31;
  bf16* Ws = reinterpret_cast<bf16*>(smem_raw);
  bf16* slab = reinterpret_cast<bf16*>(smem_raw + T::W_BYTES) + wave * 32 * 64;
  float* stat = reinterpret_cast<float*>(smem_raw + T::W_BYTES + T::SLAB_BYTES);
  for (int i = tid; i < T::BN * 10; i += 256) {
    const int r = i / 10, tap = i - 10 * r, n = (r & ~31) + 16 * (r >> 2 & 1) + 4 * (r >> 3 & 3) + (r & 3);      // row r of the operand: channel n
    bf16x8 v = zero8();
    if (n < p.N) {
      if (tap < 9) v = *reinterpret_cast<const bf16x8*>(p.w + (size_t)n * 72 + tap * 8);
      else if (p.epi.bias) v[0] = p.epi.bias[n];
    }
    *reinterpret_cast<bf16x8*>(Ws + r * T::KP + tap * 8) = v;
  }
  __syncthreads();
  const rsrc_t rx = make_rsrc(p.x, x_bytes);
  bf16x8 px[5];
  auto fetch = [&](int row0) {
    const int gm = row0 + l32, q = min(gm, p.M - 1), hw = p.Ho * p.Wo;
    const int b = fast_div(q, p.by_px), rem = q - b * hw, ho = fast_div(rem, p.by_wo), wo = rem - ho * p.Wo;
    const int hc = ho * p.stride, wc = wo * p.stride, base = (b * p.H + hc) * p.W + wc;
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      const int u = (g ? (2 * s + 1) / 3 : 2 * s / 3) - 1, v = (g ? (2 * s + 1) % 3 : 2 * s % 3) - 1;
      const bool in = gm < p.M && (unsigned)(hc + u) < (unsigned)p.H && (unsigned)(wc + v) < (unsigned)p.W;
      px[s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rx, in ? (uint32_t)(base + u * p.W + v) * 16u : OUTSIDE, 0, 0));
    }
    bf16x8 one = zero8();
    one[0] = (bf16)1.0f;
    px[4] = g ? one : px[4];
  };
  const int lc = lane & 7, lr = lane >> 3;
  int tile = blockIdx.x;
  fetch(tile * 256 + wave * 64);
  for (; tile < p.tiles_m; tile += gridDim.x) {
    float sums[TN / 2][2];
#pragma unroll
    for (int h = 0; h < TN / 2; ++h) sums[h][0] = sums[h][1] = 0.f;
#pragma unroll
    for (int band = 0; band < 2; ++band) {
      const int row0 = tile * 256 + wave * 64 + band * 32;
#pragma unroll
      for (int half = 0; half < TN / 2; ++half) {
        f32x16 acc[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
#pragma unroll
          for (int s = 0; s < 5; ++s)
            acc[j] = mfma32(*reinterpret_cast<const bf16x8*>(Ws + ((2 * half + j) * 32 + l32) * T::KP + s * 16 + 8 * g), px[s], acc[j]);
        }
        if (half == TN / 2 - 1) {
          const int next = band == 0 ? row0 + 32 : row0 - 32 + (int)gridDim.x * 256;
          if (next < p.M) fetch(next);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          bf16x8 o;
#pragma unroll
          for (int t = 0; t < 8; ++t) o[t] = (bf16)acc[c >> 1][8 * (c & 1) + t];
          const int chunk = 4 * (c >> 1) + 2 * g + (c & 1);
          *reinterpret_cast<bf16x8*>(slab + l32 * 64 + (chunk ^ (l32 & 7)) * 8) = o;
        }
        asm volatile("" ::: "memory");      // lanes of one wave exchange through the slab: LDS serves a wave in order
        const int n = 64 * half + lc * 8;
        float v[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) v[t] = 0.f;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int row = it * 8 + lr;
          const bf16x8 o = *reinterpret_cast<const bf16x8*>(slab + row * 64 + (lc ^ (row & 7)) * 8);
          if (row0 + row < p.M && n < p.N) *reinterpret_cast<bf16x8*>(p.epi.out + (size_t)(row0 + row) * p.epi.ldo + n) = o;
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            const float f = (float)o[t];
            v[t] += f; v[8 + t] = fmaf(f, f, v[8 + t]);
          }
        }
        asm volatile("" ::: "memory");
        if (p.gn_partial) {
#pragma unroll
          for (int t = 0; t < 8; ++t) v[t] = fold_halves32(v[t], v[t + 8]);
#pragma unroll
          for (int t = 0; t < 4; ++t) { v[t] = fold_halves16(v[t], v[t + 4]); v[t] += row_rotate<8>(v[t]); }
          sums[half][0] += lane & 8 ? v[2] : v[0];
          sums[half][1] += lane & 8 ? v[3] : v[1];
        }
      }
    }
    if (p.gn_partial) {      // lanes below 32 hold sums, the others sums of squares
#pragma unroll
      for (int half = 0; half < TN / 2; ++half) {
        float* d = stat + (wave * 2 + g) * T::BN + 64 * half + lc * 8 + 4 * (lane >> 4 & 1) + 2 * (lane >> 3 & 1);
        d[0] = sums[half][0]; d[1] = sums[half][1];
      }
      __syncthreads();
      const int parts = p.gn_block / 64, blocks = 4 / parts;
      for (int i = tid; i < blocks * 2 * T::BN; i += 256) {
        const int blk = i / (2 * T::BN), which = i / T::BN % 2, c = i % T::BN;
        float sum = 0.f;
        for (int q = 0; q < parts; ++q) sum += stat[((blk * parts + q) * 2 + which) * T::BN + c];
        if (c < p.N && tile * 256 + blk * p.gn_block < p.M) p.gn_partial[((size_t)(tile * blocks + blk) * p.N + c) * 2 + which] = sum;
      }
      __syncthreads();
    }
  }
}

template <class Kern>
static int launch_conv_kernel(Kern kern, std::atomic<bool>& attr_set, long n, int threads, size_t lds, const ConvParams& p, size_t x_bytes, size_t w_bytes, hipStream_t s) {
  if (!attr_set.load(std::memory_order_acquire)) {   // setting it twice is harmless; the flag only saves the call
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return set_error(DP_EHIP, "hipFuncSetAttribute(conv) failed");
    attr_set.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)n), dim3(threads), lds, s, p, (uint32_t)x_bytes, (uint32_t)w_bytes);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "conv launch failed");
}
template <class T>
static int launch_conv_pp(ConvParams& p, size_t x_bytes, size_t w_bytes, hipStream_t s) {
  constexpr size_t LDS = T::EPI_BYTES + (size_t)T::BM / 32 * 2 * T::BN * 4 > T::BYTES ? T::EPI_BYTES + (size_t)T::BM / 32 * 2 * T::BN * 4 : T::BYTES;
  static_assert(LDS <= 160 * 1024, "tile shape");
  p.tiles_m = (p.M + T::BM - 1) / T::BM; p.tiles_n = (p.N + T::BN - 1) / T::BN;
  // whole tile-rows per XCD: the tiles that share a band of input pixels run on one L2
  const long n = (long)p.tiles_m * p.tiles_n, ppx = (n + 7) / 8;
  p.group_m = (int)std::max<long>(1, std::min<long>((ppx + p.tiles_n / 2) / p.tiles_n, p.tiles_m));
  static std::atomic<bool> set_res{false}, set_plain{false};
  return p.epi.residual ? launch_conv_kernel(conv3x3_pp_kernel<T, true>, set_res, n, 512, LDS, p, x_bytes, w_bytes, s)
                        : launch_conv_kernel(conv3x3_pp_kernel<T, false>, set_plain, n, 512, LDS, p, x_bytes, w_bytes, s);
}

template <int BM, int BN, int WGM, int WGN>
static int launch_conv_cfg(ConvParams& p, hipStream_t s) {
  using S = ConvSmem<BM, BN, WGM, WGN>;
  p.tiles_m = (p.M + BM - 1) / BM; p.tiles_n = (p.N + BN - 1) / BN;
  // whole tile-rows per XCD: the tiles that share a band of input pixels run on one L2
  const long n = (long)p.tiles_m * p.tiles_n, ppx = (n + 7) / 8;
  p.group_m = (int)std::max<long>(1, std::min<long>((ppx + p.tiles_n / 2) / p.tiles_n, p.tiles_m));
  auto kern = conv3x3_bf16_kernel<BM, BN, WGM, WGN>;
  if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::BYTES) != hipSuccess)
    return set_error(DP_EHIP, "hipFuncSetAttribute(conv) failed");
  hipLaunchKernelGGL(kern, dim3((unsigned)n), dim3(WGM * WGN * 64), S::BYTES, s, p);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "conv launch failed");
}

template <class T>
static int launch_conv_small(ConvParams& p, size_t x_bytes, size_t w_bytes, hipStream_t s) {
  p.tiles_m = (p.M + T::BM - 1) / T::BM; p.tiles_n = (p.N + T::BN - 1) / T::BN;
  const long n = (long)p.tiles_m * p.tiles_n, ppx = (n + 7) / 8;
  p.group_m = (int)std::max<long>(1, std::min<long>((ppx + p.tiles_n / 2) / p.tiles_n, p.tiles_m));
  static std::atomic<bool> set_res{false}, set_plain{false};
  return p.epi.residual ? launch_conv_kernel(conv3x3_small_kernel<T, true>, set_res, n, T::NW * 64, T::BYTES, p, x_bytes, w_bytes, s)
                        : launch_conv_kernel(conv3x3_small_kernel<T, false>, set_plain, n, T::NW * 64, T::BYTES, p, x_bytes, w_bytes, s);
}

template <int TN>
static int launch_conv_in8(ConvParams& p, size_t x_bytes, hipStream_t s) {
  p.tiles_m = (p.M + 255) / 256; p.tiles_n = 1; p.group_m = 1;
  const int rounds = (p.tiles_m + 1023) / 1024;      // four workgroups per CU, each with an equal share of the tiles
  hipLaunchKernelGGL(conv3x3_in8_kernel<TN>, dim3((p.tiles_m + rounds - 1) / rounds), dim3(256), ConvIn8<TN>::BYTES, s, p, (uint32_t)x_bytes);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "conv launch failed");
}

// Pixels per statistics block for an output of `px` pixels per sample: blocks of 256, of 64 where the small tiles may run (their 64 rows).
int conv_stat_block(int px) { return px < 16384 ? 64 : 256; }

int launch_conv3x3(const ConvArgs& a, hipStream_t s) {
  if (a.dtype != BF16) return set_error(DP_EUNSUPPORTED, "conv3x3: bf16 storage only");
  if (a.B <= 0 || a.H <= 0 || a.W <= 0 || a.Cin <= 0 || a.Cout <= 0) return set_error(DP_EINVAL, "conv3x3: non-positive size");
  if (a.stride != 1 && a.stride != 2) return set_error(DP_EUNSUPPORTED, "conv3x3: stride must be 1 or 2");
  if (a.Cin % 8 || a.Cout % 8) return set_error(DP_EUNSUPPORTED, "conv3x3: channel counts must be multiples of 8");
  if (!a.x || !a.w || !a.y) return set_error(DP_EINVAL, "conv3x3: null operand");
  const void* ps[] = {a.x, a.w, a.y, a.bias, a.residual};
  for (const void* q : ps) if ((uintptr_t)q % 16) return set_error(DP_EALIGN, "conv3x3: operands must be 16-byte aligned");
  const int Ho = (a.H - 1) / a.stride + 1, Wo = (a.W - 1) / a.stride + 1;
  const long M = (long)a.B * Ho * Wo;
  if (M >= (1L << 31) - 512 || (long)9 * a.Cin >= (1L << 24)) return set_error(DP_EUNSUPPORTED, "conv3x3: too many output pixels or input channels");
  ConvParams p;
  p.x = (const bf16*)a.x; p.w = (const bf16*)a.w;
  p.H = a.H; p.W = a.W; p.Cin = a.Cin; p.Ho = Ho; p.Wo = Wo; p.stride = a.stride;
  p.M = (int)M; p.N = a.Cout; p.K = 9 * a.Cin;
  p.by_px = make_fast_div(Ho * Wo); p.by_wo = make_fast_div(Wo);
  p.taps_uniform = a.Cin % 64 == 0;
  p.gn_partial = nullptr; p.gn_block = 256;
  if (a.gn_applied) *a.gn_applied = 0;
  if (a.gn_partial && !a.gn_applied) return set_error(DP_EINVAL, "conv3x3: gn_partial comes with gn_applied");
  EpiParams<bf16>& e = p.epi;
  e.M = p.M; e.N = p.N; e.out = (bf16*)a.y; e.ldo = a.Cout;
  e.out32 = nullptr; e.ldo32 = 0; e.accumulate = 0; e.partial = nullptr;
  e.bias = (const bf16*)a.bias; e.pre_out = nullptr; e.ld_pre = 0; e.act = 0;
  e.dact_pre = nullptr; e.ld_dact = 0; e.dact_kind = 0; e.gate = nullptr; e.gate_ld = 0; e.rows_per_batch = 1;
  e.residual = a.residual; e.ld_res = a.Cout; e.residual_f32 = 0; e.out_fused_f32 = 0;
  e.geglu = 0; e.geglu_inner = 0; e.geglu_u = nullptr; e.ld_geglu = 0; e.out_scale = 1.0f;
  const double by = 2.0 * ((double)a.B * a.H * a.W * a.Cin + (double)p.N * p.K + (double)M * a.Cout * (a.residual ? 2.0 : 1.0));
  KScope ks(KK_CONV, 2.0 * (double)M * p.N * p.K, by, s, p.M, p.N, p.K);
  // the direct-to-LDS kernel: k-tiles inside one tap, 32-bit byte offsets with room for the "outside" marker
  const size_t x_bytes = 2 * (size_t)a.B * a.H * a.W * a.Cin, w_bytes = 2 * (size_t)p.N * p.K;
  // (whether this kernel is taken depends on one sample's pixel count, not on the number of samples)
  if (a.Cin == 8 && a.Cout <= 128 && !a.residual && x_bytes < (1ull << 31) && !a.force_staged) {
    p.gn_block = conv_stat_block(Ho * Wo);
    if (a.gn_partial && (Ho * Wo) % p.gn_block == 0 && ((uintptr_t)a.gn_partial % 16) == 0) { p.gn_partial = a.gn_partial; *a.gn_applied = 1; }
    return a.Cout <= 64 ? launch_conv_in8<2>(p, x_bytes, s) : launch_conv_in8<4>(p, x_bytes, s);
  }
  if (a.Cin % 64 == 0 && x_bytes < (1ull << 31) && w_bytes < (1ull << 31) && !a.force_staged) {
    p.gn_block = conv_stat_block(Ho * Wo);
    if (a.gn_partial && (Ho * Wo) % p.gn_block == 0 && ((uintptr_t)a.gn_partial % 16) == 0) { p.gn_partial = a.gn_partial; *a.gn_applied = 1; }
    // The tile with the least estimated time, rounds over the 256 CUs x (fixed part + k-tiles x time of one).  This choice may
    // depend on the number of samples: the shapes produce the same bits, statistics included.  The times of a k-tile are measured ones
    // (us at 72 k-tiles: 256x256 125, 256x128 77, 128x128 41 with one workgroup per CU each; 64x64 17 with one, 29 with two).
    const bool small = p.gn_block == 64 || !p.gn_partial;
    const struct { int bm, bn, at_once; float fixed, per_kt; } tiles[] = {{256, 256, 256, 6.0f, 1.66f}, {256, 128, 256, 5.0f, 1.00f}, {512, 64, 256, 6.0f, 1.90f},
                                                                          {512, 128, 256, 6.0f, 2.10f}, {64, 64, 512, 5.0f, 0.33f}, {128, 128, 256, 5.0f, 0.50f}};
    int best = 0;
    float best_us = 0.f;
    for (int i = 0; i < (small ? 6 : 4); ++i) {
      const long n = ((M + tiles[i].bm - 1) / tiles[i].bm) * ((a.Cout + tiles[i].bn - 1) / tiles[i].bn);
      const float per_kt = i == 4 && n <= 256 ? 0.17f : tiles[i].per_kt;        // two of the smallest tiles on a CU slow each other down
      const float us = (float)((n + tiles[i].at_once - 1) / tiles[i].at_once) * (tiles[i].fixed + (float)(p.K / 64) * per_kt);
      if (i == 0 || us < best_us) { best = i; best_us = us; }
    }
    switch (best) {
      case 0: return launch_conv_pp<PpTile<256, 128, 128, 4, 2>>(p, x_bytes, w_bytes, s);
      case 1: return launch_conv_pp<PpTile<256, 64, 64, 4, 2>>(p, x_bytes, w_bytes, s);
      case 2: return launch_conv_pp<PpTile<512, 32, 32, 8, 1>>(p, x_bytes, w_bytes, s);
      case 3: return launch_conv_pp<PpTile<512, 64, 64, 8, 1>>(p, x_bytes, w_bytes, s);
      case 4: return launch_conv_small<ConvSmallTile<64, 64, 2, 2, 4>>(p, x_bytes, w_bytes, s);
      default: return launch_conv_small<ConvSmallTile<128, 128, 4, 2, 3>>(p, x_bytes, w_bytes, s);
    }
  }
  if (a.Cout <= 64) return launch_conv_cfg<128, 64, 4, 1>(p, s);
  if ((long)Ho * Wo >= 16384) return launch_conv_cfg<256, 128, 4, 2>(p, s);
  return launch_conv_cfg<128, 128, 2, 2>(p, s);
}

}  // namespace dp
