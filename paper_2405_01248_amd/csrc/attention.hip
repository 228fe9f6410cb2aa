// Fused softmax attention, forward and backward, for self-attention (N keys),
// cross-attention to the text context (77 keys) and the text encoder's causal attention.
//
// bf16 path (MFMA 32x32x16, wave64).  A wave owns 32 queries (forward, dQ) or 32 keys
// (dK/dV) and keeps them in registers as the MFMA B operand; the other side streams
// through LDS in 64-row tiles.  Scores are produced transposed (S^T = K Q^T) so that a
// lane holds one query column: the softmax statistics are lane-local (online over the tiles; over
// all keys at once in the forward of few keys, which has them all in LDS), and the
// probability block, once rounded to bf16, already has the register layout of the B
// operand of the second product (O^T = V^T P^T).  The operand that needs its
// contraction index moved (V, and K/Q/dO in the backward) is read from its row-major
// LDS tile with the transposing LDS load.  The backward is split into a dQ kernel and
// a dK/dV kernel so that no floating-point atomics are needed (run-to-run identical).
// The streamed tiles are copied global -> LDS directly (`buffer_load ... lds`) into unpadded tiles whose
// 16-byte chunks are permuted per row, so that both ways of reading a tile stay free of bank conflicts.
//
// What bounds them (40 heads of 4096 tokens, width 64; counters): the power the card may draw.  Forward, dQ and dK/dV take 2.9, 3.6 and 5.0
// million cycles (summed over 8 XCDs) at 1.87, 1.80 and 1.82 GHz, matrix pipes busy 45, 55 and 53 % of them; before the waits for the tile copies,
// a quarter of the vector instructions and the bank conflicts of the row fragments were taken out it was 3.4, 4.3 and 6.1 million at up to 2.2 GHz:
// 212 -> 192, 280 -> 249, 351 -> 337 us.  What is left per element of the scores is one fma, one exponential, a product (backward) or a sum
// (forward) and half a conversion.
//
// fp32 path: one wave per query (or key) row, plain FMA; used by the small fp32
// configuration only.
#include "dp_device.h"
#include "dp_kernels.h"
#include "dp_errors.h"
#include "dp_ktime.h"
#include <math.h>
#include <algorithm>
#include <atomic>
#include <type_traits>

namespace dp {

struct AttnK {
  int B, H, Nq, Nk, dh;
  float scale_log2;   // scale * log2(e)
  float scale;
  const void* q; int ldq;
  const void* k; int ldk;
  const void* v; int ldv;
  void* o; int ldo;
  float* lse;
  const void* dout; int lddo;
  float* delta;
  void* dq; int lddq;
  void* dk; int lddk;
  void* dv; int lddv;
  int even;           // waves of a SIMD take turns (take_turns)
  int qsplits; float* dkv_partial;   // dK/dV kernel: query range split + fp32 partial outputs [2][qsplits][B * Nk][H * dh]
};

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// Layout of a streamed [64 x DHP] bf16 tile in LDS: 64 rows of DHP / 8 16-byte chunks, no padding; the chunk
// at position pos of a row is chunk pos ^ key(row).  A tile is read two ways -- by rows as an MFMA A operand
// (16 consecutive rows, one chunk each, per 256 bytes of LDS bandwidth) and through the transposing load (4
// consecutive rows x 64 bytes) -- and the key keeps both conflict-free:
//   DHP = 64 (128-byte rows, two to the 256 bytes of a bank line): key = row bits (1, 2, 3), a bijection of the 8 rows that
//     share a half of the line among 16 consecutive ones; its bit 2 is row bit 1, so the 4 rows of a transposing read lie in
//     4 different 64-byte bank groups;
//   DHP = 96 (192-byte rows): consecutive rows already start 192 bytes apart, i.e. in different 64-byte groups;
//     rows r and r + 4 share one, so key = (row >> 2) & 3 moves them apart inside the group.
template <int DHP> struct AttnTile;
template <> struct AttnTile<64> {
  static constexpr int PIECES = 2;     // 1 KB copy instructions per wave and tile (16 rows)
  static __device__ __forceinline__ int key(int row) { return ((row & 8) >> 3) | ((row & 4) >> 1) | ((row & 2) << 1); }
};
template <> struct AttnTile<96> {
  static constexpr int PIECES = 3;
  static __device__ __forceinline__ int key(int row) { return (row >> 2) & 3; }
};

// Global -> LDS copy of one tile (`buffer_load ... lds`: the wave's 64 x 16 bytes land contiguously in LDS).
// A wave owns rows 16 * wave .. + 15; each lane keeps the byte offset, inside the (batch, head) slice, of the
// chunk that belongs at its LDS position.  Chunks past d_head get an offset of 2^31, which stays outside the
// buffer descriptor's range whatever tile offset is added: they, like rows past the end of the slice, arrive
// as zeros without touching memory.
template <int DHP>
struct AttnTileCopy {
  using T = AttnTile<DHP>;
  uint32_t off[T::PIECES];
  __device__ __forceinline__ void init(int wave, int lane, int ld, int dh) {
#pragma unroll
    for (int j = 0; j < T::PIECES; ++j) {
      const int o = 1024 * j + 16 * lane;                     // byte inside the wave's 16-row block
      const int row = 16 * wave + o / (2 * DHP), pos = (o % (2 * DHP)) / 16;
      const int chunk = pos ^ T::key(row);
      off[j] = 8 * chunk < dh ? (uint32_t)(row * ld + 8 * chunk) * 2u : 0x80000000u;
    }
  }
  // rows row0 .. row0 + 63 of the slice behind r (the tile offset goes into the per-lane offset: only that
  // one is range-checked)
  __device__ __forceinline__ void issue(u32x4 r, int row0, int ld, bf16* stage, int wave) const {
#pragma unroll
    for (int j = 0; j < T::PIECES; ++j)
      async_copy_16B_raw(r, off[j] + (uint32_t)row0 * (uint32_t)ld * 2u, lds_address(stage) + 2u * (16 * wave * DHP + 512 * j));
  }
};

// Per-lane element offsets of the fragment reads, computed once.  A row fragment (rows 32 * t + l32, k-chunk
// c) is at row[c] + 32 * DHP * t.  A transposed fragment in the slot order of frag_from_mc_accorder (rows
// r0 .. r0 + 15 with r0 a multiple of 16, which leaves the keys alone; columns 32 * i .. + 31) is read as two
// halves at tr_lo[i] + DHP * r0 and tr_hi[i] + DHP * r0 (8 rows apart).
template <int DHP, int KC>
struct AttnFragOff {
  using T = AttnTile<DHP>;
  int row[KC], tr_lo[DHP / 32], tr_hi[DHP / 32];
  __device__ __forceinline__ void init(int lane) {
    const int g = lane >> 5, l32 = lane & 31;
#pragma unroll
    for (int c = 0; c < KC; ++c) row[c] = l32 * DHP + 8 * ((2 * c + g) ^ T::key(l32));
#pragma unroll
    for (int i = 0; i < DHP / 32; ++i) transposed(lane, i, tr_lo[i], tr_hi[i]);
  }
  static __device__ __forceinline__ void transposed(int lane, int i, int& lo, int& hi) {
    const int b = lane >> 4, j = lane & 15, r = 4 * (b >> 1) + (j >> 2), chunk = 4 * i + 2 * (b & 1) + ((j & 3) >> 1);
    lo = r * DHP + 8 * (chunk ^ T::key(r)) + 4 * (j & 1);
    hi = (r + 8) * DHP + 8 * (chunk ^ T::key(r + 8)) + 4 * (j & 1);
  }
  __device__ __forceinline__ bf16x8 row_frag(const bf16* tile, int t, int c) const {
    return *reinterpret_cast<const bf16x8*>(tile + row[c] + 32 * DHP * t);
  }
  __device__ __forceinline__ bf16x8 tr_frag(const bf16* tile, int r0, int i) const {
    const bf16x4 lo = lds_read_tr(tile + tr_lo[i] + DHP * r0);
    const bf16x4 hi = lds_read_tr(tile + tr_hi[i] + DHP * r0);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};
// byte extent of a (batch, head) slice of n rows with leading dimension ld (elements), d_head columns
__device__ __forceinline__ uint32_t attn_slice_bytes(int n, int ld, int dh) { return (uint32_t)(((size_t)(n - 1) * ld + dh) * 2); }

__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int off) {
  bf16x8 o;
#pragma unroll
  for (int u = 0; u < 8; ++u) o[u] = (bf16)v[off + u];
  return o;
}

// Among waves of one priority a SIMD serves the oldest first, so of the workgroups a CU holds one ends early and the last runs alone, at half the
// rate.  Where all workgroups of a launch are resident at once, a wave's priority falls by one every second tile and wraps, which keeps them
// together: 80 heads of 1024 tokens, 640 workgroups, forward 33.7 -> 31.3 us, dQ 45.2 -> 42.5, dK/dV 56.5 -> 52.7.  Where more wait to be
// started, the staggered ends are what lets them start: 40 heads of 4096 tokens lose 5 % with it; one workgroup per CU has nothing to share.
__device__ __forceinline__ void take_turns(int even, int i) {
  if (even) {
    const int turn = (i >> 1) & 3;
    if (turn == 0) __builtin_amdgcn_s_setprio(3);
    else if (turn == 1) __builtin_amdgcn_s_setprio(2);
    else if (turn == 2) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
  }
}

// tile(i, stage) for i = first .. last - 1, the stages of LDS in turn and known to the compiler: the fragment reads then need no address
// arithmetic and no registers beyond the offsets of AttnFragOff.
template <class F> __device__ __forceinline__ void two_stages(int first, int last, F tile) {
  for (int i = first; i < last; i += 2) {
    tile(i, std::integral_constant<int, 0>());
    if (i + 1 < last) tile(i + 1, std::integral_constant<int, 1>());
  }
}

// Maps a linear workgroup id to (tile along the sequence, batch * head).  Hardware deals
// consecutive ids round-robin to the 8 XCDs; with this map all tiles of one (batch, head) run
// on the same XCD, so its K/V (or Q/dO) stream is fetched into one L2 only.
__device__ __forceinline__ void attn_block_map(int id, int ntiles, int BH, int& tile, int& bh) {
  const int full = (BH / 8) * 8;
  if (id < full * ntiles) {
    const int grp = id / (8 * ntiles), r = id % (8 * ntiles);
    bh = grp * 8 + (r & 7);
    tile = r >> 3;
  } else {
    const int r = id - full * ntiles;
    bh = full + r / ntiles;
    tile = r % ntiles;
  }
}

// A query's row of the output and the logarithm of its sum; m: reference of its exponentials (log2 domain), lsum: their sum.
template <int DT>
__device__ __forceinline__ void attn_store_o(const AttnK& p, const f32x16 (&oacc)[DT], float lsum, float m, int b, int h, int qi, int g) {
  if (qi >= p.Nq) return;
  const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
  bf16* ob = (bf16*)p.o + ((size_t)b * p.Nq + qi) * p.ldo + h * p.dh;
#pragma unroll
  for (int i = 0; i < DT; ++i)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const int col = 32 * i + 8 * r4 + 4 * g;
      if (col < p.dh) {
        bf16x4 o;
#pragma unroll
        for (int u = 0; u < 4; ++u) o[u] = (bf16)(oacc[i][4 * r4 + u] * inv);
        *reinterpret_cast<bf16x4*>(ob + col) = o;
      }
    }
  if (p.lse && g == 0) p.lse[((size_t)b * p.H + h) * p.Nq + qi] = fmaf(m, LN2, logf(lsum));
}

// ------------------------------------------------------------------ forward (bf16)
// A workgroup covers 128 queries (32 per wave) and walks the keys in 64-row tiles, two LDS stages.
// MINW: waves per SIMD.
template <int DHP, int KC, bool CAUSAL, int MINW>
__global__ void __launch_bounds__(256, MINW) attn_fwd_bf16_kernel(const AttnK p) {
  constexpr int DT = DHP / 32, BQ = 128, TILE = 64 * DHP;
  __shared__ __attribute__((aligned(1024))) bf16 Ks[2][TILE];
  __shared__ __attribute__((aligned(1024))) bf16 Vs[2][TILE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, l32 = lane & 31;
  int qtile, bh;
  attn_block_map(blockIdx.x, (p.Nq + BQ - 1) / BQ, p.B * p.H, qtile, bh);
  const int b = bh / p.H, h = bh % p.H;
  const int q0 = qtile * BQ + wave * 32;               // first query of this wave
  const int qi = q0 + l32;
  const bf16* qb = (const bf16*)p.q + (size_t)b * p.Nq * p.ldq + h * p.dh;
  const bf16* kb = (const bf16*)p.k + (size_t)b * p.Nk * p.ldk + h * p.dh;
  const bf16* vb = (const bf16*)p.v + (size_t)b * p.Nk * p.ldv + h * p.dh;
  const u32x4 kr = make_raw_rsrc(kb, attn_slice_bytes(p.Nk, p.ldk, p.dh));
  const u32x4 vr = make_raw_rsrc(vb, attn_slice_bytes(p.Nk, p.ldv, p.dh));

  AttnFragOff<DHP, KC> fo;
  fo.init(lane);
  AttnTileCopy<DHP> ck, cv;
  ck.init(wave, lane, p.ldk, p.dh);
  cv.init(wave, lane, p.ldv, p.dh);
  ck.issue(kr, 0, p.ldk, Ks[0], wave);
  cv.issue(vr, 0, p.ldv, Vs[0], wave);

  bf16x8 qf[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) qf[c] = ld8(qb + (size_t)qi * p.ldq + 16 * c + 8 * g, qi < p.Nq && 16 * c + 8 * g < p.dh);
  f32x16 oacc[DT];
  float m = -INFINITY, lsum = 0.f;
#pragma unroll
  for (int i = 0; i < DT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;

  int nkt = (p.Nk + 63) / 64;
  if (CAUSAL) nkt = min(nkt, (min(p.Nq, qtile * BQ + BQ) + 63) / 64);
  wait_vmcnt<0>();
  __syncthreads();

  for (int kt = 0; kt < nkt; ++kt) {
    const int buf = kt & 1;
    take_turns(p.even, kt);
    if (kt + 1 < nkt) {      // every wave left stage buf ^ 1 at the barrier that ended the previous iteration
      ck.issue(kr, (kt + 1) * 64, p.ldk, Ks[buf ^ 1], wave);
      cv.issue(vr, (kt + 1) * 64, p.ldv, Vs[buf ^ 1], wave);
    }
    f32x16 s[2];
    auto scores = [&]() {      // S^T = K Q^T
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[t][r] = 0.f;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int c = 0; c < KC; ++c) s[t] = mfma32(fo.row_frag(Ks[buf], t, c), qf[c], s[t]);
      // Masking only in tiles that cross the end of the keys or the causal diagonal (one wave-uniform branch around a
      // block of selects; a test per element would be compiled into a branch per element)
      if (kt * 64 + 64 > p.Nk || (CAUSAL && kt * 64 + 63 > q0)) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = kt * 64 + 32 * t + acc_row(r, g);
            const bool dead = key >= p.Nk || (CAUSAL && key > qi);
            s[t][r] = dead ? -INFINITY : s[t][r];
          }
      }
    };
    // Online softmax, one query column per lane (shared with lane ^ 32).  The reference point m (scaled, log2 domain) only has to
    // bound the exponents, not equal the maximum, so no maximum is formed per tile: the probabilities are taken relative to the
    // old reference, and their sum, which is needed anyway and is at least the largest of them, tells whether some query of the wave
    // has outgrown it.  Only then (wave-uniform; always at the first tile) the scores are formed again, the reference is moved to 2^8
    // above the largest of them and the accumulators are rescaled.  Exact in the final O = acc / sum and LSE = ref + log sum.
    float rs;
    auto probabilities = [&]() {
      const float mref = m == -INFINITY ? 0.f : m;
      rs = 0.f;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float e = __builtin_amdgcn_exp2f(fmaf(s[t][r], p.scale_log2, -mref));
          s[t][r] = e;
          rs += e;
        }
    };
    auto move_reference = [&]() {
      float mx = -INFINITY;      // over raw scores (the scale is positive, so it commutes with max)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[t][r]);
      mx = fmaxf(m, fmaf(reduce_halves(mx, MaxOp()), p.scale_log2, 8.0f));
      if (kt > 0) {
        const float alpha = __builtin_amdgcn_exp2f(m - (mx == -INFINITY ? 0.f : mx));
        lsum *= alpha;
#pragma unroll
        for (int i = 0; i < DT; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
      }
      m = mx;
    };
    scores();
    if (kt == 0) move_reference();
    probabilities();
    if (__any(!(rs <= 256.f) || m == -INFINITY)) {
      if (kt > 0) {
        scores();
        move_reference();
        probabilities();
      }
    }
    lsum += rs;
    // O^T += V^T P^T
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        const bf16x8 pf = pack8(s[t], 8 * cc);
#pragma unroll
        for (int i = 0; i < DT; ++i) oacc[i] = mfma32(fo.tr_frag(Vs[buf], 32 * t + 16 * cc, i), pf, oacc[i]);
      }
    wait_vmcnt<0>();      // this wave's pieces of the next tile have landed
    __syncthreads();      // ... and everybody's; all reads of stage buf are done
  }

  attn_store_o<DT>(p, oacc, reduce_halves(lsum, AddOp()), m, b, h, qi, g);      // (each lane summed its own keys)
}

// ------------------------------------------------------------------ forward, at most 128 keys (bf16)
// All keys of the (batch, head) lie in LDS in NB blocks of 32 rows (the context's 77 are three, where the loop above walks over four), and a wave
// has all scores of its 32 queries in registers: one wait for memory, one maximum, one pass of exponentials, nothing to rescale, and under the
// causal mask no block past the wave's own.  What bounds it is vector instructions on many queries and, on the rows of a few samples, its chain of
// round trips.  Against the loop: 12 heads of 77 tokens, causal, 6.4 -> 4.7 us a launch, 144 heads 6.0 -> 4.2, 768 heads 11.7 -> 8.6; 77 keys
// and 8 x 5 heads of 4096 queries 17.6 -> 16.4, 8 x 10 of 1024 10.9 -> 10.4, 2 x 20 of 513 6.6 -> 5.8.
template <int DHP, int KC, int NB, bool CAUSAL, int MINW>
__global__ void __launch_bounds__(256, MINW) attn_fwd_short_bf16_kernel(const AttnK p) {
  constexpr int DT = DHP / 32, BQ = 128;
  __shared__ __attribute__((aligned(1024))) bf16 Ks[32 * NB * DHP];
  __shared__ __attribute__((aligned(1024))) bf16 Vs[32 * NB * DHP];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, l32 = lane & 31;
  int qtile, bh;
  attn_block_map(blockIdx.x, (p.Nq + BQ - 1) / BQ, p.B * p.H, qtile, bh);
  const int b = bh / p.H, h = bh % p.H;
  const int q0 = qtile * BQ + wave * 32, qi = q0 + l32;
  const bf16* qb = (const bf16*)p.q + (size_t)b * p.Nq * p.ldq + h * p.dh;
  const u32x4 kr = make_raw_rsrc((const bf16*)p.k + (size_t)b * p.Nk * p.ldk + h * p.dh, attn_slice_bytes(p.Nk, p.ldk, p.dh));
  const u32x4 vr = make_raw_rsrc((const bf16*)p.v + (size_t)b * p.Nk * p.ldv + h * p.dh, attn_slice_bytes(p.Nk, p.ldv, p.dh));
  AttnTileCopy<DHP> ck, cv;
  ck.init(wave, lane, p.ldk, p.dh);
  cv.init(wave, lane, p.ldv, p.dh);
  auto issue = [&](int row0) {      // 16 rows per wave
    if (row0 + 16 * wave >= 32 * NB) return;
    ck.issue(kr, row0, p.ldk, Ks + row0 * DHP, wave);
    cv.issue(vr, row0, p.ldv, Vs + row0 * DHP, wave);
  };
  issue(0);
  if constexpr (NB > 2) issue(64);
  AttnFragOff<DHP, KC> fo;
  fo.init(lane);
  bf16x8 qf[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) qf[c] = ld8(qb + (size_t)qi * p.ldq + 16 * c + 8 * g, qi < p.Nq && 16 * c + 8 * g < p.dh);
  wait_vmcnt<0>();
  __syncthreads();
  if (q0 >= p.Nq) return;

  const int blocks = CAUSAL ? min(NB, q0 / 32 + 1) : NB;
  f32x16 s[NB];      // S^T = K Q^T, a lane owns a query column
  float mx[2] = {-INFINITY, -INFINITY};      // of keys 0 .. 63 and of the others
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    if (CAUSAL && t >= blocks) continue;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[t][r] = 0.f;
#pragma unroll
    for (int c = 0; c < KC; ++c) s[t] = mfma32(fo.row_frag(Ks, t, c), qf[c], s[t]);
    if (32 * t + 32 > p.Nk || (CAUSAL && 32 * t + 31 > q0)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = 32 * t + acc_row(r, g);
        const bool dead = key >= p.Nk || (CAUSAL && key > qi);
        s[t][r] = dead ? -INFINITY : s[t][r];
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) mx[t / 2] = fmaxf(mx[t / 2], s[t][r]);
  }
  // The reference point of the loop, 2^8 above the largest of the first 64 keys, and its order of sums, so that the results are the loop's bit for
  // bit; where another key is more than 2^11 above them (the loop moves its reference at a sum of 2^16, 32 keys a lane), the largest of all.
  float m = fmaf(reduce_halves(mx[0], MaxOp()), p.scale_log2, 8.0f);      // (the scale is positive, so it commutes with the maximum)
  if constexpr (NB > 2) {
    const float m1 = fmaf(reduce_halves(mx[1], MaxOp()), p.scale_log2, 8.0f);
    m = m1 > m + 11.0f ? m1 : m;
  }
  const float mref = m == -INFINITY ? 0.f : m;
  f32x16 oacc[DT];
  float lsum = 0.f, rs = 0.f;
#pragma unroll
  for (int i = 0; i < DT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    if (CAUSAL && t >= blocks) continue;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[t][r] = __builtin_amdgcn_exp2f(fmaf(s[t][r], p.scale_log2, -mref));
      rs += s[t][r];
    }
    if (t & 1) lsum += rs, rs = 0.f;
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {      // O^T += V^T P^T
      const bf16x8 pf = pack8(s[t], 8 * cc);
#pragma unroll
      for (int i = 0; i < DT; ++i) oacc[i] = mfma32(fo.tr_frag(Vs, 32 * t + 16 * cc, i), pf, oacc[i]);
    }
  }
  attn_store_o<DT>(p, oacc, reduce_halves(lsum + rs, AddOp()), m, b, h, qi, g);
}

// ------------------------------------------------------------------ dQ (bf16)
template <int DHP, int KC>
__global__ void __launch_bounds__(256, DHP == 64 ? 3 : 2) attn_bwd_dq_bf16_kernel(const AttnK p) {
  constexpr int DT = DHP / 32, TILE = 64 * DHP;
  __shared__ __attribute__((aligned(1024))) bf16 Ks[2][TILE];
  __shared__ __attribute__((aligned(1024))) bf16 Vs[2][TILE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, l32 = lane & 31;
  int qtile, bh;
  attn_block_map(blockIdx.x, (p.Nq + 127) / 128, p.B * p.H, qtile, bh);
  const int b = bh / p.H, h = bh % p.H;
  const int qi = qtile * 128 + wave * 32 + l32;
  const bool qok = qi < p.Nq;
  const bf16* kb = (const bf16*)p.k + (size_t)b * p.Nk * p.ldk + h * p.dh;
  const bf16* vb = (const bf16*)p.v + (size_t)b * p.Nk * p.ldv + h * p.dh;
  const u32x4 kr = make_raw_rsrc(kb, attn_slice_bytes(p.Nk, p.ldk, p.dh));
  const u32x4 vr = make_raw_rsrc(vb, attn_slice_bytes(p.Nk, p.ldv, p.dh));
  const bf16* qrow = (const bf16*)p.q + ((size_t)b * p.Nq + qi) * p.ldq + h * p.dh;
  const bf16* dorow = (const bf16*)p.dout + ((size_t)b * p.Nq + qi) * p.lddo + h * p.dh;

  AttnFragOff<DHP, KC> fo;
  fo.init(lane);
  AttnTileCopy<DHP> ck, cv;
  ck.init(wave, lane, p.ldk, p.dh);
  cv.init(wave, lane, p.ldv, p.dh);
  ck.issue(kr, 0, p.ldk, Ks[0], wave);
  cv.issue(vr, 0, p.ldv, Vs[0], wave);

  bf16x8 qf[KC], dof[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const bool ok = qok && 16 * c + 8 * g < p.dh;
    qf[c] = ld8(qrow + 16 * c + 8 * g, ok);
    dof[c] = ld8(dorow + 16 * c + 8 * g, ok);
  }
  const size_t sidx = ((size_t)b * p.H + h) * p.Nq + qi;
  const float lse2 = qok ? p.lse[sidx] * LOG2E : INFINITY;
  // delta = rowsum(dO * O), computed here from the dO fragments the lane already holds (its half of
  // the head dimension; lane ^ 32 holds the other half) and stored for the dK/dV kernel, which runs
  // after this one on the same stream
  float dlt = 0.f;
  {
    const bf16* orow = (const bf16*)p.o + ((size_t)b * p.Nq + qi) * p.ldo + h * p.dh;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const bf16x8 of = ld8(orow + 16 * c + 8 * g, qok && 16 * c + 8 * g < p.dh);
#pragma unroll
      for (int u = 0; u < 8; ++u) dlt = fmaf((float)of[u], (float)dof[c][u], dlt);
    }
    dlt = reduce_halves(dlt, AddOp());
    if (qok && g == 0) p.delta[sidx] = dlt;
  }
  constexpr bool ONTO = KC < 6;      // dP - delta: the products accumulate onto -delta (the widest head has no registers for it)
  f32x16 ndelta;
#pragma unroll
  for (int r = 0; r < 16; ++r) ndelta[r] = ONTO ? -dlt : 0.f;

  f32x16 acc[DT];
#pragma unroll
  for (int i = 0; i < DT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

  const int nkt = (p.Nk + 63) / 64;
  wait_vmcnt<0>();
  __syncthreads();
  auto tile = [&](int kt, auto bc) {
    take_turns(p.even, kt);
    constexpr int buf = bc();
    if (kt + 1 < nkt) {      // every wave left stage buf ^ 1 at the barrier that ended the previous iteration
      ck.issue(kr, (kt + 1) * 64, p.ldk, Ks[buf ^ 1], wave);
      cv.issue(vr, (kt + 1) * 64, p.ldv, Vs[buf ^ 1], wave);
    }
    // Keys past Nk: their K and V rows are zero in LDS, so their dS multiplies a zero K row; it only has to be finite, which the exponential
    // is not where all logits of a query lie below -88
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x16 s, dp = ndelta;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        s = mfma32(fo.row_frag(Ks[buf], t, c), qf[c], s);
        dp = mfma32(fo.row_frag(Vs[buf], t, c), dof[c], dp);
      }
      if (kt * 64 + 64 > p.Nk) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = kt * 64 + 32 * t + acc_row(r, g) < p.Nk ? s[r] : -INFINITY;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], p.scale_log2, -lse2)) * (ONTO ? dp[r] : dp[r] - dlt);
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        const bf16x8 dsf = pack8(s, 8 * cc);
#pragma unroll
        for (int i = 0; i < DT; ++i) acc[i] = mfma32(fo.tr_frag(Ks[buf], 32 * t + 16 * cc, i), dsf, acc[i]);
      }
    }
    wait_vmcnt<0>();
    __syncthreads();
  };
  two_stages(0, nkt, tile);
  if (qok) {
    bf16* ob = (bf16*)p.dq + ((size_t)b * p.Nq + qi) * p.lddq + h * p.dh;
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int col = 32 * i + 8 * r4 + 4 * g;
        if (col < p.dh) {
          bf16x4 o;
#pragma unroll
          for (int u = 0; u < 4; ++u) o[u] = (bf16)(acc[i][4 * r4 + u] * p.scale);
          *reinterpret_cast<bf16x4*>(ob + col) = o;
        }
      }
  }
}

// A wave's dK and dV (lane: key ki): fp32 parts of a query share, reduced in a fixed order by attn_dkv_reduce_kernel, or the result.
template <int DT>
__device__ __forceinline__ void attn_store_dkv(const AttnK& p, const f32x16 (&dkacc)[DT], const f32x16 (&dvacc)[DT], int qs, int b, int h, int ki, bool kok, int g) {
  if (kok && p.qsplits > 1) {
    const size_t hd = (size_t)p.H * p.dh, rows = (size_t)p.B * p.Nk;
    float* pk = p.dkv_partial + ((size_t)qs * rows + (size_t)b * p.Nk + ki) * hd + h * p.dh;
    float* pv = pk + (size_t)p.qsplits * rows * hd;
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int col = 32 * i + 8 * r4 + 4 * g;
        if (col < p.dh) {
          f32x4 ok_, ov;
#pragma unroll
          for (int u = 0; u < 4; ++u) { ok_[u] = dkacc[i][4 * r4 + u] * p.scale; ov[u] = dvacc[i][4 * r4 + u]; }
          *reinterpret_cast<f32x4*>(pk + col) = ok_;
          *reinterpret_cast<f32x4*>(pv + col) = ov;
        }
      }
  } else if (kok) {
    bf16* dkb = (bf16*)p.dk + ((size_t)b * p.Nk + ki) * p.lddk + h * p.dh;
    bf16* dvb = (bf16*)p.dv + ((size_t)b * p.Nk + ki) * p.lddv + h * p.dh;
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int col = 32 * i + 8 * r4 + 4 * g;
        if (col < p.dh) {
          bf16x4 ok_, ov;
#pragma unroll
          for (int u = 0; u < 4; ++u) { ok_[u] = (bf16)(dkacc[i][4 * r4 + u] * p.scale); ov[u] = (bf16)dvacc[i][4 * r4 + u]; }
          *reinterpret_cast<bf16x4*>(dkb + col) = ok_;
          *reinterpret_cast<bf16x4*>(dvb + col) = ov;
        }
      }
  }
}

// ------------------------------------------------------------------ dK, dV (bf16)
// grid.x = ceil(Nk / 128) * qsplits; each wave owns 32 keys and walks its share of the query tiles.
// MINW: waves per SIMD, exactly: told only the least, the compiler schedules the variant of two for three as well, without the fragments
// fetched ahead that two need (8 x 4096 queries, 77 keys: 102 us instead of 75).
template <int DHP, int KC, int MINW>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MINW, MINW))) attn_bwd_dkv_bf16_kernel(const AttnK p) {
  constexpr int DT = DHP / 32, TILE = 64 * DHP;
  __shared__ __attribute__((aligned(1024))) bf16 Qs[2][TILE];
  __shared__ __attribute__((aligned(1024))) bf16 Ds[2][TILE];
  __shared__ __attribute__((aligned(16))) float lse_s[2][64];
  __shared__ __attribute__((aligned(16))) float dlt_s[2][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, l32 = lane & 31;
  int ktile, bh;
  const int qs = blockIdx.x % p.qsplits;
  attn_block_map(blockIdx.x / p.qsplits, (p.Nk + 127) / 128, p.B * p.H, ktile, bh);
  const int b = bh / p.H, h = bh % p.H;
  const int ki = ktile * 128 + wave * 32 + l32;
  const bool kok = ki < p.Nk;
  const bf16* qb = (const bf16*)p.q + (size_t)b * p.Nq * p.ldq + h * p.dh;
  const bf16* dob = (const bf16*)p.dout + (size_t)b * p.Nq * p.lddo + h * p.dh;
  const u32x4 qr = make_raw_rsrc(qb, attn_slice_bytes(p.Nq, p.ldq, p.dh));
  const u32x4 dr = make_raw_rsrc(dob, attn_slice_bytes(p.Nq, p.lddo, p.dh));
  const bf16* krow = (const bf16*)p.k + ((size_t)b * p.Nk + ki) * p.ldk + h * p.dh;
  const bf16* vrow = (const bf16*)p.v + ((size_t)b * p.Nk + ki) * p.ldv + h * p.dh;
  const float* lse_b = p.lse + ((size_t)b * p.H + h) * p.Nq;
  const float* dlt_b = p.delta + ((size_t)b * p.H + h) * p.Nq;

  // this workgroup's share of the 64-query tiles
  const int nqt_all = (p.Nq + 63) / 64, tps = (nqt_all + p.qsplits - 1) / p.qsplits;
  const int qt0 = qs * tps, nqt = min(nqt_all, qt0 + tps);
  AttnFragOff<DHP, KC> fo;
  fo.init(lane);
  AttnTileCopy<DHP> cq, cd;
  cq.init(wave, lane, p.ldq, p.dh);
  cd.init(wave, lane, p.lddo, p.dh);
  if (qt0 < nqt) {
    cq.issue(qr, qt0 * 64, p.ldq, Qs[0], wave);
    cd.issue(dr, qt0 * 64, p.lddo, Ds[0], wave);
  }
  // Statistics of a query tile: wave 0 fetches lse, wave 1 delta.  The value stays as loaded until the end of the tile before (a conversion
  // behind the load would wait for it there, and with it for the tile copies issued ahead of it: 373 -> 356 us at 40 heads of 4096 tokens).
  float stat = 0.f;
  const float* stat_b = wave == 0 ? lse_b : dlt_b;
  auto load_stats = [&](int qt) {
    if (wave < 2) stat = stat_b[min((uint32_t)(qt * 64 + lane), (uint32_t)p.Nq - 1u)];
  };
  auto store_stats = [&](int qt, int buf) {
    const bool ok = qt * 64 + lane < p.Nq;
    if (wave == 0) lse_s[buf][lane] = ok ? stat * LOG2E : INFINITY;
    if (wave == 1) dlt_s[buf][lane] = ok ? -stat : 0.f;
  };
  load_stats(qt0);

  bf16x8 kf[KC], vf[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const bool ok = kok && 16 * c + 8 * g < p.dh;
    kf[c] = ld8(krow + 16 * c + 8 * g, ok);
    vf[c] = ld8(vrow + 16 * c + 8 * g, ok);
  }
  f32x16 dkacc[DT], dvacc[DT];
#pragma unroll
  for (int i = 0; i < DT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dkacc[i][r] = 0.f; dvacc[i][r] = 0.f; }

  store_stats(qt0, 0);
  wait_vmcnt<0>();
  __syncthreads();

  auto tile = [&](int qt, auto bc) {
    take_turns(p.even, qt);
    constexpr int buf = bc();
    const bool more = qt + 1 < nqt;
    if (more) {
      cq.issue(qr, (qt + 1) * 64, p.ldq, Qs[buf ^ 1], wave);
      cd.issue(dr, (qt + 1) * 64, p.lddo, Ds[buf ^ 1], wave);
      load_stats(qt + 1);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (MINW > 2) __builtin_amdgcn_sched_barrier(0);      // (the halves' fragments would overlap in registers, past the 168 of three waves per SIMD)
      f32x16 s, dp;      // dP - delta: the products accumulate onto -delta
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 d4 = *reinterpret_cast<const f32x4*>(&dlt_s[buf][32 * t + 8 * r4 + 4 * g]);
#pragma unroll
        for (int u = 0; u < 4; ++u) { s[4 * r4 + u] = 0.f; dp[4 * r4 + u] = d4[u]; }
      }
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        s = mfma32(fo.row_frag(Qs[buf], t, c), kf[c], s);
        dp = mfma32(fo.row_frag(Ds[buf], t, c), vf[c], dp);
      }
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(&lse_s[buf][32 * t + 8 * r4 + 4 * g]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r = 4 * r4 + u;
          // a lane whose key is past Nk computes garbage that stays in its own accumulator columns,
          // which are never stored; queries past Nq have lse = +inf, hence pr = 0
          s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], p.scale_log2, -l4[u]));
          dp[r] *= s[r];
        }
      }
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        const bf16x8 pf = pack8(s, 8 * cc);
        const bf16x8 dsf = pack8(dp, 8 * cc);
#pragma unroll
        for (int i = 0; i < DT; ++i) {
          dvacc[i] = mfma32(fo.tr_frag(Ds[buf], 32 * t + 16 * cc, i), pf, dvacc[i]);
          dkacc[i] = mfma32(fo.tr_frag(Qs[buf], 32 * t + 16 * cc, i), dsf, dkacc[i]);
        }
      }
    }
    if (MINW > 2) __builtin_amdgcn_sched_barrier(0);
    if (more) store_stats(qt + 1, buf ^ 1);
    wait_vmcnt<0>();
    __syncthreads();
  };
  two_stages(qt0, nqt, tile);
  attn_store_dkv<DT>(p, dkacc, dvacc, qs, b, h, ki, kok, g);
}

// ------------------------------------------------------------------ dQ, dK, dV at once (bf16, at most 32 NW keys)
// A workgroup has all keys of its (batch, head), 32 per wave, and walks the queries (of its share) in tiles of 64: scores, dP and the
// exponentials are formed once where the two kernels above form them twice, and delta and the statistics need no pass of their own.
// Per tile: every wave adds to its keys' dK and dV and leaves dS in LDS ([key][query], the layout of a 64-wide tile); behind a barrier
// the dQ of the tile, 2 DHP / 32 blocks of 32 x 32, is formed from it and the keys in LDS, by as many waves, while the next
// tile's delta = rowsum(dO * O) is formed from its O (registers, fetched a tile ahead) and its dO (LDS).
//
// Why: what these kernels are bound by, power and issue slots, is spent in proportion to the products, five instead of seven, and the
// exponentials, one instead of two.  Both kernels -> this one, inside a step: 32 x 16 heads of 256 tokens, width 72, 91 -> 68 us; 77 keys and
// 8 x 5 heads of 4096 queries 59 -> 40, 8 x 10 of 1024 40 -> 22, 2 x 20 of 513 23 -> 15.  A workgroup of the first shape takes 32 us: 6 until the
// keys are there (K and V are read by rows through LDS; fragments straight from memory took 9), 5.4 per tile of which 3 are the products of the
// first part, 3 to store.
template <int DHP, int NW> struct AttnShort {
  static constexpr int TILE = 64 * DHP, K = 32 * NW * DHP, DS = 32 * NW * 64;                            // elements
  static_assert(K <= 2 * TILE + DS, "V passes through the second stage and dS");
  static constexpr size_t BYTES = (size_t)(K + 4 * TILE + DS) * sizeof(bf16) + 2 * 64 * sizeof(float);
};
template <int DHP, int KC, int NW>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) attn_bwd_short_bf16_kernel(const AttnK p) {
  using S = AttnShort<DHP, NW>;
  constexpr int DT = DHP / 32, TILE = S::TILE;
  constexpr int LPR = DHP == 64 ? 8 : 16, RPP = 64 / LPR, PASSES = 64 / (NW * RPP);      // delta: lanes a row, rows a pass of a wave
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  // what the products of every tile read comes first: an LDS instruction reaches 64 KB past its base register
  bf16* const QD = reinterpret_cast<bf16*>(smem);      // two stages of Q and dO
  bf16* const dS = QD + 4 * TILE;
  bf16* const Vt = QD + 2 * TILE;                      // V on its way to the registers: where the second stage and dS will be
  bf16* const Kt = dS + S::DS;
  float* const lse_s = reinterpret_cast<float*>(Kt + S::K);
  float* const dlt_s = lse_s + 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, l32 = lane & 31;
  int qs, bh;
  attn_block_map(blockIdx.x, p.qsplits, p.B * p.H, qs, bh);
  const int b = bh / p.H, h = bh % p.H, ki = 32 * wave + l32, groups = (p.Nk + 31) / 32;      // (a wave past the last group has copies, dQ and delta)
  const bool kok = ki < p.Nk;
  const bf16* qb = (const bf16*)p.q + (size_t)b * p.Nq * p.ldq + h * p.dh;
  const bf16* dob = (const bf16*)p.dout + (size_t)b * p.Nq * p.lddo + h * p.dh;
  const bf16* ob = (const bf16*)p.o + (size_t)b * p.Nq * p.ldo + h * p.dh;
  const bf16* kb = (const bf16*)p.k + (size_t)b * p.Nk * p.ldk + h * p.dh;
  const bf16* vb = (const bf16*)p.v + (size_t)b * p.Nk * p.ldv + h * p.dh;
  const float* lse_b = p.lse + ((size_t)b * p.H + h) * p.Nq;
  const u32x4 qr = make_raw_rsrc(qb, attn_slice_bytes(p.Nq, p.ldq, p.dh)), dr = make_raw_rsrc(dob, attn_slice_bytes(p.Nq, p.lddo, p.dh));
  const u32x4 kr = make_raw_rsrc(kb, attn_slice_bytes(p.Nk, p.ldk, p.dh)), vr = make_raw_rsrc(vb, attn_slice_bytes(p.Nk, p.ldv, p.dh));
  const int nqt_all = (p.Nq + 63) / 64, tps = (nqt_all + p.qsplits - 1) / p.qsplits;
  const int qt0 = qs * tps, nqt = min(nqt_all, qt0 + tps);      // no share is empty

  AttnFragOff<DHP, KC> fo;
  fo.init(lane);
  // four waves copy a query tile of both kinds, eight one kind each
  AttnTileCopy<DHP> ck, cv, cq, cd;
  ck.init(wave, lane, p.ldk, p.dh);
  cv.init(wave, lane, p.ldv, p.dh);
  cq.init(wave & 3, lane, p.ldq, p.dh);
  cd.init(wave & 3, lane, p.lddo, p.dh);
  auto issue = [&](int qt) {
    const int at = (qt - qt0) & 1;
    if (NW == 4 || wave < 4) cq.issue(qr, qt * 64, p.ldq, QD + at * 2 * TILE, wave & 3);
    if (NW == 4 || wave >= 4) cd.issue(dr, qt * 64, p.lddo, QD + (at * 2 + 1) * TILE, wave & 3);
  };
  // O and the logarithms of the sums of a tile, kept as loaded until delta is due
  bf16x8 of[PASSES];
  float stat = 0.f;
  const int drow = wave * RPP + lane / LPR, dchunk = lane % LPR;
  auto load_o = [&](int qt) {
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      const int q = qt * 64 + i * NW * RPP + drow;
      of[i] = ld8(ob + (size_t)q * p.ldo + 8 * dchunk, q < p.Nq && 8 * dchunk < p.dh);
    }
    if (wave == 0) stat = lse_b[min((uint32_t)(qt * 64 + lane), (uint32_t)p.Nq - 1u)];
  };
  auto statistics = [&](int qt) {
    const bf16* tile = QD + (((qt - qt0) & 1) * 2 + 1) * TILE;
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      const int row = i * NW * RPP + drow;
      float v = 0.f;
      if (dchunk < DHP / 8) {
        const bf16x8 df = *reinterpret_cast<const bf16x8*>(tile + row * DHP + 8 * (dchunk ^ AttnTile<DHP>::key(row)));
#pragma unroll
        for (int u = 0; u < 8; ++u) v = fmaf((float)of[i][u], (float)df[u], v);
      }
      v += lane_dpp<0xB1>(v);       // quad_perm:[1,0,3,2]
      v += lane_dpp<0x4E>(v);       // quad_perm:[2,3,0,1]
      v += lane_dpp<0x141>(v);      // row_half_mirror: the other quad of eight
      if (LPR == 16) v += lane_dpp<0x128>(v);      // row_ror:8
      if (dchunk == 0) dlt_s[row] = -v;
    }
    if (wave == 0) lse_s[lane] = qt * 64 + lane < p.Nq ? stat * LOG2E : INFINITY;
  };

  ck.issue(kr, 0, p.ldk, Kt, wave);
  cv.issue(vr, 0, p.ldv, Vt, wave);
  ck.issue(kr, 16 * NW, p.ldk, Kt + 16 * NW * DHP, wave);
  cv.issue(vr, 16 * NW, p.ldv, Vt + 16 * NW * DHP, wave);
  issue(qt0);
  load_o(qt0);
  f32x16 dkacc[DT], dvacc[DT];
#pragma unroll
  for (int i = 0; i < DT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dkacc[i][r] = 0.f; dvacc[i][r] = 0.f; }
  wait_vmcnt<0>();
  __syncthreads();
  bf16x8 kf[KC], vf[KC];      // rows past the last key are zero
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    kf[c] = fo.row_frag(Kt + 32 * wave * DHP, 0, c);
    vf[c] = fo.row_frag(Vt + 32 * wave * DHP, 0, c);
  }
  statistics(qt0);
  lds_barrier();
  if (wave >= groups) {      // keys that are not there: the products for dQ run over all of them
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(dS + 32 * wave * 64 + 512 * i + 8 * lane) = u32x4{0u, 0u, 0u, 0u};
  }
  if (qt0 + 1 < nqt) {
    issue(qt0 + 1);
    load_o(qt0 + 1);
  }

  auto frag = [](const bf16* lo, const bf16* hi) {
    const bf16x4 a = lds_read_tr(lo), c = lds_read_tr(hi);
    return __builtin_shufflevector(a, c, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto tile = [&](int qt, auto bc) {
    const bf16* Q = QD + bc() * 2 * TILE;
    const bf16* D = Q + TILE;
    if (wave < groups) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x16 s, dp;      // dP - delta: the products accumulate onto -delta
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const f32x4 d4 = *reinterpret_cast<const f32x4*>(dlt_s + 32 * t + 8 * r4 + 4 * g);
#pragma unroll
          for (int u = 0; u < 4; ++u) { s[4 * r4 + u] = 0.f; dp[4 * r4 + u] = d4[u]; }
        }
#pragma unroll
        for (int c = 0; c < KC; ++c) {
          s = mfma32(fo.row_frag(Q, t, c), kf[c], s);
          dp = mfma32(fo.row_frag(D, t, c), vf[c], dp);
        }
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const f32x4 l4 = *reinterpret_cast<const f32x4*>(lse_s + 32 * t + 8 * r4 + 4 * g);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int r = 4 * r4 + u;
            s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], p.scale_log2, -l4[u]));      // queries past Nq have lse = +inf, hence 0
            dp[r] *= s[r];
          }
        }
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
          const bf16x8 pf = pack8(s, 8 * cc);
          const bf16x8 dsf = pack8(dp, 8 * cc);
          // a key past Nk computes garbage that stays in its own columns of dK and dV, which are never stored; its dS meets a zero
          // row of K, so it only has to be finite
#pragma unroll
          for (int q4 = 0; q4 < 2; ++q4) {
            const bf16x4 v = q4 ? __builtin_shufflevector(dsf, dsf, 4, 5, 6, 7) : __builtin_shufflevector(dsf, dsf, 0, 1, 2, 3);
            *reinterpret_cast<u32x2*>(dS + ki * 64 + 8 * ((4 * t + 2 * cc + q4) ^ AttnTile<64>::key(l32)) + 4 * g) =
                kok ? __builtin_bit_cast(u32x2, v) : u32x2{0u, 0u};
          }
#pragma unroll
          for (int i = 0; i < DT; ++i) {
            dvacc[i] = mfma32(fo.tr_frag(D, 32 * t + 16 * cc, i), pf, dvacc[i]);
            dkacc[i] = mfma32(fo.tr_frag(Q, 32 * t + 16 * cc, i), dsf, dkacc[i]);
          }
        }
      }
    }
    wait_vmcnt<0>();
    __syncthreads();      // dS is there, and the next tile
    const bool more = qt + 1 < nqt;
    if (more) statistics(qt + 1);
    if (qt + 2 < nqt) {
      issue(qt + 2);
      load_o(qt + 2);
    }
    // dQ of the tile: blocks of 32 columns (di) x 32 queries (dt)
    for (int n = wave; n < 2 * DT; n += NW) {
      const int di = n % DT, dt = n / DT;
      int kt_lo, kt_hi, ds_lo, ds_hi;
      AttnFragOff<DHP, KC>::transposed(lane, di, kt_lo, kt_hi);
      AttnFragOff<64, KC>::transposed(lane, dt, ds_lo, ds_hi);
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
      for (int r = 0; r < 32 * NW; r += 16) acc = mfma32(frag(Kt + kt_lo + r * DHP, Kt + kt_hi + r * DHP), frag(dS + ds_lo + r * 64, dS + ds_hi + r * 64), acc);
      const int q = qt * 64 + 32 * dt + l32;
      if (q < p.Nq) {
        bf16* o = (bf16*)p.dq + ((size_t)b * p.Nq + q) * p.lddq + h * p.dh;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const int col = 32 * di + 8 * r4 + 4 * g;
          if (col < p.dh) {
            bf16x4 v;
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = (bf16)(acc[4 * r4 + u] * p.scale);
            *reinterpret_cast<bf16x4*>(o + col) = v;
          }
        }
      }
    }
    lds_barrier();      // dS has been read, the statistics of the next tile are there
  };
  two_stages(qt0, nqt, tile);
  attn_store_dkv<DT>(p, dkacc, dvacc, qs, b, h, ki, kok, g);
}

// dk[row, col] = sum_qs partial_k[qs][row][col] (ascending qs), same for dv; 4 columns per thread.
__global__ void attn_dkv_reduce_kernel(const float* __restrict__ partial, int qsplits, size_t rows, int hd, bf16* __restrict__ dk, int lddk,
                                       bf16* __restrict__ dv, int lddv) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  const int per_row = hd / 4;
  if (i >= rows * per_row) return;
  const size_t row = i / per_row; const int col = (int)(i % per_row) * 4;
  f32x4 sk = {0.f, 0.f, 0.f, 0.f}, sv = sk;
  const size_t plane = rows * hd;
  for (int q = 0; q < qsplits; ++q) {
    sk += *reinterpret_cast<const f32x4*>(partial + (size_t)q * plane + row * hd + col);
    sv += *reinterpret_cast<const f32x4*>(partial + ((size_t)qsplits + q) * plane + row * hd + col);
  }
  bf16x4 ok_, ov;
#pragma unroll
  for (int u = 0; u < 4; ++u) { ok_[u] = (bf16)sk[u]; ov[u] = (bf16)sv[u]; }
  *reinterpret_cast<bf16x4*>(dk + row * lddk + col) = ok_;
  *reinterpret_cast<bf16x4*>(dv + row * lddv + col) = ov;
}

// ------------------------------------------------------------------ fp32 path (one wave per row)
constexpr int F32_MAX_DH = 256;

// Small problems: bound by the latency of one load after the other, so the loops request sixteen values at a time (order of the sums as written).  2 x 64
// rows, 4 heads of 16: 6.0 -> 5.0 us forward, 4.9 -> 4.3 dQ; the dK/dV kernel, which reads two operands a step, takes 10.7 instead of 6.2 that way.
__global__ void __launch_bounds__(64) attn_fwd_f32_kernel(const AttnK p, int causal) {
  extern __shared__ float sc[];        // [Nk]
  __shared__ float qs[F32_MAX_DH];
  const int lane = threadIdx.x, i = blockIdx.x, b = blockIdx.y / p.H, h = blockIdx.y % p.H;
  const float* q = (const float*)p.q + ((size_t)b * p.Nq + i) * p.ldq + h * p.dh;
  const float* kb = (const float*)p.k + (size_t)b * p.Nk * p.ldk + h * p.dh;
  const float* vb = (const float*)p.v + (size_t)b * p.Nk * p.ldv + h * p.dh;
  for (int t = lane; t < p.dh; t += 64) qs[t] = q[t];
  __syncthreads();
  float mx = -INFINITY;
  for (int j = lane; j < p.Nk; j += 64) {
    float s = 0.f;
#pragma unroll 16
    for (int t = 0; t < p.dh; ++t) s = fmaf(qs[t], kb[(size_t)j * p.ldk + t], s);
    s *= p.scale;
    if (causal && j > i) s = -INFINITY;
    sc[j] = s;
    mx = fmaxf(mx, s);
  }
  mx = wave_max(mx);
  float sum = 0.f;
  for (int j = lane; j < p.Nk; j += 64) {
    const float e = expf(sc[j] - mx);
    sc[j] = e;
    sum += e;
  }
  sum = wave_sum(sum);
  __syncthreads();
  float* o = (float*)p.o + ((size_t)b * p.Nq + i) * p.ldo + h * p.dh;
  for (int t = lane; t < p.dh; t += 64) {
    float a = 0.f;
#pragma unroll 16
    for (int j = 0; j < p.Nk; ++j) a = fmaf(sc[j], vb[(size_t)j * p.ldv + t], a);
    o[t] = a / sum;
  }
  if (p.lse && lane == 0) p.lse[((size_t)b * p.H + h) * p.Nq + i] = mx + logf(sum);
}

__device__ __forceinline__ void attn_bwd_dq_f32_row(const AttnK& p, int i, float* sc, float* qs, float* dos) {      // sc: [Nk]
  const int lane = threadIdx.x, b = blockIdx.y / p.H, h = blockIdx.y % p.H;
  const float* q = (const float*)p.q + ((size_t)b * p.Nq + i) * p.ldq + h * p.dh;
  const float* dor = (const float*)p.dout + ((size_t)b * p.Nq + i) * p.lddo + h * p.dh;
  const float* kb = (const float*)p.k + (size_t)b * p.Nk * p.ldk + h * p.dh;
  const float* vb = (const float*)p.v + (size_t)b * p.Nk * p.ldv + h * p.dh;
  // delta = rowsum(dO * O), also stored for the dK/dV kernel that follows on the stream
  const float* orow = (const float*)p.o + ((size_t)b * p.Nq + i) * p.ldo + h * p.dh;
  const size_t sidx = ((size_t)b * p.H + h) * p.Nq + i;
  const float lse = p.lse[sidx];
  float dlt = 0.f;
  for (int t = lane; t < p.dh; t += 64) { qs[t] = q[t]; dos[t] = dor[t]; dlt = fmaf(dor[t], orow[t], dlt); }
  dlt = wave_sum(dlt);
  if (lane == 0) p.delta[sidx] = dlt;
  __syncthreads();
  for (int j = lane; j < p.Nk; j += 64) {
    float s = 0.f, dp = 0.f;
#pragma unroll 16
    for (int t = 0; t < p.dh; ++t) {
      s = fmaf(qs[t], kb[(size_t)j * p.ldk + t], s);
      dp = fmaf(dos[t], vb[(size_t)j * p.ldv + t], dp);
    }
    sc[j] = expf(s * p.scale - lse) * (dp - dlt);
  }
  __syncthreads();
  float* dq = (float*)p.dq + ((size_t)b * p.Nq + i) * p.lddq + h * p.dh;
  for (int t = lane; t < p.dh; t += 64) {
    float a = 0.f;
#pragma unroll 16
    for (int j = 0; j < p.Nk; ++j) a = fmaf(sc[j], kb[(size_t)j * p.ldk + t], a);
    dq[t] = a * p.scale;
  }
}

// OWN_DELTA: forms delta itself, four sums side by side, instead of reading what the dQ kernel left.
template <bool OWN_DELTA>
__device__ __forceinline__ void attn_bwd_dkv_f32_row(const AttnK& p, int j, float* sc, float* ks, float* vs) {      // sc: [2][Nq], p and ds
  const int lane = threadIdx.x, b = blockIdx.y / p.H, h = blockIdx.y % p.H;
  const float* kr = (const float*)p.k + ((size_t)b * p.Nk + j) * p.ldk + h * p.dh;
  const float* vr = (const float*)p.v + ((size_t)b * p.Nk + j) * p.ldv + h * p.dh;
  const float* qb = (const float*)p.q + (size_t)b * p.Nq * p.ldq + h * p.dh;
  const float* dob = (const float*)p.dout + (size_t)b * p.Nq * p.lddo + h * p.dh;
  const float* lse_b = p.lse + ((size_t)b * p.H + h) * p.Nq;
  const float* dlt_b = p.delta + ((size_t)b * p.H + h) * p.Nq;
  for (int t = lane; t < p.dh; t += 64) { ks[t] = kr[t]; vs[t] = vr[t]; }
  __syncthreads();
  float* pp = sc; float* dsp = sc + p.Nq;
  for (int i = lane; i < p.Nq; i += 64) {
    float s = 0.f, dp = 0.f, dlt = 0.f;
    if constexpr (OWN_DELTA) {
      const float* ob = (const float*)p.o + ((size_t)b * p.Nq + i) * p.ldo + h * p.dh;
      float part[4] = {0.f, 0.f, 0.f, 0.f};
      int t = 0;
      for (; t + 4 <= p.dh; t += 4)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float dor = dob[(size_t)i * p.lddo + t + u];
          s = fmaf(qb[(size_t)i * p.ldq + t + u], ks[t + u], s);
          dp = fmaf(dor, vs[t + u], dp);
          part[u] = fmaf(dor, ob[t + u], part[u]);
        }
      for (; t < p.dh; ++t) {
        const float dor = dob[(size_t)i * p.lddo + t];
        s = fmaf(qb[(size_t)i * p.ldq + t], ks[t], s);
        dp = fmaf(dor, vs[t], dp);
        part[0] = fmaf(dor, ob[t], part[0]);
      }
      dlt = (part[0] + part[1]) + (part[2] + part[3]);
    } else {
      for (int t = 0; t < p.dh; ++t) {
        s = fmaf(qb[(size_t)i * p.ldq + t], ks[t], s);
        dp = fmaf(dob[(size_t)i * p.lddo + t], vs[t], dp);
      }
      dlt = dlt_b[i];
    }
    const float pr = expf(s * p.scale - lse_b[i]);
    pp[i] = pr;
    dsp[i] = pr * (dp - dlt);
  }
  __syncthreads();
  float* dk = (float*)p.dk + ((size_t)b * p.Nk + j) * p.lddk + h * p.dh;
  float* dv = (float*)p.dv + ((size_t)b * p.Nk + j) * p.lddv + h * p.dh;
  for (int t = lane; t < p.dh; t += 64) {
    float a = 0.f, c = 0.f;
    for (int i = 0; i < p.Nq; ++i) {
      a = fmaf(dsp[i], qb[(size_t)i * p.ldq + t], a);
      c = fmaf(pp[i], dob[(size_t)i * p.lddo + t], c);
    }
    dk[t] = a * p.scale;
    dv[t] = c;
  }
}

__global__ void __launch_bounds__(64) attn_bwd_dq_f32_kernel(const AttnK p) {
  extern __shared__ float sc[];
  __shared__ float qs[F32_MAX_DH], dos[F32_MAX_DH];
  attn_bwd_dq_f32_row(p, blockIdx.x, sc, qs, dos);
}
__global__ void __launch_bounds__(64) attn_bwd_dkv_f32_kernel(const AttnK p) {
  extern __shared__ float sc[];
  __shared__ float ks[F32_MAX_DH], vs[F32_MAX_DH];
  attn_bwd_dkv_f32_row<false>(p, blockIdx.x, sc, ks, vs);
}
// Both in one launch: workgroups 0 .. Nk - 1 take keys, which are the longer work, the others queries.
__global__ void __launch_bounds__(64) attn_bwd_both_f32_kernel(const AttnK p) {
  extern __shared__ float sc[];
  __shared__ float r0[F32_MAX_DH], r1[F32_MAX_DH];
  if ((int)blockIdx.x < p.Nk) attn_bwd_dkv_f32_row<true>(p, blockIdx.x, sc, r0, r1);
  else attn_bwd_dq_f32_row(p, blockIdx.x - p.Nk, sc, r0, r1);
}

// ------------------------------------------------------------------ host side
static AttnK make_k(const AttnArgs& a) {
  AttnK k;
  k.B = a.B; k.H = a.H; k.Nq = a.Nq; k.Nk = a.Nk; k.dh = a.d_head;
  k.scale = a.scale; k.scale_log2 = a.scale * LOG2E;
  k.q = a.q; k.ldq = a.ldq; k.k = a.k; k.ldk = a.ldk; k.v = a.v; k.ldv = a.ldv; k.o = a.o; k.ldo = a.ldo; k.lse = a.lse;
  k.dout = a.dout; k.lddo = a.lddo; k.delta = a.delta; k.dq = a.dq; k.lddq = a.lddq; k.dk = a.dk; k.lddk = a.lddk;
  k.dv = a.dv; k.lddv = a.lddv;
  k.even = 0; k.qsplits = 1; k.dkv_partial = nullptr;
  return k;
}

static int check_attn(const AttnArgs& a, bool bwd) {
  if (a.B <= 0 || a.H <= 0 || a.Nq <= 0 || a.Nk <= 0 || a.d_head <= 0) return set_error(DP_EINVAL, "attention: non-positive size");
  if (!a.q || !a.k || !a.v || !a.o) return set_error(DP_EINVAL, "attention: null operand");
  if ((size_t)a.B * a.H > 65535) return set_error(DP_EUNSUPPORTED, "attention: batch * heads exceeds 65535");
  const int span = a.H * a.d_head;
  if (a.ldq < span || a.ldk < span || a.ldv < span || a.ldo < span) return set_error(DP_EINVAL, "attention: leading dim smaller than heads * d_head");
  if (bwd) {
    if (!a.dout || !a.lse || !a.delta || !a.dq || !a.dk || !a.dv) return set_error(DP_EINVAL, "attention backward: null operand");
    if (a.lddo < span || a.lddq < span || a.lddk < span || a.lddv < span) return set_error(DP_EINVAL, "attention backward: leading dim too small");
    if (a.causal) return set_error(DP_EUNSUPPORTED, "attention backward: causal mask not supported (the causal encoder is frozen)");
  }
  if (a.dtype == BF16) {
    if (a.d_head % 8 || a.d_head > 96) return set_error(DP_EUNSUPPORTED, "attention(bf16): d_head must be a multiple of 8, at most 96");
    const int lds[] = {a.ldq, a.ldk, a.ldv, a.ldo, bwd ? a.lddo : 8, bwd ? a.lddq : 8, bwd ? a.lddk : 8, bwd ? a.lddv : 8};
    for (int x : lds) if (x % 8) return set_error(DP_EUNSUPPORTED, "attention(bf16): leading dims must be multiples of 8");
    const void* ps[] = {a.q, a.k, a.v, a.o, bwd ? a.dout : a.q, bwd ? a.dq : a.q, bwd ? a.dk : a.q, bwd ? a.dv : a.q};
    for (const void* x : ps) if ((uintptr_t)x % 16) return set_error(DP_EALIGN, "attention(bf16): operands must be 16-byte aligned");
    // the tile copies address one (batch, head) slice with 32-bit byte offsets and keep bit 31 for "no data"
    const size_t maxld = (size_t)std::max(std::max(a.ldq, a.ldk), std::max(a.ldv, bwd ? a.lddo : 8));
    if ((size_t)std::max(a.Nq, a.Nk) * maxld * 2 >= (1ull << 31)) return set_error(DP_EUNSUPPORTED, "attention(bf16): one batch element's q / k / v rows must span less than 2 GiB");
  } else {
    if (a.d_head > F32_MAX_DH) return set_error(DP_EUNSUPPORTED, "attention(fp32): d_head > 256");
    if ((size_t)a.Nk * 4 > 60000 || (bwd && (size_t)a.Nq * 8 > 60000)) return set_error(DP_EUNSUPPORTED, "attention(fp32): sequence too long for the fp32 path");
  }
  return DP_OK;
}

// Whether `blocks` workgroups, `per_cu` of which fit a CU, are all resident and share CUs.
static int takes_turns(long blocks, int per_cu) { return blocks > 256 && blocks <= 256L * per_cu; }

size_t attn_dkv_ws_bytes(int B, int H, int Nk, int d_head) { return 2 * (size_t)16 * B * Nk * H * d_head * sizeof(float); }

// Calls f(padded head width of the tiles, 16-column steps of the products over the head dimension): tiles are 64 or 96 columns wide for the
// copies and the transposing reads, the steps end with the head (d_head 72: five of six).
template <class F> static void attn_dispatch(int d_head, F f) {
  using std::integral_constant;
  if (d_head <= 48) f(integral_constant<int, 64>(), integral_constant<int, 3>());
  else if (d_head <= 64) f(integral_constant<int, 64>(), integral_constant<int, 4>());
  else if (d_head <= 80) f(integral_constant<int, 96>(), integral_constant<int, 5>());
  else f(integral_constant<int, 96>(), integral_constant<int, 6>());
}

// Whether the forward has all keys in LDS at once.  Beyond 120 keys a fourth block of 32 is full or nearly so, and its workgroups begin when all of it
// is there, where the loop fetches the second tile beside its work on the first: many heads of one tile of queries, which are bound by memory, are faster in the loop (128 keys
// and queries, 512 / 768 / 1024 heads, loop and all at once, us: width 40 9.4 / 13.2 / 17.1 and 9.8 / 14.3 / 18.0, 72 12.9 / 17.8 / 22.6 and 13.8 / 19.0 / 23.7, 96 14.1 / 19.3 /
// 24.6 and 15.1 / 20.8 / 25.9; 384 heads 8.1 / 10.7 / 11.7 and 8.1 / 10.4 / 11.1; width 64 7.7 / 12.4 / 16.0 and 7.6 / 12.9 / 16.2, 2048 heads 28.1 and 27.0; 113 keys, 768 heads of
// width 72 16.6 and 17.3, 1536 29.8 and 29.0; causal 512 of 96 1.04x, 1024 0.99x).
static bool attn_all_keys(const AttnArgs& a, long blocks) {
  if (a.Nk <= 120) return true;
  return a.Nk <= 128 && (a.causal || a.Nq > 128 || blocks < 512 || (a.d_head > 48 && a.d_head <= 64));
}

int launch_attn_fwd(const AttnArgs& a, hipStream_t s) {
  if (int e = check_attn(a, false)) return e;
  AttnK k = make_k(a);
  k.even = takes_turns((long)((a.Nq + 127) / 128) * a.B * a.H, a.d_head <= 64 ? 4 : 3);
  const double fl = 4.0 * a.B * a.H * (double)a.Nq * a.Nk * a.d_head;
  const double by = dtype_size(a.dtype) * (double)a.B * a.H * a.d_head * (2.0 * a.Nq + 2.0 * a.Nk);
  KScope ks(a.dtype == BF16 ? KK_ATTN_FWD : KK_ATTN_F32, fl, by, s, a.Nq, a.Nk, a.d_head);
  if (a.dtype == BF16) {
    dim3 grid(((a.Nq + 127) / 128) * a.B * a.H);
    attn_dispatch(a.d_head, [&](auto dhp, auto kc) {
      if (attn_all_keys(a, grid.x)) {
        auto launch = [&](auto nb) {
          constexpr int W = dhp == 64 && nb < 4 ? 4 : 3;
          if (a.causal) hipLaunchKernelGGL((attn_fwd_short_bf16_kernel<dhp, kc, nb, true, W>), grid, dim3(256), 0, s, k);
          else hipLaunchKernelGGL((attn_fwd_short_bf16_kernel<dhp, kc, nb, false, W>), grid, dim3(256), 0, s, k);
        };
        using std::integral_constant;
        if (a.Nk <= 32) launch(integral_constant<int, 1>());
        else if (a.Nk <= 64) launch(integral_constant<int, 2>());
        else if (a.Nk <= 96) launch(integral_constant<int, 3>());
        else launch(integral_constant<int, 4>());
        return;
      }
      // The causal mask costs the kernel of four waves per SIMD two spilled registers at widths above 48: it is for the launches that a CU holds with
      // four workgroups and not with three, which would start in two rounds (three -> four: 400 heads of 256 tokens 20.1 -> 17.6 us, 512 20.3 -> 19.0, 200
      // of 512 27.9 -> 23.2, 256 28.4 -> 24.6, 128 of 1024 37.9 -> 37.0; on either side 384 of 256 15.2 and 15.3, 520 21.8 -> 24.2, 600 22.8 -> 25.3)
      constexpr bool FOUR = dhp == 64 && kc == 4;
      if (FOUR && a.causal && grid.x > 3 * 256 && grid.x <= 4 * 256) hipLaunchKernelGGL((attn_fwd_bf16_kernel<dhp, kc, true, FOUR ? 4 : 3>), grid, dim3(256), 0, s, k);
      else if (a.causal) hipLaunchKernelGGL((attn_fwd_bf16_kernel<dhp, kc, true, 3>), grid, dim3(256), 0, s, k);
      else hipLaunchKernelGGL((attn_fwd_bf16_kernel<dhp, kc, false, dhp == 64 ? 4 : 3>), grid, dim3(256), 0, s, k);
    });
  } else {
    hipLaunchKernelGGL(attn_fwd_f32_kernel, dim3(a.Nq, a.B * a.H), dim3(64), (size_t)a.Nk * sizeof(float), s, k, a.causal);
  }
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "attention forward launch failed");
}

static size_t dkv_partial_bytes(const AttnArgs& a, int qsplit) { return 2 * (size_t)qsplit * a.B * a.Nk * a.H * a.d_head * sizeof(float); }
static bool dkv_ws_fits(const AttnArgs& a, int qsplit) { return qsplit <= 1 || (a.dkv_ws && a.dkv_ws_bytes >= dkv_partial_bytes(a, qsplit) && (uintptr_t)a.dkv_ws % 16 == 0); }
static void launch_dkv_reduce(const AttnArgs& a, int qsplit, hipStream_t s) {
  const size_t rows = (size_t)a.B * a.Nk; const int hd = a.H * a.d_head;
  KScope ks(KK_REDUCE, 0.0, (double)dkv_partial_bytes(a, qsplit) + 4.0 * rows * hd, s, (int)rows, hd, qsplit);
  hipLaunchKernelGGL(attn_dkv_reduce_kernel, dim3((rows * (hd / 4) + 255) / 256), dim3(256), 0, s, a.dkv_ws, qsplit, rows, hd,
                     (bf16*)a.dk, a.lddk, (bf16*)a.dv, a.lddv);
}

// Shares of the queries for the kernel that has all keys in a workgroup, `resident` of which run at a time: as many as run beside each other, of
// two tiles at least.
static int short_shares(const AttnArgs& a, int resident) {
  const long blocks = (long)a.B * a.H;
  const int nqt = (a.Nq + 63) / 64;
  return blocks >= 256 ? 1 : (int)std::max<long>(1, std::min<long>(std::min<long>(16, nqt / 2), (resident + blocks - 1) / blocks));
}
// Whether the backward runs as one kernel: all keys fit a workgroup, and the queries can be shared out or are few.  Without scratch for the
// shares' sums 8 x 5 heads of 4096 queries and 77 keys would walk 64 tiles on 40 CUs: 121 us, two kernels 97; 8 x 10 of 1024: 36 and 37.
static bool attn_short(const AttnArgs& a) { return a.Nk <= 256 && ((long)a.B * a.H >= 256 || a.Nq <= 24 * 64 || dkv_ws_fits(a, short_shares(a, 512))); }
template <int DHP, int KC, int NW>
static int launch_short(const AttnArgs& a, AttnK k, hipStream_t s) {
  auto kern = attn_bwd_short_bf16_kernel<DHP, KC, NW>;
  constexpr size_t BYTES = AttnShort<DHP, NW>::BYTES;
  static std::atomic<bool> attr_set{false};      // setting it twice is harmless; the flag only saves the call
  if (!attr_set.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)BYTES) != hipSuccess) return set_error(DP_EHIP, "hipFuncSetAttribute(attention) failed");
    attr_set.store(true, std::memory_order_release);
  }
  const long blocks = (long)a.B * a.H;
  const int nqt = (a.Nq + 63) / 64;
  int qsplit = short_shares(a, 256 * (BYTES <= 80 * 1024 ? 2 : 1));
  if (!dkv_ws_fits(a, qsplit)) qsplit = 1;
  const int tps = (nqt + qsplit - 1) / qsplit;
  qsplit = (nqt + tps - 1) / tps;
  k.qsplits = qsplit; k.dkv_partial = a.dkv_ws;
  {
    // algorithmic work of the whole backward, 2x the forward's
    KScope ks(KK_ATTN_BWD_DKV, 8.0 * a.B * a.H * (double)a.Nq * a.Nk * a.d_head, 2.0 * (double)a.B * a.H * a.d_head * (4.0 * a.Nq + 4.0 * a.Nk), s, a.Nq, a.Nk, a.d_head);
    hipLaunchKernelGGL(kern, dim3((unsigned)(blocks * qsplit)), dim3(NW * 64), BYTES, s, k);
  }
  if (qsplit > 1) launch_dkv_reduce(a, qsplit, s);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "attention backward launch failed");
}
static int launch_attn_bwd_short(const AttnArgs& a, const AttnK& k, hipStream_t s) {
  int rc = DP_OK;
  attn_dispatch(a.d_head, [&](auto dhp, auto kc) { rc = a.Nk <= 128 ? launch_short<dhp, kc, 4>(a, k, s) : launch_short<dhp, kc, 8>(a, k, s); });
  return rc;
}

// Whether a result of the fp32 backward lies in the place of something that it reads.  dQ over O, dK over K and dV over V are fine for the two kernels one after
// the other, each of which reads of those rows only what it replaces; side by side, one would overwrite what the other still reads.
static bool writes_over_inputs(const AttnArgs& a) {
  struct Span { uintptr_t first, end; };
  auto span = [&](const void* x, int n, int ld) { return Span{(uintptr_t)x, (uintptr_t)x + (((size_t)a.B * n - 1) * ld + (size_t)a.H * a.d_head) * sizeof(float)}; };
  const Span in[] = {span(a.q, a.Nq, a.ldq), span(a.k, a.Nk, a.ldk), span(a.v, a.Nk, a.ldv), span(a.o, a.Nq, a.ldo), span(a.dout, a.Nq, a.lddo)};
  const Span out[] = {span(a.dq, a.Nq, a.lddq), span(a.dk, a.Nk, a.lddk), span(a.dv, a.Nk, a.lddv)};
  for (const Span& i : in)
    for (const Span& o : out)
      if (i.first < o.end && o.first < i.end) return true;
  return false;
}

int launch_attn_bwd(const AttnArgs& a, hipStream_t s) {
  if (int e = check_attn(a, true)) return e;
  AttnK k = make_k(a);
  if (a.dtype == BF16 && attn_short(a)) return launch_attn_bwd_short(a, k, s);
  if (a.dtype == BF16) {
    k.even = takes_turns((long)((a.Nq + 127) / 128) * a.B * a.H, a.d_head <= 64 ? 3 : 2);
    dim3 gq(((a.Nq + 127) / 128) * a.B * a.H), gk(((a.Nk + 127) / 128) * a.B * a.H);
    // algorithmic backward work = 2x forward, split evenly between the two kernels for accounting
    const double fl = 4.0 * a.B * a.H * (double)a.Nq * a.Nk * a.d_head;
    const double by = 2.0 * (double)a.B * a.H * a.d_head * (3.0 * a.Nq + 2.0 * a.Nk);
    {
      KScope ks(KK_ATTN_BWD_DQ, fl, by, s, a.Nq, a.Nk, a.d_head);
      attn_dispatch(a.d_head, [&](auto dhp, auto kc) { hipLaunchKernelGGL((attn_bwd_dq_bf16_kernel<dhp, kc>), gq, dim3(256), 0, s, k); });
    }
    {
      // few key tiles (cross-attention to 77 keys): split the query range over more workgroups
      AttnK k2 = k;
      const long base_blocks = (long)((a.Nk + 127) / 128) * a.B * a.H;
      const int nqt = (a.Nq + 63) / 64;
      int qsplit = 1;
      if (base_blocks < 256) qsplit = (int)std::min<long>(std::min<long>(16, nqt / 2 > 0 ? nqt / 2 : 1), (512 + base_blocks - 1) / base_blocks);
      if (!dkv_ws_fits(a, qsplit)) qsplit = 1;
      k2.even = takes_turns((long)gk.x * qsplit, a.d_head <= 64 && qsplit == 1 && gk.x > 2 * 256 ? 3 : 2);
      k2.qsplits = qsplit; k2.dkv_partial = a.dkv_ws;
      dim3 gk2(gk.x * qsplit);
      {
        KScope ks(KK_ATTN_BWD_DKV, fl, by, s, a.Nq, a.Nk, a.d_head);
        // Two workgroups per CU hold 512 at a time; a larger grid gains more from a third than the tighter register budget costs (80
        // heads of 1024 tokens, 640 workgroups: 69 -> 53 us), a smaller one only pays for it (77 keys, 1024 queries: 24 -> 31 us)
        attn_dispatch(a.d_head, [&](auto dhp, auto kc) {
          if (dhp == 64 && qsplit == 1 && gk.x > 2 * 256) hipLaunchKernelGGL((attn_bwd_dkv_bf16_kernel<dhp, kc, dhp == 64 ? 3 : 2>), gk2, dim3(256), 0, s, k2);
          else hipLaunchKernelGGL((attn_bwd_dkv_bf16_kernel<dhp, kc, 2>), gk2, dim3(256), 0, s, k2);
        });
      }
      if (qsplit > 1) launch_dkv_reduce(a, qsplit, s);
    }
  } else {
    // One launch where the dK/dV workgroups are at most two per CU and their loops short: forming delta costs each of them half as many loads again.  B x H, queries x
    // keys, width: 2 x 4, 64 x 64, 16 12.0 -> 9.8 us; 2 x 2, 128 x 128, 16 15.6 -> 12.1; 4 x 5, 256 x 16, 32 24.4 -> 23.5; beyond the lines 4 x 4, 200 x 77, 24 44.6 -> 50.9;
    // 1 x 1, 1024 x 1024, 64 173 -> 204.  Step of a U-Net block 2 x 64 x 64: 119 -> 112.5 us.
    if ((long)a.Nk * a.B * a.H <= 512 && a.Nq <= 256 && !writes_over_inputs(a)) {
      hipLaunchKernelGGL(attn_bwd_both_f32_kernel, dim3(a.Nk + a.Nq, a.B * a.H), dim3(64), std::max((size_t)a.Nk, (size_t)2 * a.Nq) * sizeof(float), s, k);
      return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "attention backward launch failed");
    }
    hipLaunchKernelGGL(attn_bwd_dq_f32_kernel, dim3(a.Nq, a.B * a.H), dim3(64), (size_t)a.Nk * sizeof(float), s, k);
    hipLaunchKernelGGL(attn_bwd_dkv_f32_kernel, dim3(a.Nk, a.B * a.H), dim3(64), (size_t)2 * a.Nq * sizeof(float), s, k);
  }
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "attention backward launch failed");
}

}  // namespace dp
