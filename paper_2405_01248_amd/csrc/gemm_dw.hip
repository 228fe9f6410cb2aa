// Weight gradients dW = dy^T x of several projections in one launch (bf16 operands, fp32 output).
//
// One weight gradient of a U-Net stage has few output tiles and a long contraction (640 x 640 over 8192 rows: 25 tiles of
// 128 x 128), so on its own it has to be cut along the contraction many times to fill the chip, and the fp32 partial sums
// cost more traffic than the operands.  The gradients of a whole block together have enough tiles: one launch over all
// of them needs no split, or a small one.
#include "dp_device.h"
#include "dp_kernels.h"
#include "dp_errors.h"
#include "dp_host.h"
#include "dp_ktime.h"
#include "dp_gemm_pp.h"

#include <algorithm>
#include <atomic>
#include <cstring>

namespace dp {

struct DwProblem {
  const bf16* A; const bf16* B;      // dy [K, M], x [K, N]
  float* out; float* colsum;         // [M, N]; [M] or nullptr: sum of A over the contraction
  float* partial;                    // splits > 1: [splits][M][N], then [splits][M] column sums
  int M, N, K, lda, ldb;
  uint32_t a_bytes, b_bytes;
  int tiles_m, tiles_n, group_m;
  int first;                         // first workgroup of the problem
  int splits, kt_per_split;
  int accumulate;
};
struct DwGroup { DwProblem p[DW_GROUP_MAX]; int n, total; };

// What bounds it: the transposing LDS reads (about 75 B per clock and CU against 128 or more of the plain ones), which keep the
// matrix pipe at two thirds with 256x256 tiles; hence the tile with the least fragment bytes per FLOP wherever the
// outputs are large enough.
template <class T>
__global__ void __launch_bounds__(512, 2) gemm_dw_group_kernel(const DwGroup grp) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / T::WGN, wn = wave % T::WGN;
  // every XCD takes a contiguous range of (problem, split, tile): neighbours share operand panels in its L2
  const int id0 = xcd_contiguous_id(blockIdx.x, grp.total);
  int q = 0;
  while (q + 1 < grp.n && id0 >= grp.p[q + 1].first) ++q;
  const DwProblem& p = grp.p[q];
  const int tiles = p.tiles_m * p.tiles_n, split = (id0 - p.first) / tiles;
  int tile_m, tile_n;
  tile_of_id((id0 - p.first) % tiles, p.tiles_m, p.tiles_n, p.group_m, tile_m, tile_n);
  const int m0 = tile_m * T::BM, n0 = tile_n * T::BN, M = p.M, N = p.N, K = p.K, lda = p.lda, ldb = p.ldb;
  const int kt0 = split * p.kt_per_split, kt_all = (K + 63) / 64, nk = min(kt_all, kt0 + p.kt_per_split) - kt0;
  const int k_end = K - kt0 * 64;                       // contraction rows from this split's first one on
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;
  const bf16* A = p.A; const bf16* B = p.B;
  const uint32_t a_bytes = p.a_bytes, b_bytes = p.b_bytes;
  // columns past the edge are fetched from the last valid chunk (they only feed outputs that are never stored), rows past the
  // end of the contraction from outside the buffers (zeros)
  uint32_t va[2][T::LA], vb0[T::LB0], vb1[T::LB1];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < T::LA; ++j) {
      const int k = pp_mc_piece_k<T::BM / 2>(wave * T::LA + j, lane), c = pp_mc_piece_chunk<T::BM / 2>(k, lane);
      va[h][j] = 2u * ((uint32_t)(kt0 * 64 + k) * lda + min(m0 + h * (T::BM / 2) + c * 8, M - 8));
    }
#pragma unroll
  for (int j = 0; j < T::LB0; ++j) {
    const int k = pp_mc_piece_k<T::BN0>(wave * T::LB0 + j, lane), c = pp_mc_piece_chunk<T::BN0>(k, lane);
    vb0[j] = 2u * ((uint32_t)(kt0 * 64 + k) * ldb + min(n0 + c * 8, N - 8));
  }
#pragma unroll
  for (int j = 0; j < T::LB1; ++j) {
    const int k = pp_mc_piece_k<T::BN1>(wave * T::LB1 + j, lane), c = pp_mc_piece_chunk<T::BN1>(k, lane);
    vb1[j] = 2u * ((uint32_t)(kt0 * 64 + k) * ldb + min(n0 + T::BN0 + c * 8, N - 8));
  }
  const bool ragged = k_end < nk * 64;
  auto tail = [&](uint32_t v, int k, int t) { return ragged && t == nk - 1 && t * 64 + k >= k_end ? OUTSIDE : v; };
  const bool do_colsum = p.colsum != nullptr && tile_n == 0 && wn == 0;
  typename T::acc_t acc[2][T::TM][T::TN];
  float csum[2][T::TM];
  pp_main_loop<T, false, true>(acc, smem_raw, nk, wm, wn, wave >= 4, lane,
      [&](int h, int t, unsigned char* dst) {
        const rsrc_t r = make_rsrc(A, t < nk ? a_bytes : 0u);
        const uint32_t off = t < nk ? (uint32_t)t * 128u * (uint32_t)lda : 0u;
#pragma unroll
        for (int j = 0; j < T::LA; ++j)
          async_copy_16B_buf(r, tail(va[h][j], pp_mc_piece_k<T::BM / 2>(wave * T::LA + j, lane), t), off, dst + (wave * T::LA + j) * 1024);
      },
      [&](auto hc, int t, unsigned char* dst) {
        constexpr int h = decltype(hc)::value, L = h ? T::LB1 : T::LB0, COLS = h ? T::BN1 : T::BN0;
        const rsrc_t r = make_rsrc(B, t < nk ? b_bytes : 0u);
        const uint32_t off = t < nk ? (uint32_t)t * 128u * (uint32_t)ldb : 0u;
#pragma unroll
        for (int j = 0; j < L; ++j)
          async_copy_16B_buf(r, tail(h ? vb1[h ? j : 0] : vb0[h ? 0 : j], pp_mc_piece_k<COLS>(wave * L + j, lane), t), off, dst + (wave * L + j) * 1024);
      }, do_colsum, csum);
  const DwProblem& e0 = grp.p[q];
  if (do_colsum) {
    float* cs = e0.splits > 1 ? e0.partial + (size_t)e0.splits * M * N + (size_t)split * M : e0.colsum;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < T::TM; ++i) {
        const float s = csum[h][i] + __shfl_xor(csum[h][i], 32, 64);
        const int m = m0 + h * (T::BM / 2) + wm * T::SM + i * 32 + lane;
        if (lane < 32 && m < M) cs[m] = e0.accumulate && e0.splits == 1 ? cs[m] + s : s;
      }
  }
  EpiParams<bf16> e{};
  e.M = M; e.N = N; e.out32 = e0.out; e.ldo32 = N; e.accumulate = e0.accumulate;
  e.partial = e0.splits > 1 ? e0.partial + (size_t)split * M * N : nullptr;
  pp_epilogue<T, PE_F32>(acc, smem_raw, e, m0, n0, wave, wm, wn, lane);
}

// out (+)= sum of the partial planes in ascending order, for every split problem of the group and its column sums.
struct DwReduce {
  struct { float* out; const float* partial; long n4; int planes, accumulate; } p[2 * DW_GROUP_MAX];
  long first[2 * DW_GROUP_MAX + 1];      // first group of 4 values of each entry
  int n;
};
__global__ void __launch_bounds__(256) gemm_dw_reduce_kernel(const DwReduce r) {
  const long id = (long)blockIdx.x * 256 + threadIdx.x;
  if (id >= r.first[r.n]) return;
  int q = 0;
  while (id >= r.first[q + 1]) ++q;
  const long i = (id - r.first[q]) * 4, plane = r.p[q].n4 * 4;
  const float* src = r.p[q].partial + i;
  const int planes = r.p[q].planes;
  f32x4 v = *reinterpret_cast<const f32x4*>(src);
  for (int z = 1; z < planes; ++z) v += *reinterpret_cast<const f32x4*>(src + z * plane);
  float* o = r.p[q].out + i;
  if (r.p[q].accumulate) v += *reinterpret_cast<const f32x4*>(o);
  *reinterpret_cast<f32x4*>(o) = v;
}

// ------------------------------------------------------------------ host side
struct DwTile { int bm, bn; float us; };        // us: time of a k-tile with the chip full
static const DwTile kDwTiles[] = {{256, 256, 1.5f}, {256, 128, 0.85f}, {128, 256, 0.85f}};
constexpr int kDwTileCount = 3;

struct DwPlan { int tile, kt_per_wg; size_t ws_bytes; };

static size_t dw_plan_eval(const GemmArgs* a, int n, int tile, int L, double& us) {
  const DwTile& t = kDwTiles[tile];
  long wgs = 0;
  double bytes = 0;
  size_t ws = 0;
  int longest = 0;
  for (int i = 0; i < n; ++i) {
    const long tiles = (long)((a[i].M + t.bm - 1) / t.bm) * ((a[i].N + t.bn - 1) / t.bn);
    const int kt = (a[i].K + 63) / 64, splits = (kt + L - 1) / L;
    wgs += tiles * splits;
    longest = std::max(longest, (kt + splits - 1) / splits);
    if (splits > 1) {
      ws += ((size_t)splits * ((size_t)a[i].M * a[i].N + a[i].M) * sizeof(float) + 255) / 256 * 256;
      bytes += 2.0 * splits * 4.0 * a[i].M * a[i].N;
    }
  }
  const double per_wg = longest * t.us + 4.0;
  us = (double)((wgs + 255) / 256) * per_wg + bytes / 4.0e6 + (ws ? 4.0 : 0.0);
  return ws;
}

// Tile and split: the pair with the least estimated time, (rounds of 256 workgroups) x (k-tiles per workgroup x time of a
// k-tile + prologue and epilogue) + the partial sums' traffic.
static DwPlan dw_plan(const GemmArgs* a, int n, int force_tile, size_t ws_limit) {
  int kt_max = 0;
  for (int i = 0; i < n; ++i) kt_max = std::max(kt_max, (a[i].K + 63) / 64);
  DwPlan best{-1, 0, 0};
  double best_us = 0;
  for (int tile = 0; tile < kDwTileCount; ++tile) {
    if (force_tile && tile != force_tile - 1) continue;
    for (int s = 1; s <= 64 && s <= kt_max; ++s) {
      const int L = (kt_max + s - 1) / s;
      if (s > 1 && L < 4) break;
      double us;
      const size_t ws = dw_plan_eval(a, n, tile, L, us);
      if (ws > ws_limit) continue;
      if (best.tile < 0 || us < best_us) { best = {tile, L, ws}; best_us = us; }
    }
  }
  return best;
}

bool gemm_dw_group_supported(const GemmArgs& a) {
  if (a.dtype != BF16 || !a.a_mc || !a.b_mc || !a.out_f32 || a.ldo32 != a.N) return false;
  if (a.M % 8 || a.N % 8 || a.lda % 8 || a.ldb % 8 || a.M < 8 || a.N < 8 || a.K < 1 || a.lda < a.M || a.ldb < a.N) return false;
  if ((uintptr_t)a.A % 16 || (uintptr_t)a.B % 16 || (uintptr_t)a.out_f32 % 16 || (uintptr_t)a.colsum_out % 16) return false;
  // 32-bit offsets, also of the k-tile past the last one
  return operand_extent_bytes(a.K + 128, a.M, a.lda) < 0xFFFFFFF0ull && operand_extent_bytes(a.K + 128, a.N, a.ldb) < 0xFFFFFFF0ull;
}

size_t gemm_dw_group_ws_bytes(const GemmArgs* a, int n) { return dw_plan(a, n, 0, (size_t)-1).ws_bytes; }

template <class T>
static int launch_dw_tile(DwGroup& g, hipStream_t s) {
  auto kern = gemm_dw_group_kernel<T>;
  static std::atomic<bool> attr_set{false};   // setting it twice is harmless; the flag only saves the call
  if (!attr_set.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::BYTES) != hipSuccess)
      return set_error(DP_EHIP, "hipFuncSetAttribute(gemm dW) failed");
    attr_set.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(kern, dim3(g.total), dim3(512), T::BYTES, s, g);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm dW launch failed");
}

int launch_gemm_dw_group(const GemmArgs* a, int n, int force_tile, hipStream_t s) {
  if (n < 1 || n > DW_GROUP_MAX) return set_error(DP_EINVAL, "gemm dW: bad number of problems");
  for (int i = 0; i < n; ++i)
    if (!gemm_dw_group_supported(a[i])) return set_error(DP_EUNSUPPORTED, "gemm dW: problem not supported");
  const DwPlan plan = dw_plan(a, n, force_tile, a[0].splitk_ws ? a[0].splitk_ws_bytes : 0);
  if (plan.tile < 0) return set_error(DP_EUNSUPPORTED, "gemm dW: bad tile");
  const DwTile& t = kDwTiles[plan.tile];
  DwGroup g;
  DwReduce r;
  g.n = n; g.total = 0; r.n = 0; r.first[0] = 0;
  char* ws = (char*)a[0].splitk_ws;
  double flops = 0, bytes = 0, red = 0;
  for (int i = 0; i < n; ++i) {
    DwProblem& p = g.p[i];
    p.A = (const bf16*)a[i].A; p.B = (const bf16*)a[i].B; p.out = a[i].out_f32; p.colsum = a[i].colsum_out; p.partial = nullptr;
    p.M = a[i].M; p.N = a[i].N; p.K = a[i].K; p.lda = a[i].lda; p.ldb = a[i].ldb; p.accumulate = a[i].accumulate;
    p.a_bytes = (uint32_t)operand_extent_bytes(a[i].K, a[i].M, a[i].lda);
    p.b_bytes = (uint32_t)operand_extent_bytes(a[i].K, a[i].N, a[i].ldb);
    p.tiles_m = (p.M + t.bm - 1) / t.bm; p.tiles_n = (p.N + t.bn - 1) / t.bn;
    p.group_m = std::min(p.tiles_m, 8);
    const int kt = (p.K + 63) / 64;
    p.splits = (kt + plan.kt_per_wg - 1) / plan.kt_per_wg;
    p.kt_per_split = (kt + p.splits - 1) / p.splits;
    p.splits = (kt + p.kt_per_split - 1) / p.kt_per_split;
    p.first = g.total;
    g.total += p.tiles_m * p.tiles_n * p.splits;
    const size_t mn = (size_t)p.M * p.N;
    if (p.splits > 1) {
      p.partial = (float*)ws;
      ws += ((size_t)p.splits * (mn + p.M) * sizeof(float) + 255) / 256 * 256;
      auto add = [&](float* out, const float* part, size_t count) {
        r.p[r.n] = {out, part, (long)(count / 4), p.splits, p.accumulate};
        r.first[r.n + 1] = r.first[r.n] + (long)(count / 4);
        ++r.n;
      };
      add(p.out, p.partial, mn);
      if (p.colsum) add(p.colsum, p.partial + (size_t)p.splits * mn, p.M);
      red += 4.0 * (p.splits + 1.0) * mn;
    }
    flops += 2.0 * mn * p.K; bytes += 2.0 * p.K * ((double)p.M + p.N) + 4.0 * mn * (p.accumulate ? 2.0 : 1.0);
  }
  {
    KScope ks(KK_GEMM_TN, flops, bytes, s, g.p[0].M, g.p[0].N, g.p[0].K);
    int rc = DP_OK;
    switch (plan.tile) {
      case 0: rc = launch_dw_tile<PpTile<256, 128, 128, 4, 2>>(g, s); break;
      case 1: rc = launch_dw_tile<PpTile<256, 64, 64, 4, 2>>(g, s); break;
      default: rc = launch_dw_tile<PpTile<128, 128, 128, 2, 4>>(g, s); break;
    }
    DP_TRY(rc);
  }
  if (r.n) {
    KScope ks(KK_REDUCE, 0.0, red, s, g.p[0].M, g.p[0].N, r.n);
    hipLaunchKernelGGL(gemm_dw_reduce_kernel, dim3((unsigned)((r.first[r.n] + 255) / 256)), dim3(256), 0, s, r);
    if (hipGetLastError() != hipSuccess) return set_error(DP_EHIP, "gemm dW reduction launch failed");
  }
  return DP_OK;
}

}  // namespace dp
