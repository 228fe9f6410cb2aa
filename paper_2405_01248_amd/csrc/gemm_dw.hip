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
  int run_first, run;                // the run of problems of equally long workgroups that it is part of: first workgroup and number of them
  int splits, kt_per_split;
  int accumulate;
};
struct DwGroup { DwProblem p[DW_GROUP_MAX]; int n, total; };

// What bounds it: instruction issue and LDS beside the matrix work, and the latency of the operands.  Without its copies the launch of a U-Net block
// 8 x 1024 x 640 takes 118 us of what was 143, without its matrix work 139, with every copy an L2 hit 130.  Two things bring the latter about, 143 -> 130 us by itself, 134
// inside a step (a block of 8 x 4096 x 320 181 -> 170; a DiT block of 32 x 256 x 1152 is not faster, its 4 x 256 one 1 %):
// - an XCD's workgroups are tiles of one region of one problem, or of two, whatever the problems' number: 434 MB read past the L2s for 254 MB of operands
//   where a share of every problem to every XCD read 862;
// - tiles that share operands run in step, so that each k-tile would come from memory for all of them at once.  Every other tile takes its k-tiles in
//   pairs turned round: while half of the tiles have the first of a pair fetched, the other half has the second, and both find the other one in the L2.
//   Windows of four and eight k-tiles gave 131 and 130 us.
template <class T>
__global__ void __launch_bounds__(512, 2) gemm_dw_group_kernel(const DwGroup grp) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / T::WGN, wn = wave % T::WGN;
  // The hardware deals workgroups round-robin to the 8 XCDs.  Over a run of problems of equally long workgroups every XCD takes a contiguous
  // range of (problem, split, tile), so that its tiles share operand panels in its L2 and the XCDs' queues are equally long.
  auto problem_of = [&](int id) {
    int q = 0;
    while (q + 1 < grp.n && id >= grp.p[q + 1].first) ++q;
    return q;
  };
  const int q0 = problem_of(blockIdx.x), place = grp.p[q0].run_first + xcd_contiguous_id(blockIdx.x - grp.p[q0].run_first, grp.p[q0].run), q = problem_of(place);
  const DwProblem& p = grp.p[q];
  const int tiles = p.tiles_m * p.tiles_n, id = place - p.first, split = id / tiles;
  int tile_m, tile_n;
  tile_of_id(id % tiles, p.tiles_m, p.tiles_n, p.group_m, tile_m, tile_n);
  const int m0 = tile_m * T::BM, n0 = tile_n * T::BN, M = p.M, N = p.N, lda = p.lda, ldb = p.ldb;
  const int kt0 = split * p.kt_per_split, kt_all = (p.K + 63) / 64, nk = min(kt_all, kt0 + p.kt_per_split) - kt0;
  const uint32_t k_end = (uint32_t)(kt0 + nk) * 128u;      // twice the contraction row behind this split's last one
  const rsrc_t ra = make_rsrc(p.A, min(p.a_bytes, k_end * (uint32_t)lda)), rb = make_rsrc(p.B, min(p.b_bytes, k_end * (uint32_t)ldb));
  const uint32_t step_a = 128u * (uint32_t)lda, step_b = 128u * (uint32_t)ldb;
  // Columns past the edge are fetched from the last valid chunk (they only feed outputs that are never stored); rows past the end of the contraction, in its last k-tile,
  // lie outside the buffers and arrive as zeros.  The lanes' offsets take the steps along the contraction: one addition a copy, where a copy with the step in a scalar and
  // the last k-tile's rows picked out took four vector instructions.  The loop also copies the two k-tiles behind the last one, rows up to K + 190: their offsets
  // may go past 4 GiB and come round to rows that are there (the buffer's size keeps every read inside it), and nothing multiplies what they bring.
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
  const bool do_colsum = p.colsum != nullptr && tile_n == 0 && wn == 0;
  typename T::acc_t acc[2][T::TM][T::TN];
  float csum[2][T::TM];
  const uint32_t turn = (uint32_t)(tile_m + tile_n) & 1u, pairs = (uint32_t)nk & ~1u;      // (an odd last k-tile stays)
  auto k_of = [&](int t) { return (uint32_t)t < pairs ? (uint32_t)t ^ turn : (uint32_t)t; };
  pp_main_loop<T, false, true>(acc, smem_raw, nk, wm, wn, wave >= 4, lane,
      [&](auto hc, int t, unsigned char* dst) {
        constexpr int h = decltype(hc)::value;
#pragma unroll
        for (int j = 0; j < T::LA; ++j) async_copy_16B_buf(ra, va[h][j] + k_of(t) * step_a, 0, dst + (wave * T::LA + j) * 1024);
      },
      [&](auto hc, int t, unsigned char* dst) {
        constexpr int h = decltype(hc)::value, L = h ? T::LB1 : T::LB0;
#pragma unroll
        for (int j = 0; j < L; ++j) async_copy_16B_buf(rb, (h ? vb1[h ? j : 0] : vb0[h ? 0 : j]) + k_of(t) * step_b, 0, dst + (wave * L + j) * 1024);
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
  pp_epilogue<T, PE_F32>(acc, smem_raw, e, m0, n0, wave, wm, wn, lane, []() {});
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
// us: time of a k-tile with the chip full.  Over 33 blocks (U-Net of 256 to 1280 columns and 1026 to 32768 rows, DiT of 384 to 1152 and 300 to 12288), each plan within a quarter of
// the least estimate timed, the one that is chosen takes 0.9 % more than the fastest on average and 7 % at most; with 1.63, 1.06, 1.06 and 1.33, the times before the copies lost
// their overhead, 2.2 and 19 % (us: DiT 8192 x 768 126 -> 120, 12288 x 384 64.5 -> 60.6, 3000 x 432 37.9 -> 34.9; U-Net 8192 x 400 82.7 -> 76.8, 4096 x 256 32.5 -> 27.4; the
// one that loses, DiT 10000 x 648, 135.6 -> 137.0).  The reduction at 5 TB/s and 6 us and the 5 us of a tile (dw_plan_us) are within 0.1 % of the best values there.
struct DwTile { int bm, bn; float us; };
static const DwTile kDwTiles[] = {{256, 256, 1.53f}, {256, 128, 0.86f}, {128, 256, 0.86f}, {256, 192, 1.21f}};
constexpr int kDwTileCount = 4;

// A problem, or a range of output rows of one, as it is launched.
struct DwPart { int problem, row0, rows, splits, kt_per_split; };

static int dw_tiles(const GemmArgs& a, const DwTile& t) { return ((a.M + t.bm - 1) / t.bm) * ((a.N + t.bn - 1) / t.bn); }

// The parts of a plan in launch order: the problems with long contractions, their first `whole` tiles unsplit (to whole tile-rows)
// and the rest split along the contraction; then the ones with short contractions, unsplit.  At most n + 1 of them.
static int dw_parts(const GemmArgs* a, int n, const DwGroupPlan& plan, DwPart* out) {
  const DwTile& t = kDwTiles[plan.tile];
  int kt_max = 0, cnt = 0, left = plan.whole;
  for (int i = 0; i < n; ++i) kt_max = std::max(kt_max, (a[i].K + 63) / 64);
  auto add = [&](int i, int row0, int rows, int splits) {
    const int kt = (a[i].K + 63) / 64, per = (kt + splits - 1) / splits;
    if (rows > 0) out[cnt++] = {i, row0, rows, (kt + per - 1) / per, per};
  };
  for (int i = 0; i < n; ++i) {
    if ((a[i].K + 63) / 64 * 2 < kt_max) continue;
    const int tn = (a[i].N + t.bn - 1) / t.bn, tm = (a[i].M + t.bm - 1) / t.bm, rows = std::min(a[i].M, std::min(tm, left / tn) * t.bm);
    if (rows < a[i].M && left > 0) left = 0; else left -= std::min(left, tm * tn);
    add(i, 0, rows, 1);
    add(i, rows, a[i].M - rows, plan.splits);
  }
  for (int i = 0; i < n; ++i)
    if ((a[i].K + 63) / 64 * 2 < kt_max) add(i, 0, a[i].M, 1);
  return cnt;
}
// Rows of tiles that the order of a problem's tiles walks down before it goes to the next column: as many as make the 32 tiles in a row that an XCD
// works on together nearly square, in groups of equal height.
static int dw_group_rows(int tiles_m) {
  const int groups = std::max(1, (tiles_m + 2) / 5);
  return (tiles_m + groups - 1) / groups;
}
static size_t dw_part_ws_bytes(const GemmArgs& a, const DwPart& d) {
  return d.splits > 1 ? ((size_t)d.splits * ((size_t)d.rows * a.N + d.rows) * sizeof(float) + 255) / 256 * 256 : 0;
}

// Estimated time: on each XCD its eighth of the workgroups, in launch order, on 32 CUs, each taking the one that is free first
// (kept as groups of CUs that are free at the same time); then the traffic of the partial sums.
static double dw_plan_us(const GemmArgs* a, const DwGroupPlan& plan, const DwPart* d, int n) {
  const DwTile& t = kDwTiles[plan.tile];
  struct Slots { double at; int count; } q[33];
  int nq = 1;
  q[0] = {0.0, 32};
  double bytes = 0, us = 0;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& g = a[d[i].problem];
    int jobs = (((d[i].rows + t.bm - 1) / t.bm) * ((g.N + t.bn - 1) / t.bn) * d[i].splits + 7) / 8;
    const double dur = d[i].kt_per_split * t.us + 5.0;
    while (jobs > 0) {
      int e = 0;
      for (int k = 1; k < nq; ++k) if (q[k].at < q[e].at) e = k;
      if (jobs >= q[e].count) { jobs -= q[e].count; q[e].at += dur; }
      else { q[nq++] = {q[e].at + dur, jobs}; q[e].count -= jobs; jobs = 0; }
      for (int k = 0; k < nq; ++k)           // groups that became free at the same time are one
        for (int m = nq - 1; m > k; --m)
          if (q[m].at == q[k].at) { q[k].count += q[m].count; q[m] = q[--nq]; }
    }
    if (d[i].splits > 1) bytes += 2.0 * d[i].splits * 4.0 * d[i].rows * g.N;
  }
  for (int k = 0; k < nq; ++k) us = std::max(us, q[k].at);
  return us + bytes / 5.0e6 + (bytes > 0 ? 6.0 : 0.0);
}

// Tile, number of unsplit tiles and split of the rest with the least estimated time.  Whole rounds of 256 workgroups run
// unsplit; what is left over, which would leave most CUs idle for the length of a whole contraction, is cut to fill the chip.
DwGroupPlan gemm_dw_group_plan(const GemmArgs* a, int n, int force_tile, size_t ws_limit) {
  DwGroupPlan best{-1, 0, 1, 0};
  double best_us = 0;
  int kt_max = 0;
  for (int i = 0; i < n; ++i) kt_max = std::max(kt_max, (a[i].K + 63) / 64);
  for (int tile = 0; tile < kDwTileCount; ++tile) {
    if (force_tile && tile != force_tile - 1) continue;
    int total = 0;
    for (int i = 0; i < n; ++i) if ((a[i].K + 63) / 64 * 2 >= kt_max) total += dw_tiles(a[i], kDwTiles[tile]);
    for (int rounds = 0; rounds <= total / 256; ++rounds) {
      if (rounds > 2 && rounds < total / 256 - 1) continue;
      for (int s = 1; s <= 64 && (s == 1 || (kt_max + s - 1) / s >= 4); s += 1 + s / 8) {
        const DwGroupPlan plan{tile, 256 * rounds, s, 0};
        DwPart parts[2 * DW_GROUP_MAX];
        const int np = dw_parts(a, n, plan, parts);
        size_t ws = 0;
        for (int i = 0; i < np; ++i) ws += dw_part_ws_bytes(a[parts[i].problem], parts[i]);
        if (ws > ws_limit) continue;
        const double us = dw_plan_us(a, plan, parts, np);
        if (best.tile < 0 || us < best_us) { best = plan; best.ws_bytes = ws; best_us = us; }
        if (rounds == 0 && s == 1 && total >= 256 * 8) break;       // many rounds: nothing to gain from a split
      }
    }
  }
  return best;
}

bool gemm_dw_group_supported(const GemmArgs& a) {
  if (a.dtype != BF16 || !a.a_mc || !a.b_mc || !a.out_f32 || a.ldo32 != a.N) return false;
  if (a.M % 8 || a.N % 8 || a.lda % 8 || a.ldb % 8 || a.M < 8 || a.N < 8 || a.K < 1 || a.lda < a.M || a.ldb < a.N) return false;
  if ((uintptr_t)a.A % 16 || (uintptr_t)a.B % 16 || (uintptr_t)a.out_f32 % 16 || (uintptr_t)a.colsum_out % 16) return false;
  // 32-bit offsets of the rows that reach registers: the last k-tile's and, unused, the one's behind it
  return operand_extent_bytes(a.K + 128, a.M, a.lda) < 0xFFFFFFF0ull && operand_extent_bytes(a.K + 128, a.N, a.ldb) < 0xFFFFFFF0ull;
}

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

int launch_gemm_dw_group(const GemmArgs* a, int n, const DwGroupPlan& plan, hipStream_t s) {
  if (n < 1 || n >= DW_GROUP_MAX) return set_error(DP_EINVAL, "gemm dW: bad number of problems");
  for (int i = 0; i < n; ++i)
    if (!gemm_dw_group_supported(a[i])) return set_error(DP_EUNSUPPORTED, "gemm dW: problem not supported");
  if (plan.tile < 0 || plan.tile >= kDwTileCount) return set_error(DP_EUNSUPPORTED, "gemm dW: bad tile");
  if (plan.ws_bytes && (!a[0].splitk_ws || a[0].splitk_ws_bytes < plan.ws_bytes)) return set_error(DP_EWORKSPACE, "gemm dW: split-K workspace too small");
  const DwTile& t = kDwTiles[plan.tile];
  static_assert(sizeof(DwGroup) <= 4096 && sizeof(DwReduce) <= 4096, "kernel arguments");
  DwPart parts[2 * DW_GROUP_MAX];
  const int np = dw_parts(a, n, plan, parts);
  DwGroup g;
  DwReduce r;
  g.n = np; g.total = 0; r.n = 0; r.first[0] = 0;
  char* ws = (char*)a[0].splitk_ws;
  double flops = 0, bytes = 0, red = 0;
  for (int i = 0; i < np; ++i) {
    const GemmArgs& b = a[parts[i].problem];
    const int row0 = parts[i].row0;
    DwProblem& p = g.p[i];
    p.A = (const bf16*)b.A + row0; p.B = (const bf16*)b.B; p.out = b.out_f32 + (size_t)row0 * b.N;
    p.colsum = b.colsum_out ? b.colsum_out + row0 : nullptr; p.partial = nullptr;
    p.M = parts[i].rows; p.N = b.N; p.K = b.K; p.lda = b.lda; p.ldb = b.ldb; p.accumulate = b.accumulate;
    p.a_bytes = (uint32_t)operand_extent_bytes(b.K, p.M, b.lda);
    p.b_bytes = (uint32_t)operand_extent_bytes(b.K, b.N, b.ldb);
    p.tiles_m = (p.M + t.bm - 1) / t.bm; p.tiles_n = (p.N + t.bn - 1) / t.bn;
    p.group_m = dw_group_rows(p.tiles_m);
    p.splits = parts[i].splits; p.kt_per_split = parts[i].kt_per_split;
    p.first = g.total;
    g.total += p.tiles_m * p.tiles_n * p.splits;
    const size_t mn = (size_t)p.M * p.N;
    if (p.splits > 1) {
      p.partial = (float*)ws;
      ws += dw_part_ws_bytes(b, parts[i]);
      auto add = [&](float* out, const float* part, size_t count) {
        r.p[r.n] = {out, part, (long)(count / 4), p.splits, p.accumulate};
        r.first[r.n + 1] = r.first[r.n] + (long)(count / 4);
        ++r.n;
      };
      add(p.out, p.partial, mn);
      if (p.colsum) add(p.colsum, p.partial + (size_t)p.splits * mn, p.M);
      red += 4.0 * (p.splits + 1.0) * mn;
    }
    // a run: neighbours in launch order that differ in the length of their workgroups by less than one k-tile in eight
    const bool same = i && 8 * std::abs(p.kt_per_split - g.p[i - 1].kt_per_split) < p.kt_per_split;
    p.run_first = same ? g.p[i - 1].run_first : p.first;
    for (int j = 0; j <= i; ++j)
      if (g.p[j].run_first == p.run_first) g.p[j].run = g.total - p.run_first;
    flops += 2.0 * mn * p.K; bytes += 2.0 * p.K * ((double)p.M + p.N) + 4.0 * mn * (p.accumulate ? 2.0 : 1.0);
  }
  {
    KScope ks(KK_GEMM_TN, flops, bytes, s, g.p[0].M, g.p[0].N, g.p[0].K);
    int rc = DP_OK;
    switch (plan.tile) {
      case 0: rc = launch_dw_tile<PpTile<256, 128, 128, 4, 2>>(g, s); break;
      case 1: rc = launch_dw_tile<PpTile<256, 64, 64, 4, 2>>(g, s); break;
      case 3: rc = launch_dw_tile<PpTile<256, 128, 64, 4, 2>>(g, s); break;
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
