// fp32 GEMM (every operand layout) for the fp32 stages: small problems, so what counts is the time of one dependent launch.
//
// A workgroup owns a 32 x 32 tile of the output; its waves share the contraction in chunks of 16 and fetch their fragments straight
// from global memory, several chunks in flight, for v_mfma_f32_16x16x4_f32 (full fp32 products and sums); the waves' partial tiles
// are added through LDS in ascending order.  Against a tile walked 16 contraction steps at a time through LDS by all waves, each step two
// barriers and a memory round trip deep: 128 x 64 x 64 13 -> 5 us, 64 x 256 x 128 (a weight gradient) 24 -> 5 us.
#include "dp_kernels.h"
#include "dp_errors.h"
#include "dp_host.h"
#include "dp_ktime.h"
#include "dp_gemm_epilogue.h"

#include <algorithm>

namespace dp {

struct GemmF32Params {
  const float* A; const float* B;
  int M, N, K, lda, ldb;
  int fold_m;                         // more tiles than a grid's first two dimensions take: the third counts row folds, then column folds
  float* colsum; int colsum_acc;      // A contraction-strided: sum of A over the contraction, per row of the output
  EpiParams<float> epi;
};

// problems of a grouped launch, and the tiles from which a problem fills the chip several times over by itself
constexpr int GEMM_F32_GROUP_MAX = 8, GEMM_F32_GROUP_TILES = 4096;
constexpr long GEMM_F32_GRID_X = 1l << 22, GEMM_F32_GRID_Y = 65535;      // (the threads of a grid's first dimension are counted in 32 bits)
// One tile.  ANY: contractions and leading dimensions that are not multiples of 4 (one value per load instead of 16 bytes along the contraction), and any
// number of tiles.  A kernel of its own: looking for the folds costs each of a small stage's launches 0.1 to 0.3 us.
template <int NW, bool A_MC, bool B_MC, bool ANY>
__device__ __forceinline__ void gemm_f32_tile(const GemmF32Params& p, int tile_m, int tile_n) {
  constexpr int U = 4;                // chunks in flight per wave
  __shared__ float red[NW][32][33];
  __shared__ float csred[NW][32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, q = lane >> 4;
  const int m0 = tile_m * 32, n0 = tile_n * 32, chunks = (p.K + 15) / 16;
  f32x4 acc[2][2];
  float cs[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int am[2] = {min(m0 + l16, p.M - 1), min(m0 + 16 + l16, p.M - 1)};
  const int bn[2] = {min(n0 + l16, p.N - 1), min(n0 + 16 + l16, p.N - 1)};
  const bool do_cs = A_MC && p.colsum != nullptr && tile_n == 0;
  // a lane's four contraction values of chunk c: k = 16 c + 4 q + 0..3, the same for both operands
  auto fetch = [&](const float* base, int ld, bool mc, int row, int c) {
    const int k = c * 16 + 4 * q;
    if (!ANY && !mc) return *reinterpret_cast<const f32x4*>(base + (size_t)row * ld + min(k, p.K - 4));
    f32x4 v;
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = mc ? base[(size_t)min(k + t, p.K - 1) * ld + row] : base[(size_t)row * ld + min(k + t, p.K - 1)];
    return v;
  };
  for (int c0 = wave; c0 < chunks; c0 += NW * U) {
    f32x4 a[U][2], b[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int c = min(c0 + NW * u, chunks - 1);      // a chunk past the wave's last one is fetched, but not multiplied
        a[u][i] = fetch(p.A, p.lda, A_MC, am[i], c);
        b[u][i] = fetch(p.B, p.ldb, B_MC, bn[i], c);
      }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + NW * u;
      if (c >= chunks) continue;
      if (c * 16 + 16 > p.K) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (c * 16 + 4 * q + t >= p.K) { a[u][i][t] = 0.f; b[u][i][t] = 0.f; }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][t], b[u][j][t], acc[i][j], 0, 0, 0);
      if (do_cs) {
#pragma unroll
        for (int i = 0; i < 2; ++i) cs[i] += (a[u][i][0] + a[u][i][1]) + (a[u][i][2] + a[u][i][3]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][16 * i + 4 * q + r][16 * j + l16] = acc[i][j][r];
  if (do_cs) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      cs[i] += __shfl_xor(cs[i], 16, 64);
      cs[i] += __shfl_xor(cs[i], 32, 64);
      if (q == 0) csred[wave][16 * i + l16] = cs[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 1024 / (NW * 64); ++e) {
    const int id = tid + e * NW * 64, r = id / 32, c = id % 32;
    float v = red[0][r][c];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w][r][c];
    epi_store<float>(p.epi, m0 + r, n0 + c, v);
  }
  if (do_cs && tid < 32 && m0 + tid < p.M) {
    float s = csred[0][tid];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += csred[w][tid];
    float* o = p.colsum + m0 + tid;
    *o = p.colsum_acc ? *o + s : s;
  }
}

template <int NW, bool A_MC, bool B_MC, bool ANY>
__global__ void __launch_bounds__(NW * 64) gemm_f32_kernel(const GemmF32Params p) {
  int tile_m = blockIdx.y, tile_n = blockIdx.x;
  if (ANY) {
    tile_m += (int)(blockIdx.z % p.fold_m * GEMM_F32_GRID_Y); tile_n += (int)(blockIdx.z / p.fold_m * GEMM_F32_GRID_X);
    if ((long)tile_m * 32 >= p.M || (long)tile_n * 32 >= p.N) return;
  }
  gemm_f32_tile<NW, A_MC, B_MC, ANY>(p, tile_m, tile_n);
}
// Several weight gradients (both operands contraction-strided) in one launch: problem i has the workgroups from first[i] on.
struct GemmF32Group { GemmF32Params p[GEMM_F32_GROUP_MAX]; int first[GEMM_F32_GROUP_MAX], n; };
template <int NW>
__global__ void __launch_bounds__(NW * 64) gemm_f32_group_kernel(const GemmF32Group g) {
  int i = 0;
  while (i + 1 < g.n && (int)blockIdx.x >= g.first[i + 1]) ++i;
  const GemmF32Params& p = g.p[i];
  const int tiles_n = (p.N + 31) / 32, id = blockIdx.x - g.first[i];
  gemm_f32_tile<NW, true, true, false>(p, id / tiles_n, id % tiles_n);
}

template <int NW, bool ANY>
static void launch_f32(const GemmF32Params& p, int a_mc, int b_mc, dim3 grid, hipStream_t s) {
  const dim3 block(NW * 64);
  if (a_mc && b_mc) hipLaunchKernelGGL((gemm_f32_kernel<NW, true, true, ANY>), grid, block, 0, s, p);
  else if (a_mc) hipLaunchKernelGGL((gemm_f32_kernel<NW, true, false, ANY>), grid, block, 0, s, p);
  else if (b_mc) hipLaunchKernelGGL((gemm_f32_kernel<NW, false, true, ANY>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((gemm_f32_kernel<NW, false, false, ANY>), grid, block, 0, s, p);
}

static GemmF32Params f32_params(const GemmArgs& a) {
  GemmF32Params p;
  p.A = (const float*)a.A; p.B = (const float*)a.B;
  p.M = a.M; p.N = a.N; p.K = a.K; p.lda = a.lda; p.ldb = a.ldb; p.fold_m = 1; p.colsum = a.colsum_out; p.colsum_acc = a.accumulate;
  EpiParams<float>& e = p.epi;
  e = EpiParams<float>();
  e.M = a.M; e.N = a.N; e.out = (float*)a.out; e.ldo = a.ldo; e.out32 = a.out_f32; e.ldo32 = a.ldo32; e.accumulate = a.accumulate;
  e.bias = (const float*)a.bias; e.pre_out = (float*)a.pre_out; e.ld_pre = a.ld_pre; e.act = a.act;
  e.dact_pre = (const float*)a.dact_pre; e.ld_dact = a.ld_dact; e.dact_kind = a.dact_kind;
  e.gate = (const float*)a.gate; e.gate_ld = a.gate_ld; e.rows_per_batch = a.rows_per_batch > 0 ? a.rows_per_batch : 1;
  e.residual = a.residual; e.ld_res = a.ld_res; e.out_scale = 1.0f;
  return p;
}
int launch_gemm_f32(const GemmArgs& a, hipStream_t s) {
  const bool wide = (a.a_mc || (a.K % 4 == 0 && a.lda % 4 == 0 && (uintptr_t)a.A % 16 == 0)) && (a.b_mc || (a.K % 4 == 0 && a.ldb % 4 == 0 && (uintptr_t)a.B % 16 == 0));
  const long tiles_m = ((long)a.M + 31) / 32, tiles_n = ((long)a.N + 31) / 32;
  const long fold_m = (tiles_m + GEMM_F32_GRID_Y - 1) / GEMM_F32_GRID_Y, fold_n = (tiles_n + GEMM_F32_GRID_X - 1) / GEMM_F32_GRID_X;
  const dim3 grid((unsigned)std::min(tiles_n, GEMM_F32_GRID_X), (unsigned)std::min(tiles_m, GEMM_F32_GRID_Y), (unsigned)(fold_m * fold_n));
  GemmF32Params p = f32_params(a);
  p.fold_m = (int)fold_m;
  KScope ks(KK_GEMM_F32, 2.0 * a.M * a.N * a.K, 4.0 * ((double)a.M * a.K + (double)a.N * a.K + (double)a.M * a.N), s, a.M, a.N, a.K);
  // eight waves share a contraction that gives four of them more than two chunks each
  const bool any = !wide || grid.z > 1;
  if (a.K > 128) any ? launch_f32<8, true>(p, a.a_mc, a.b_mc, grid, s) : launch_f32<8, false>(p, a.a_mc, a.b_mc, grid, s);
  else any ? launch_f32<4, true>(p, a.a_mc, a.b_mc, grid, s) : launch_f32<4, false>(p, a.a_mc, a.b_mc, grid, s);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm(f32) launch failed");
}

// Weight gradients whose operands are all there, one launch for those of each number of waves: each alone fills a few of the CUs and costs 3.2 to 5 us of
// dependent launch.  Every tile is computed as by a launch of its own, so no bit changes.
int launch_gemm_f32_group(const GemmArgs* a, int n, hipStream_t s) {
  for (int wide = 0; wide < 2; ++wide) {
    GemmF32Group g;
    long total = 0;
    double flops = 0.0, bytes = 0.0;
    const GemmArgs* first = nullptr;
    g.n = 0;
    auto flush = [&]() {
      if (!g.n) return (int)DP_OK;
      KScope ks(KK_GEMM_F32, flops, bytes, s, first->M, first->N, first->K);
      if (wide) hipLaunchKernelGGL(gemm_f32_group_kernel<8>, dim3((unsigned)total), dim3(512), 0, s, g);
      else hipLaunchKernelGGL(gemm_f32_group_kernel<4>, dim3((unsigned)total), dim3(256), 0, s, g);
      g.n = 0; total = 0; flops = bytes = 0.0;
      return hipGetLastError() == hipSuccess ? (int)DP_OK : set_error(DP_EHIP, "gemm(f32) launch failed");
    };
    for (int i = 0; i < n; ++i) {
      if ((a[i].K > 128) != (wide == 1)) continue;
      const long tiles = (((long)a[i].M + 31) / 32) * (((long)a[i].N + 31) / 32);
      if (tiles > GEMM_F32_GROUP_TILES || !a[i].a_mc || !a[i].b_mc) { DP_TRY(launch_gemm(a[i], s)); continue; }
      if (g.n == GEMM_F32_GROUP_MAX || total + tiles > GEMM_F32_GRID_X) DP_TRY(flush());
      if (!g.n) first = &a[i];
      g.first[g.n] = (int)total; g.p[g.n++] = f32_params(a[i]);
      total += tiles;
      flops += 2.0 * a[i].M * a[i].N * a[i].K;
      bytes += 4.0 * ((double)a[i].M * a[i].K + (double)a[i].N * a[i].K + (double)a[i].M * a[i].N);
    }
    DP_TRY(flush());
  }
  return DP_OK;
}

}  // namespace dp
