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
// The rows operand is LN(x), see GemmArgs::norm_x.  An argument of its own: a group's problems are 1.5 KB of kernel arguments already.
struct GemmF32Norm { const float *x, *gamma, *beta; float eps; float *out, *mean, *rstd, *copy; };

// problems of a grouped launch, and the tiles from which a problem fills the chip several times over by itself
constexpr int GEMM_F32_GROUP_MAX = 8, GEMM_F32_GROUP_TILES = 4096;
constexpr long GEMM_F32_GRID_X = 1l << 22, GEMM_F32_GRID_Y = 65535;      // (the threads of a grid's first dimension are counted in 32 bits)
// One tile.  ANY: contractions and leading dimensions that are not multiples of 4 (one value per load instead of 16 bytes along the contraction), and any
// number of tiles.  A kernel of its own: looking for the folds costs each of a small stage's launches 0.1 to 0.3 us.
// GG: the GeGLU around the product.  1, forward: the tile's columns of the values and of the gates, summed one after the other through the same LDS;
// stores both and value * gelu(gate).  2, backward: the product is the gradient of value * gelu(gate); stores those of the values and of the gates.
// NORM: the 32 rows are normalised by the workgroup itself and wait in the LDS of the final sums (rows of K + 4 values; eight waves have room for 256 columns, four for
// 128); the workgroups of the first column tile store what the backward needs.  What bounds a small stage is its chain of dependent launches: each such LayerNorm
// inside its product saves 1.75 us of it (step of a block 2 x 64 x 64: 25 launches 110.4 us, 22 launches 105.1; 106.7 with the weights fetched after the rows instead of
// before).
constexpr int GEMM_F32_NORM_K = 256;
template <int NW> __device__ __forceinline__ float (*gemm_f32_sums())[32][33] {      // one array a kernel, also where it holds two kinds of tiles
  __shared__ __attribute__((aligned(16))) float red[NW][32][33];
  return red;
}
template <int NW>
__device__ __forceinline__ void gemm_f32_rows(const GemmF32Params& p, const GemmF32Norm& n, int m0, bool store, float* rows) {
  constexpr int L = NW * 2, NC = GEMM_F32_NORM_K / 64;      // lanes a row; chunks of four columns a lane (four waves have at most 128 columns)
  static_assert((L == 8 || L == 16) && 32 * (NW * 32 + 4) <= NW * 32 * 33, "rows");
  const int l = threadIdx.x % L, r = threadIdx.x / L, m = min(m0 + r, p.M - 1);
  const float* src = n.x + (size_t)m * p.K;
  auto column = [&](int c) { return (c * L + l) * 4; };
  f32x4 x[NC], ga[NC], be[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    x[c] = ga[c] = be[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (column(c) < p.K) x[c] = *reinterpret_cast<const f32x4*>(src + column(c));
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (column(c) < p.K) { ga[c] = *reinterpret_cast<const f32x4*>(n.gamma + column(c)); be[c] = *reinterpret_cast<const f32x4*>(n.beta + column(c)); }
  auto row_sum = [&](float v) {
    if (L == 16) v += lane_dpp<0x128>(v);      // row_ror:8
    v += lane_dpp<0xB1>(v);                    // quad_perm:[1,0,3,2]
    v += lane_dpp<0x4E>(v);                    // quad_perm:[2,3,0,1]
    return v + lane_dpp<0x141>(v);             // row_half_mirror
  };
  float sum = 0.f, q = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) sum += (x[c][0] + x[c][1]) + (x[c][2] + x[c][3]);
  const float mu = row_sum(sum) / p.K;
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (column(c) < p.K) {
#pragma unroll
      for (int t = 0; t < 4; ++t) q += (x[c][t] - mu) * (x[c][t] - mu);
    }
  const float rs = rsqrtf(row_sum(q) / p.K + n.eps);
  store = store && m0 + r < p.M;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int k = column(c);
    if (k >= p.K) continue;
    f32x4 o;
#pragma unroll
    for (int t = 0; t < 4; ++t) o[t] = (x[c][t] - mu) * rs * ga[c][t] + be[c][t];
    *reinterpret_cast<f32x4*>(rows + r * (p.K + 4) + k) = o;
    if (store) {
      *reinterpret_cast<f32x4*>(n.out + (size_t)m * p.K + k) = o;
      if (n.copy) *reinterpret_cast<f32x4*>(n.copy + (size_t)m * p.K + k) = x[c];
    }
  }
  if (store && l == 0) { n.mean[m] = mu; n.rstd[m] = rs; }
  __syncthreads();
}
template <int NW, bool A_MC, bool B_MC, bool ANY, int GG = 0, bool NORM = false>
__device__ __forceinline__ void gemm_f32_tile(const GemmF32Params& p, int tile_m, int tile_n, const GemmF32Norm& norm = GemmF32Norm()) {
  constexpr int U = GG == 1 || NORM ? 2 : 4;  // chunks in flight per wave (NORM: all there are)
  constexpr int BJ = GG == 1 ? 4 : 2, E = 1024 / (NW * 64);
  float (*const red)[32][33] = gemm_f32_sums<NW>();
  __shared__ float csred[NW][32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, q = lane >> 4;
  const int m0 = tile_m * 32, n0 = tile_n * 32, chunks = (p.K + 15) / 16;
  f32x4 acc[2][BJ];
  float cs[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int am[2] = {min(m0 + l16, p.M - 1), min(m0 + 16 + l16, p.M - 1)};
  int bn[BJ];
#pragma unroll
  for (int j = 0; j < BJ; ++j) bn[j] = min(n0 + 16 * (j & 1) + l16, p.N - 1) + (j >> 1) * p.epi.geglu_inner;
  float u0[GG == 2 ? E : 1], u1[GG == 2 ? E : 1];      // the saved values and gates
  if constexpr (GG == 2) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int id = tid + e * NW * 64;
      const float* u = p.epi.geglu_u + (size_t)min(m0 + id / 32, p.M - 1) * p.epi.ld_geglu + min(n0 + id % 32, p.N - 1);
      u0[e] = u[0]; u1[e] = u[p.epi.geglu_inner];
    }
  }
  const bool do_cs = A_MC && p.colsum != nullptr && tile_n == 0;
  float* const norm_rows = &red[0][0][0];
  // a lane's four contraction values of chunk c: k = 16 c + 4 q + 0..3, the same for both operands
  auto fetch = [&](const float* base, int ld, bool mc, int row, int c) {
    const int k = c * 16 + 4 * q;
    if (!ANY && !mc) return *reinterpret_cast<const f32x4*>(base + (size_t)row * ld + min(k, p.K - 4));
    f32x4 v;
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = mc ? base[(size_t)min(k + t, p.K - 1) * ld + row] : base[(size_t)row * ld + min(k + t, p.K - 1)];
    return v;
  };
  f32x4 a[U][2], b[U][BJ];
  auto chunk = [&](int c0, int u) { return min(c0 + NW * u, chunks - 1); };      // a chunk past the wave's last one is fetched, but not multiplied
  auto fetch_b = [&](int c0, int u) {
#pragma unroll
    for (int j = 0; j < BJ; ++j) b[u][j] = fetch(p.B, p.ldb, B_MC, bn[j], chunk(c0, u));
  };
  auto multiply = [&](int c0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + NW * u;
      if (c >= chunks) continue;
      if (c * 16 + 16 > p.K) {
#pragma unroll
        for (int i = 0; i < BJ; ++i)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (c * 16 + 4 * q + t >= p.K) { if (i < 2) a[u][i][t] = 0.f; b[u][i][t] = 0.f; }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < BJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][t], b[u][j][t], acc[i][j], 0, 0, 0);
      if (do_cs) {
#pragma unroll
        for (int i = 0; i < 2; ++i) cs[i] += (a[u][i][0] + a[u][i][1]) + (a[u][i][2] + a[u][i][3]);
      }
    }
  };
  if constexpr (NORM) {
    // the weights' round trip passes under that of the rows
#pragma unroll
    for (int u = 0; u < U; ++u) fetch_b(wave, u);
    gemm_f32_rows<NW>(p, norm, m0, tile_n == 0, norm_rows);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i) a[u][i] = *reinterpret_cast<const f32x4*>(norm_rows + (16 * i + l16) * (p.K + 4) + min(chunk(wave, u) * 16 + 4 * q, p.K - 4));
    multiply(wave);
  } else {
    for (int c0 = wave; c0 < chunks; c0 += NW * U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int i = 0; i < 2; ++i) a[u][i] = fetch(p.A, p.lda, A_MC, am[i], chunk(c0, u));
        fetch_b(c0, u);
      }
      multiply(c0);
    }
  }
  auto put = [&](int half) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][16 * i + 4 * q + r][16 * j + l16] = acc[i][2 * half + j][r];
  };
  auto total = [&](int e) {
    const int id = tid + e * NW * 64, r = id / 32, c = id % 32;
    float v = red[0][r][c];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w][r][c];
    return v;
  };
  if constexpr (NORM) __syncthreads();      // the last reads of the rows
  put(0);
  if (do_cs) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      cs[i] += __shfl_xor(cs[i], 16, 64);
      cs[i] += __shfl_xor(cs[i], 32, 64);
      if (q == 0) csred[wave][16 * i + l16] = cs[i];
    }
  }
  __syncthreads();
  float value[GG == 1 ? E : 1];
  if constexpr (GG == 1) {
#pragma unroll
    for (int e = 0; e < E; ++e) value[e] = total(e);
    __syncthreads();
    put(1);
    __syncthreads();
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int id = tid + e * NW * 64, m = m0 + id / 32, n = n0 + id % 32;
    const float v = total(e);
    if constexpr (GG == 0) epi_store<float>(p.epi, m, n, v);
    if (GG && m < p.M && n < p.N) {
      const int inner = p.epi.geglu_inner;
      float* o = p.epi.out + (size_t)m * p.epi.ldo + n;
      if constexpr (GG == 1) {
        const float uv = value[e] + (p.epi.bias ? p.epi.bias[n] : 0.f), ug = v + (p.epi.bias ? p.epi.bias[inner + n] : 0.f);
        if (p.epi.pre_out) {
          float* u = p.epi.pre_out + (size_t)m * p.epi.ld_pre + n;
          u[0] = uv; u[inner] = ug;
        }
        *o = uv * gelu_erf_f(ug);
      } else {
        o[0] = v * gelu_erf_f(u1[e]); o[inner] = v * u0[e] * gelu_erf_grad_f(u1[e]);
      }
    }
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
template <int NW>
__global__ void __launch_bounds__(NW * 64) gemm_f32_norm_kernel(const GemmF32Params p, const GemmF32Norm n) { gemm_f32_tile<NW, false, false, false, 0, true>(p, blockIdx.y, blockIdx.x, n); }
template <int NW, bool B_MC, int GG>
__global__ void __launch_bounds__(NW * 64) gemm_f32_geglu_kernel(const GemmF32Params p) { gemm_f32_tile<NW, false, B_MC, false, GG>(p, blockIdx.y, blockIdx.x); }
template <int NW>
__global__ void __launch_bounds__(NW * 64) gemm_f32_norm_geglu_kernel(const GemmF32Params p, const GemmF32Norm n) { gemm_f32_tile<NW, false, false, false, 1, true>(p, blockIdx.y, blockIdx.x, n); }
// Several products in one launch, both operands contraction-strided (MC) or neither: problem i has the workgroups from first[i] on.
struct GemmF32Group { GemmF32Params p[GEMM_F32_GROUP_MAX]; int first[GEMM_F32_GROUP_MAX], n; };
__device__ __forceinline__ int gemm_f32_group_problem(const GemmF32Group& g) {
  int i = 0;
  while (i + 1 < g.n && (int)blockIdx.x >= g.first[i + 1]) ++i;
  return i;
}
template <int NW, bool MC>
__global__ void __launch_bounds__(NW * 64) gemm_f32_group_kernel(const GemmF32Group g) {
  const int i = gemm_f32_group_problem(g);
  const GemmF32Params& p = g.p[i];
  const int tiles_n = (p.N + 31) / 32, id = blockIdx.x - g.first[i];
  gemm_f32_tile<NW, MC, MC, false>(p, id / tiles_n, id % tiles_n);
}
// The first problem's rows are to be normalised.
template <int NW>
__global__ void __launch_bounds__(NW * 64) gemm_f32_norm_group_kernel(const GemmF32Group g, const GemmF32Norm n) {
  const int i = gemm_f32_group_problem(g);
  const GemmF32Params& p = g.p[i];
  const int tiles_n = (p.N + 31) / 32, id = blockIdx.x - g.first[i];
  if (i == 0) gemm_f32_tile<NW, false, false, false, 0, true>(p, id / tiles_n, id % tiles_n, n);
  else gemm_f32_tile<NW, false, false, false>(p, id / tiles_n, id % tiles_n);
}

template <int NW, bool ANY>
static void launch_f32(const GemmF32Params& p, int a_mc, int b_mc, dim3 grid, hipStream_t s) {
  const dim3 block(NW * 64);
  if (a_mc && b_mc) hipLaunchKernelGGL((gemm_f32_kernel<NW, true, true, ANY>), grid, block, 0, s, p);
  else if (a_mc) hipLaunchKernelGGL((gemm_f32_kernel<NW, true, false, ANY>), grid, block, 0, s, p);
  else if (b_mc) hipLaunchKernelGGL((gemm_f32_kernel<NW, false, true, ANY>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((gemm_f32_kernel<NW, false, false, ANY>), grid, block, 0, s, p);
}

// 16-byte loads along the contraction
static bool f32_wide(const GemmArgs& a) {
  return (a.a_mc || (a.K % 4 == 0 && a.lda % 4 == 0 && (uintptr_t)a.A % 16 == 0)) && (a.b_mc || (a.K % 4 == 0 && a.ldb % 4 == 0 && (uintptr_t)a.B % 16 == 0));
}
// The fused GeGLU (GemmArgs::geglu 1 and 2): a launch less, 2.6 us and the gap behind it, and no trip of the gradient through memory.  The products of
// these sizes are bound by latency, so a tile of values and gates takes hardly longer than one of either.
bool gemm_f32_geglu_supported(const GemmArgs& a) {
  const long rows = ((long)a.M + 31) / 32, cols = ((long)a.geglu_inner + 31) / 32;
  return a.dtype == F32 && !a.a_mc && a.geglu_inner > 0 && f32_wide(a) && rows <= GEMM_F32_GRID_Y && cols <= GEMM_F32_GRID_X && (a.geglu == 2 ? a.N == a.geglu_inner : !a.b_mc && a.N == 2 * a.geglu_inner);
}
// LayerNorm inside the product (GemmArgs::norm_x), also in a group and in front of the GeGLU forward.
// Every column tile normalises its rows again, so not above the tiles that fill the chip several times over; below, it is never slower (us a step, a launch of its own and
// inside: 4 x 256 x 160, two blocks 775 -> 766, 2 x 64 x 256 160.1 -> 156.7, 4 x 256 x 256 525.3 -> 524.9, 16 x 256 x 256 1718 -> 1708, 16 x 1024 x 128 7865 -> 7834).
bool gemm_f32_norm_supported(const GemmArgs& a) {
  for (const void* q : {(const void*)a.norm_x, a.norm_gamma, a.norm_beta, (const void*)a.norm_out, (const void*)a.norm_copy}) if ((uintptr_t)q % 16) return false;
  return a.norm_x && a.norm_out && a.norm_mean && a.norm_rstd && a.dtype == F32 && !a.a_mc && !a.b_mc && !a.out_f32 && a.K <= GEMM_F32_NORM_K && a.lda == a.K && f32_wide(a) && a.geglu != 2 && (!a.geglu || gemm_f32_geglu_supported(a)) &&
         (((long)a.M + 31) / 32) * (((long)a.N + 31) / 32) <= GEMM_F32_GROUP_TILES;
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
  e.geglu_inner = a.geglu_inner; e.geglu_u = (const float*)a.geglu_u; e.ld_geglu = a.ld_geglu;
  return p;
}
static GemmF32Norm f32_norm(const GemmArgs& a) {
  return {a.norm_x, (const float*)a.norm_gamma, (const float*)a.norm_beta, a.norm_eps, a.norm_out, a.norm_mean, a.norm_rstd, a.norm_copy};
}
int launch_gemm_f32(const GemmArgs& a, hipStream_t s) {
  const bool wide = f32_wide(a);
  const long tiles_m = ((long)a.M + 31) / 32, tiles_n = ((long)a.N + 31) / 32;
  const long fold_m = (tiles_m + GEMM_F32_GRID_Y - 1) / GEMM_F32_GRID_Y, fold_n = (tiles_n + GEMM_F32_GRID_X - 1) / GEMM_F32_GRID_X;
  const dim3 grid((unsigned)std::min(tiles_n, GEMM_F32_GRID_X), (unsigned)std::min(tiles_m, GEMM_F32_GRID_Y), (unsigned)(fold_m * fold_n));
  GemmF32Params p = f32_params(a);
  p.fold_m = (int)fold_m;
  if (a.norm_x && !gemm_f32_norm_supported(a)) return set_error(DP_EUNSUPPORTED, "gemm(f32): the rows of this problem cannot be normalised inside the product");
  KScope ks(KK_GEMM_F32, 2.0 * a.M * a.N * a.K, 4.0 * ((double)a.M * a.K + (double)a.N * a.K + (double)a.M * a.N), s, a.M, a.N, a.K);
  if (a.geglu) {
    if (!gemm_f32_geglu_supported(a)) return set_error(DP_EUNSUPPORTED, "gemm(f32): fused GeGLU not available for this problem");
    p.N = p.epi.N = a.geglu_inner;
    const dim3 half((unsigned)((a.geglu_inner + 31) / 32), (unsigned)tiles_m), block(a.K > 128 ? 512 : 256);
    auto kern = a.K > 128 ? (a.geglu == 1 ? gemm_f32_geglu_kernel<8, false, 1> : (a.b_mc ? gemm_f32_geglu_kernel<8, true, 2> : gemm_f32_geglu_kernel<8, false, 2>))
                          : (a.geglu == 1 ? gemm_f32_geglu_kernel<4, false, 1> : (a.b_mc ? gemm_f32_geglu_kernel<4, true, 2> : gemm_f32_geglu_kernel<4, false, 2>));
    if (a.norm_x) hipLaunchKernelGGL((a.K > 128 ? gemm_f32_norm_geglu_kernel<8> : gemm_f32_norm_geglu_kernel<4>), half, block, 0, s, p, f32_norm(a));
    else hipLaunchKernelGGL(kern, half, block, 0, s, p);
    return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm(f32) launch failed");
  }
  if (a.norm_x) {
    hipLaunchKernelGGL((a.K > 128 ? gemm_f32_norm_kernel<8> : gemm_f32_norm_kernel<4>), grid, dim3(a.K > 128 ? 512 : 256), 0, s, p, f32_norm(a));
    return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm(f32) launch failed");
  }
  // eight waves share a contraction that gives four of them more than two chunks each
  const bool any = !wide || grid.z > 1;
  if (a.K > 128) any ? launch_f32<8, true>(p, a.a_mc, a.b_mc, grid, s) : launch_f32<8, false>(p, a.a_mc, a.b_mc, grid, s);
  else any ? launch_f32<4, true>(p, a.a_mc, a.b_mc, grid, s) : launch_f32<4, false>(p, a.a_mc, a.b_mc, grid, s);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm(f32) launch failed");
}

// Products whose operands are all there, one launch for those of each layout and number of waves: each alone fills a few of the CUs and costs 3.2 to 5 us of
// dependent launch (a block's seven weight gradients in two launches instead of seven: step of a U-Net block 2 x 64 x 64 144 -> 128.5 us).
// Every tile is computed as by a launch of its own, so no bit changes.
int launch_gemm_f32_group(const GemmArgs* a, int n, hipStream_t s) {
  for (int kind = 0; kind < 4; ++kind) {
    const bool eight = kind & 1, mc = kind & 2;
    GemmF32Group g;
    long total = 0;
    double flops = 0.0, bytes = 0.0;
    const GemmArgs* first = nullptr;
    g.n = 0;
    auto flush = [&]() {
      if (!g.n) return (int)DP_OK;
      KScope ks(KK_GEMM_F32, flops, bytes, s, first->M, first->N, first->K);
      auto kern = eight ? (mc ? gemm_f32_group_kernel<8, true> : gemm_f32_group_kernel<8, false>) : (mc ? gemm_f32_group_kernel<4, true> : gemm_f32_group_kernel<4, false>);
      const dim3 grid((unsigned)total), block(eight ? 512 : 256);
      if (first->norm_x) hipLaunchKernelGGL((eight ? gemm_f32_norm_group_kernel<8> : gemm_f32_norm_group_kernel<4>), grid, block, 0, s, g, f32_norm(*first));
      else hipLaunchKernelGGL(kern, grid, block, 0, s, g);
      g.n = 0; total = 0; flops = bytes = 0.0;
      return hipGetLastError() == hipSuccess ? (int)DP_OK : set_error(DP_EHIP, "gemm(f32) launch failed");
    };
    for (int i = 0; i < n; ++i) {
      if ((a[i].K > 128) != eight || (a[i].a_mc != 0) != mc) continue;
      const long tiles = (((long)a[i].M + 31) / 32) * (((long)a[i].N + 31) / 32);
      if (tiles > GEMM_F32_GROUP_TILES || (a[i].b_mc != 0) != mc || !f32_wide(a[i])) { DP_TRY(launch_gemm(a[i], s)); continue; }
      if (a[i].norm_x && !gemm_f32_norm_supported(a[i])) return set_error(DP_EUNSUPPORTED, "gemm(f32): the rows of this problem cannot be normalised inside the product");
      if (g.n == GEMM_F32_GROUP_MAX || total + tiles > GEMM_F32_GRID_X || a[i].norm_x) DP_TRY(flush());
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
