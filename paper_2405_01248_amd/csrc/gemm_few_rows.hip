// y = x W^T + bias for at most 48 rows and several weights in one launch (bf16): the modulation vectors of a stage's DiT blocks.
//
// Bound by the weights' way from memory (7 blocks of 6912 x 1152: 111 MB).  One launch per block through the tile kernels took
// 17 us each, k-tile by k-tile and latency bound; together 31 us (3.6 TB/s).  A workgroup owns all rows and 16, 32 or 64
// columns; its eight waves share the contraction (wave w takes the 32-deep steps w, w + 8, ...), fetch their fragments straight from
// global memory into registers, a batch of steps ahead, and add their partial tiles through LDS in a fixed order.
#include "dp_device.h"
#include "dp_kernels.h"
#include "dp_errors.h"
#include "dp_host.h"
#include "dp_ktime.h"
#include "dp_gemm_pp.h"

#include <cstring>

namespace dp {

struct FewRowsParams {
  const bf16* A;
  int M, N, K, lda, ldb, ldo;
  const bf16* B[GEMM_BATCH_MAX]; const bf16* bias[GEMM_BATCH_MAX]; bf16* out[GEMM_BATCH_MAX];
};

// MT x NT: 16-row and 16-column tiles of a workgroup.
template <int MT, int NT>
__global__ void __launch_bounds__(512, 2) gemm_few_rows_kernel(const FewRowsParams p) {
  constexpr int BM = 16 * MT, BN = 16 * NT, C_LD = BN + 4, U = MT * NT > 10 ? 2 : 3;              // U: steps per batch; two batches in registers
  __shared__ __attribute__((aligned(16))) float red[4 * BM * C_LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, q = lane >> 4;
  const int n0 = blockIdx.x * BN, nks = p.K / 32, n_steps = nks > wave ? (nks - wave + 7) / 8 : 0;
  const bf16* bp[NT];
  const bf16* ap[MT];
#pragma unroll
  for (int j = 0; j < NT; ++j) bp[j] = p.B[blockIdx.y] + (size_t)min(n0 + 16 * j + l16, p.N - 1) * p.ldb + 8 * q;
#pragma unroll
  for (int i = 0; i < MT; ++i) ap[i] = p.A + (size_t)min(16 * i + l16, p.M - 1) * p.lda + 8 * q;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 fa[2][U][MT], fb[2][U][NT];
  auto load = [&](int s0, auto set) {           // steps past the wave's last one: a valid address, not multiplied
    constexpr int t = decltype(set)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(wave + 8 * (s0 + u), nks - 1) * 32;
#pragma unroll
      for (int j = 0; j < NT; ++j) fb[t][u][j] = *reinterpret_cast<const bf16x8*>(bp[j] + k);
#pragma unroll
      for (int i = 0; i < MT; ++i) fa[t][u][i] = *reinterpret_cast<const bf16x8*>(ap[i] + k);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mul = [&](int s0, auto set) {
    constexpr int t = decltype(set)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u >= n_steps) continue;
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[t][u][i], fb[t][u][j], acc[i][j], 0, 0, 0);
    }
  };
  constexpr std::integral_constant<int, 0> S0{};
  constexpr std::integral_constant<int, 1> S1{};
  load(0, S0);
  for (int s = 0; s < n_steps; s += 2 * U) {
    if (s + U < n_steps) load(s + U, S1);
    mul(s, S0);
    if (s + U < n_steps) {
      if (s + 2 * U < n_steps) load(s + 2 * U, S0);
      mul(s + U, S1);
    }
  }
  // the eight partial tiles: w + (w + 4) for w = 0..3, then these four in ascending order
  float* plane = red + (wave & 3) * BM * C_LD;
  auto at = [&](int i, int j, int r) -> float& { return plane[(16 * i + 4 * q + r) * C_LD + 16 * j + l16]; };
  if (wave >= 4) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) at(i, j, r) = acc[i][j][r];
  }
  __syncthreads();
  if (wave < 4) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) at(i, j, r) += acc[i][j][r];
  }
  __syncthreads();
  for (int c = tid; c < BM * BN / 8; c += 512) {
    const int row = c / (BN / 8), lc = c % (BN / 8) * 8, n = n0 + lc;
    if (row >= p.M || n >= p.N) continue;
    float v[8], t[8];
    pp_bias(p.bias[blockIdx.y], n, t);
    pp_slab_row(&red[row * C_LD + lc], v);
#pragma unroll
    for (int z = 1; z < 4; ++z) {
      float w[8];
      pp_slab_row(&red[z * BM * C_LD + row * C_LD + lc], w);
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] += w[u];
    }
    bf16x8 o;
#pragma unroll
    for (int u = 0; u < 8; ++u) o[u] = (bf16)(v[u] + t[u]);
    *reinterpret_cast<bf16x8*>(p.out[blockIdx.y] + (size_t)row * p.ldo + n) = o;
  }
}

// ------------------------------------------------------------------ host side
bool gemm_few_rows_supported(const GemmArgs& a) {
  return a.dtype == BF16 && !a.a_mc && !a.b_mc && !a.out_f32 && !a.geglu && !a.pre_out && !a.dact_pre && !a.gate && !a.residual && !a.act &&
         a.M >= 1 && a.M <= 48 && a.K % 32 == 0 && a.K >= 32 && a.N % 8 == 0 && a.N >= 8 && a.lda % 8 == 0 && a.ldb % 8 == 0 && a.ldo % 8 == 0;
}

template <int MT>
static void launch_few_rows(const FewRowsParams& p, int n, hipStream_t s) {
  // columns per workgroup: more of them read the rows less often, fewer give more workgroups
  const long t64 = (long)((p.N + 63) / 64) * n;
  if (t64 >= 256) hipLaunchKernelGGL((gemm_few_rows_kernel<MT, 4>), dim3((p.N + 63) / 64, n), dim3(512), 0, s, p);
  else if (2 * t64 >= 160) hipLaunchKernelGGL((gemm_few_rows_kernel<MT, 2>), dim3((p.N + 31) / 32, n), dim3(512), 0, s, p);
  else hipLaunchKernelGGL((gemm_few_rows_kernel<MT, 1>), dim3((p.N + 15) / 16, n), dim3(512), 0, s, p);
}

int launch_gemm_few_rows(const GemmArgs& a, const GemmBatch& batch, hipStream_t s) {
  if (!a.A || batch.n < 1 || batch.n > GEMM_BATCH_MAX) return set_error(DP_EINVAL, "gemm: bad arguments");
  if (!gemm_few_rows_supported(a)) return set_error(DP_EUNSUPPORTED, "gemm: problem not supported by the few-rows kernel");
  FewRowsParams p;
  memset(&p, 0, sizeof(p));
  p.A = (const bf16*)a.A; p.M = a.M; p.N = a.N; p.K = a.K; p.lda = a.lda; p.ldb = a.ldb; p.ldo = a.ldo;
  for (int i = 0; i < batch.n; ++i) { p.B[i] = (const bf16*)batch.B[i]; p.bias[i] = (const bf16*)batch.bias[i]; p.out[i] = (bf16*)batch.out[i]; }
  KScope ks(KK_GEMM_NT, 2.0 * a.M * a.N * a.K * batch.n, batch.n * 2.0 * ((double)a.M * a.K + (double)a.N * a.K + (double)a.M * a.N), s, a.M, a.N, a.K);
  if (a.M <= 16) launch_few_rows<1>(p, batch.n, s);
  else if (a.M <= 32) launch_few_rows<2>(p, batch.n, s);
  else launch_few_rows<3>(p, batch.n, s);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gemm launch failed");
}

}  // namespace dp
