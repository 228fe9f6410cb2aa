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

#include <algorithm>
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

// ------------------------------------------------------------------ conditioning gradient
// sum over the blocks of dm_b [M, K] W_b [K, N] for at most 48 rows: the modulation projections backwards.  Bound by the weights' way from
// memory (7 blocks of 6912 x 1152: 111 MB); one product, sum of partials, and activation gradient per block took 7 x 28 us, together 34 (3.8 TB/s).
// The contraction runs over all blocks and is cut into parts; a workgroup owns all rows and 128 columns of one part.  Its waves share
// the part's k-tiles of 48 (a DiT's 6 d is always a multiple): a wave copies 48 weight rows into LDS of its own, reads them transposed
// while its next ones are on their way, and takes the rows of dm straight from memory.
struct CondGradParams {
  int M, N, K, lda, ldb, tiles, tiles_per_part;       // k-tiles: of all blocks, of a part
  const bf16* A[GEMM_BATCH_MAX]; const bf16* B[GEMM_BATCH_MAX];
  float* partial;                                     // [part][M][N]
};
template <int MT>
__global__ void __launch_bounds__(256, MT == 1 ? 2 : 1) cond_grad_kernel(const CondGradParams p) {
  constexpr int BK = 48, BN = 128, STAGE = BK * BN * 2, S_LD = 68;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[4 * STAGE];
  static_assert(4 * 32 * S_LD * 4 <= 4 * STAGE, "slab");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, l32 = lane & 31;
  const int n0 = blockIdx.x * BN, t_end = min(p.tiles, (int)(blockIdx.y + 1) * p.tiles_per_part), per_block = p.K / BK;
  unsigned char* own = smem + wave * STAGE;
  bf16x8 fa[3][MT];
  // 48 weight rows of 256 bytes: 12 pieces of 4 rows; row k's 16-byte chunks are permuted (frag_from_mc_swz)
  auto fetch = [&](int t) {
    const int b = t / per_block, k0 = (t - b * per_block) * BK;
    const bf16* w = p.B[b] + (size_t)k0 * p.ldb;
    const bf16* a = p.A[b] + k0 + 8 * g;
#pragma unroll
    for (int j = 0; j < 12; ++j) {
      const int k = 4 * j + (lane >> 4), c = mc_swizzle(lane & 15, k);
      async_copy_16B(w + (size_t)k * p.ldb + min(n0 + c * 8, p.N - 8), own + j * 1024);
    }
#pragma unroll
    for (int ks = 0; ks < 3; ++ks)
#pragma unroll
      for (int i = 0; i < MT; ++i) fa[ks][i] = *reinterpret_cast<const bf16x8*>(a + (size_t)min(32 * i + l32, p.M - 1) * p.lda + ks * 16);
  };
  f32x16 acc[MT][4];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  int t = blockIdx.y * p.tiles_per_part + wave;
  if (t < t_end) fetch(t);
#pragma unroll 1
  for (; t < t_end; t += 4) {
    wait_vmcnt<0>();
    bf16x8 fb[3][4], ca[3][MT];
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) {
#pragma unroll
      for (int j = 0; j < 4; ++j) fb[ks][j] = frag_from_mc_swz(reinterpret_cast<const bf16*>(own), BN, ks * 16, 32 * j, lane);
#pragma unroll
      for (int i = 0; i < MT; ++i) ca[ks][i] = fa[ks][i];
    }
    wait_lgkmcnt0();
    if (t + 4 < t_end) fetch(t + 4);
#pragma unroll
    for (int ks = 0; ks < 3; ++ks)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma32(ca[ks][i], fb[ks][j], acc[i][j]);
  }
  // the four waves' sums in wave order, 32 rows and 64 columns at a time
  float* slab = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) slab[(wave * 32 + acc_row(r, g)) * S_LD + 32 * j + l32] = acc[i][2 * h + j][r];
      __syncthreads();
      const int row = tid >> 3, c = (tid & 7) * 8, m = 32 * i + row, n = n0 + 64 * h + c;
      if (m < p.M && n < p.N) {
        float v[8];
        pp_slab_row(&slab[row * S_LD + c], v);
#pragma unroll
        for (int w = 1; w < 4; ++w) {
          float x[8];
          pp_slab_row(&slab[(w * 32 + row) * S_LD + c], x);
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] += x[u];
        }
        float* o = p.partial + ((size_t)blockIdx.y * p.M + m) * p.N + n;
        *reinterpret_cast<f32x4*>(o) = *reinterpret_cast<const f32x4*>(&v[0]);
        *reinterpret_cast<f32x4*>(o + 4) = *reinterpret_cast<const f32x4*>(&v[4]);
      }
    }
}
// d_cond = SiLU'(cond) * sum of the parts, in ascending order within a thread's share (every eighth part) and over the shares.
__global__ void __launch_bounds__(256) cond_grad_finish_kernel(const float* __restrict__ partial, int parts, const bf16* __restrict__ cond, float* __restrict__ d_cond, int n) {
  __shared__ f32x4 red[8][32];
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5, i = (blockIdx.x * 32 + x) * 4;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if (i < n)
#pragma unroll 4
    for (int z = y; z < parts; z += 8) s += *reinterpret_cast<const f32x4*>(partial + (size_t)z * n + i);
  red[y][x] = s;
  __syncthreads();
  if (y || i >= n) return;
#pragma unroll
  for (int z = 1; z < 8; ++z) s += red[z][x];
  const bf16x4 c = *reinterpret_cast<const bf16x4*>(cond + i);
#pragma unroll
  for (int u = 0; u < 4; ++u) s[u] *= silu_grad_f((float)c[u]);
  *reinterpret_cast<f32x4*>(d_cond + i) = s;
}

bool cond_grad_supported(int dtype, int batch, int d) { return dtype == BF16 && batch <= 48 && d % 8 == 0; }
// Parts of the contraction over `blocks` blocks: two workgroups per CU, at least four k-tiles each.
static int cond_grad_parts(int blocks, int d) {
  const int tiles = blocks * (6 * d / 48), per = std::max(4, (tiles * ((d + 127) / 128) + 511) / 512);
  return (tiles + per - 1) / per;
}
size_t cond_grad_ws_bytes(int blocks, int batch, int d) {
  size_t parts = 0;
  for (int b = 0; b < blocks; b += GEMM_BATCH_MAX) parts += cond_grad_parts(std::min(blocks - b, GEMM_BATCH_MAX), d);
  return parts * batch * d * sizeof(float);
}
int launch_cond_grad(const void* const* dm, const void* const* w, int blocks, int batch, int d, float* ws, const void* cond, float* d_cond, hipStream_t s) {
  int parts = 0;
  if (!dm || !w || !ws || blocks < 1 || batch < 1 || !cond_grad_supported(BF16, batch, d)) return set_error(DP_EINVAL, "cond_grad: bad arguments");
  for (int b0 = 0; b0 < blocks; b0 += GEMM_BATCH_MAX) {
    CondGradParams p;
    memset(&p, 0, sizeof(p));
    const int n = std::min(blocks - b0, GEMM_BATCH_MAX);
    p.M = batch; p.N = d; p.K = 6 * d; p.lda = 6 * d; p.ldb = d; p.tiles = n * (6 * d / 48);
    const int np = cond_grad_parts(n, d);
    p.tiles_per_part = (p.tiles + np - 1) / np;
    for (int i = 0; i < n; ++i) { p.A[i] = (const bf16*)dm[b0 + i]; p.B[i] = (const bf16*)w[b0 + i]; }
    p.partial = ws + (size_t)parts * batch * d;
    parts += np;
    KScope ks(KK_GEMM_NN, 2.0 * batch * d * 6.0 * d * n, n * 2.0 * (6.0 * d * d + 6.0 * batch * d) + 4.0 * np * batch * d, s, batch, d, 6 * d * n);
    const dim3 grid((d + 127) / 128, np);
    if (batch <= 32) hipLaunchKernelGGL(cond_grad_kernel<1>, grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL(cond_grad_kernel<2>, grid, dim3(256), 0, s, p);
  }
  const int n = batch * d;
  KScope ks(KK_OTHER, 0.0, 4.0 * (parts + 1.0) * n + 2.0 * n, s, batch, d, parts);
  hipLaunchKernelGGL(cond_grad_finish_kernel, dim3((n + 127) / 128), dim3(256), 0, s, ws, parts, (const bf16*)cond, d_cond, n);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "cond_grad launch failed");
}

}  // namespace dp
