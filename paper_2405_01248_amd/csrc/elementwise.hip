// Bandwidth-bound kernels of a stage: LayerNorm forward/backward (affine or adaLN
// modulated), GeGLU, SiLU, gated-residual backward, column sums (bias gradients),
// split-K partial reduction, embedding gather.  Accesses of 16 bytes (8 for bf16 rows of a LayerNorm); 16, 32
// or 64 lanes or a workgroup per token row, or columns per thread; all reductions are in a fixed order (no
// float atomics), so results are run-to-run identical.  Templated on the storage type (bf16 or fp32); math is fp32.
#include "dp_device.h"
#include "dp_kernels.h"
#include "dp_errors.h"
#include "dp_ktime.h"

#include <type_traits>

namespace dp {

template <typename T> struct Vec;
template <> struct Vec<bf16> { static constexpr int N = 8; typedef bf16x8 type; };
template <> struct Vec<float> { static constexpr int N = 4; typedef f32x4 type; };

template <typename T> __device__ __forceinline__ void load_vec(const T* p, float* out) {
  typename Vec<T>::type v = *reinterpret_cast<const typename Vec<T>::type*>(p);
#pragma unroll
  for (int i = 0; i < Vec<T>::N; ++i) out[i] = to_f<T>(v[i]);
}
template <typename T> __device__ __forceinline__ void store_vec(T* p, const float* in) {
  typename Vec<T>::type v;
#pragma unroll
  for (int i = 0; i < Vec<T>::N; ++i) v[i] = from_f<T>(in[i]);
  *reinterpret_cast<typename Vec<T>::type*>(p) = v;
}

// V consecutive fp32 values (V = 4 or 8)
template <int V> __device__ __forceinline__ void load_f32(const float* p, float* out) {
#pragma unroll
  for (int i = 0; i < V; i += 4) *reinterpret_cast<f32x4*>(out + i) = *reinterpret_cast<const f32x4*>(p + i);
}
template <int V> __device__ __forceinline__ void store_f32(float* p, const float* in) {
#pragma unroll
  for (int i = 0; i < V; i += 4) *reinterpret_cast<f32x4*>(p + i) = *reinterpret_cast<const f32x4*>(in + i);
}

// ------------------------------------------------------------------ rows of a LayerNorm
// L lanes share a row (256 / L rows per workgroup at a time); lane l has columns 4 (c L + l) .. + 3 for c = 0 .. NC - 1, so every access of a group
// is L x 16 bytes in a row (fp32) and only the last chunk can be partly empty.  A wave of several rows asks for more bytes at a time and
// adds up fewer lanes; a row's lanes are all in one wave, so nothing waits at a barrier.
// Either side of the lines, 16 / 32 / 64 lanes, us: 32768 rows of 160 columns 5.9 / 7.1 / 8.3, 256 8.6 / 9.1 / 9.7, 384 11.9 / 11.8 / 12.2, 400 13.2 / 12.5 / 12.4, 768 27.9 / 20.9 /
// 20.6, 800 - / 22.2 / 21.5, 1152 - / 34.5 / 29.9; 8192 of 320 3.8 / 4.0 / 4.6, of 400 4.5 / 4.7 / 4.8; 4096 of 400 4.1 / 3.4 / 3.4, of 768 6.4 / 4.2 / 4.4; 2048 of 768 5.9 / 3.4 / 3.2.
constexpr int LN_MAX_CHUNKS = 8;      // d <= 64 * 4 * 8
struct LnShape { int lanes, chunks; };
static LnShape ln_shape(int rows, int d) {
  int l = d <= 384 ? 16 : (d <= 768 ? 32 : 64);
  while (l < 64 && l * 4 < d && rows / (256 / l) < 1024) l *= 2;      // few rows: more of them side by side
  return {l, (d + 4 * l - 1) / (4 * l)};
}
template <int FIRST, int LAST, class F> static void ln_with_chunks(int n, F f) {
  if constexpr (FIRST <= LAST) {
    if (n == FIRST) f(std::integral_constant<int, FIRST>());
    else ln_with_chunks<FIRST + 1, LAST>(n, f);
  }
}
// f(lanes, chunks) for the shapes that ln_shape() gives
template <class F> static void ln_dispatch(LnShape sh, F f) {
  using std::integral_constant;
  if (sh.lanes == 16) ln_with_chunks<1, 6>(sh.chunks, [&](auto c) { f(integral_constant<int, 16>(), c); });
  else if (sh.lanes == 32) ln_with_chunks<1, 6>(sh.chunks, [&](auto c) { f(integral_constant<int, 32>(), c); });
  else ln_with_chunks<1, LN_MAX_CHUNKS>(sh.chunks, [&](auto c) { f(integral_constant<int, 64>(), c); });
}
template <int L> __device__ __forceinline__ float ln_row_sum(float v) {      // over the L lanes of a row
  if constexpr (L == 64) v = reduce_halves(v, AddOp());
  if constexpr (L >= 32) v = reduce_row_pairs(v, AddOp());
  return reduce_row(v, AddOp());
}
template <typename T> struct Vec4 { typedef __attribute__((ext_vector_type(4))) T type; };
template <typename T> __device__ __forceinline__ typename Vec4<T>::type load4(const T* p) { return *reinterpret_cast<const typename Vec4<T>::type*>(p); }
template <typename T> __device__ __forceinline__ void store4(T* p, const float* in) {
  typename Vec4<T>::type v;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = from_f<T>(in[i]);
  *reinterpret_cast<typename Vec4<T>::type*>(p) = v;
}

// ------------------------------------------------------------------ LayerNorm forward
// Bound by memory.  With a wave per row and eight columns a lane, the second chunk of 640 columns had 16 of 64 lanes: 32768 x 320 16.9 -> 12.5 us,
// 8192 x 640 10.0 -> 8.3, 8192 x 1152 14.6 -> 12.7, 4928 x 768 6.6 -> 5.8.
template <typename TX, typename T, int L, int NC>
__global__ void __launch_bounds__(256) ln_fwd_kernel(int rows, int d, float eps, const TX* __restrict__ x, T* __restrict__ y,
                                                     const T* __restrict__ gamma, const T* __restrict__ beta,
                                                     const T* __restrict__ scale, const T* __restrict__ shift, int mod_ld,
                                                     int rows_per_batch, float* __restrict__ mean, float* __restrict__ rstd,
                                                     float* __restrict__ x32_out) {
  const int l = threadIdx.x % L, row_wanted = blockIdx.x * (256 / L) + threadIdx.x / L, row = min(row_wanted, rows - 1);
  const bool live = row_wanted < rows;
  const size_t at = (size_t)row * d;
  auto column = [&](int c) { return (c * L + l) * 4; };
  auto on = [&](int c) { return c + 1 < NC || column(c) < d; };
  typename Vec4<TX>::type xr[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (on(c)) xr[c] = load4(x + at + column(c));
  // gain and shift are fetched right behind the row, not after the two reductions: on a few rows the kernel's
  // time is its chain of memory round trips
  typename Vec4<T>::type ga[NC], sh[NC];
  const size_t mrow = scale ? (size_t)(row / rows_per_batch) * mod_ld : 0;
  const T* gsrc = scale ? scale + mrow : gamma;
  const T* ssrc = scale ? shift + mrow : beta;
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (on(c) && gsrc) { ga[c] = load4(gsrc + column(c)); sh[c] = load4(ssrc + column(c)); }
  float v[NC][4], s = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (!on(c)) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[c][i] = to_f<TX>(xr[c][i]); s += v[c][i]; }
    if (x32_out && live) store4(x32_out + at + column(c), v[c]);
  }
  const float mu = ln_row_sum<L>(s) / d;
  float q = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (!on(c)) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[c][i] -= mu; q += v[c][i] * v[c][i]; }
  }
  const float rs = rsqrtf(ln_row_sum<L>(q) / d + eps);
  if (!live) return;
  if (l == 0) {
    if (mean) mean[row] = mu;
    if (rstd) rstd[row] = rs;
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (!on(c)) continue;
    float o[4];
    if (scale) {
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = v[c][i] * rs * (1.0f + to_f<T>(ga[c][i])) + to_f<T>(sh[c][i]);
    } else if (gamma) {
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = v[c][i] * rs * to_f<T>(ga[c][i]) + to_f<T>(sh[c][i]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = v[c][i] * rs;
    }
    store4(y + at + column(c), o);
  }
}

template <typename TX, typename T>
static int ln_fwd_t(const LnArgs& a, hipStream_t s) {
  ln_dispatch(ln_shape(a.row_invariant ? 0 : a.rows, a.d), [&](auto l, auto nc) {
    constexpr int ROWS = 256 / l;
    hipLaunchKernelGGL((ln_fwd_kernel<TX, T, l, nc>), dim3((a.rows + ROWS - 1) / ROWS), dim3(256), 0, s, a.rows, a.d, a.eps, (const TX*)a.x, (T*)a.y,
                       (const T*)a.gamma, (const T*)a.beta, (const T*)a.scale, (const T*)a.shift, a.mod_ld,
                       a.rows_per_batch > 0 ? a.rows_per_batch : a.rows, a.mean, a.rstd, a.x32_out);
  });
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "ln_fwd launch failed");
}

// Split-K reduction onto the fp32 residual stream fused with the LayerNorm that follows (bf16 storage).  One workgroup per row, four columns
// per thread.  On a slice of a few samples the time is the chain of memory round trips, so the planes of partial sums are loaded eight at a time
// (and added in ascending order), bias, gain and shift with the first.  Encoder of one sample (24 launches
// of 77 rows of 768): 583 us with a wave per row and LDS-permute reductions, 528; twelve samples 882, 846.
constexpr int RRLN_PLANES = 8;
__global__ void __launch_bounds__(512) reduce_residual_ln_kernel(int rows, int d, float eps, const float* __restrict__ partial, int splits,
                                                                 const bf16* __restrict__ bias, float* __restrict__ x, bf16* __restrict__ y,
                                                                 const bf16* __restrict__ gamma, const bf16* __restrict__ beta) {
  constexpr int V = 4;
  __shared__ float red[2][8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6, col = tid * V;
  const bool on = col < d;
  const size_t plane = (size_t)rows * d, o = (size_t)blockIdx.x * d + col;
  float v[V] = {}, acc[V] = {};
  bf16x4 bi = {}, ga = {}, be = {};
  if (on) {
    load_f32<V>(x + o, v);
    if (bias) bi = *reinterpret_cast<const bf16x4*>(bias + col);
    ga = *reinterpret_cast<const bf16x4*>(gamma + col);
    be = *reinterpret_cast<const bf16x4*>(beta + col);
    for (int z = 0; z < splits; z += RRLN_PLANES) {
      float t[RRLN_PLANES][V];
#pragma unroll
      for (int u = 0; u < RRLN_PLANES; ++u)
        if (z + u < splits) load_f32<V>(partial + (z + u) * plane + o, t[u]);
#pragma unroll
      for (int u = 0; u < RRLN_PLANES; ++u)
        if (z + u < splits) {
#pragma unroll
          for (int i = 0; i < V; ++i) acc[i] = z + u ? acc[i] + t[u][i] : t[u][i];
        }
    }
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] += acc[i] + (float)bi[i];
    store_f32<V>(x + o, v);
  }
  auto row_sum = [&](float s, float* r) {
    s = wave_sum(s);
    if (waves == 1) return s;
    if (lane == 0) r[wave] = s;
    __syncthreads();
    s = r[0];
    for (int w = 1; w < waves; ++w) s += r[w];
    return s;
  };
  const float mu = row_sum((v[0] + v[1]) + (v[2] + v[3]), red[0]) / d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < V; ++i) { v[i] = on ? v[i] - mu : 0.f; q += v[i] * v[i]; }
  const float rs = rsqrtf(row_sum(q, red[1]) / d + eps);
  if (!on) return;
  bf16x4 out;
#pragma unroll
  for (int i = 0; i < V; ++i) out[i] = (bf16)(v[i] * rs * (float)ga[i] + (float)be[i]);
  *reinterpret_cast<bf16x4*>(y + o) = out;
}

int launch_reduce_residual_ln(const float* partial, int splits, int rows, int d, const void* bias, float* x, void* y,
                              const void* gamma, const void* beta, float eps, hipStream_t s) {
  if (!partial || splits < 1 || rows <= 0 || !x || !y || !gamma || !beta) return set_error(DP_EINVAL, "reduce_residual_ln: bad arguments");
  if (d <= 0 || d % 8 || d > 512 * 4) return set_error(DP_EUNSUPPORTED, "reduce_residual_ln: d must be a multiple of 8, at most 2048");
  KScope ks(KK_REDUCE, 0.0, (double)rows * d * (4.0 * splits + 8.0 + 2.0), s, rows, d, splits);
  hipLaunchKernelGGL(reduce_residual_ln_kernel, dim3(rows), dim3((d / 4 + 63) / 64 * 64), 0, s, rows, d, eps, partial, splits, (const bf16*)bias, x,
                     (bf16*)y, (const bf16*)gamma, (const bf16*)beta);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "reduce_residual_ln launch failed");
}

static int check_ln_dim(int dtype, int d) {
  const int V = dtype == BF16 ? 8 : 4;
  if (d <= 0 || d % V) return set_error(DP_EUNSUPPORTED, "layernorm: d must be a positive multiple of 8 (bf16) / 4 (fp32)");
  if (d > 256 * V) return set_error(DP_EUNSUPPORTED, "layernorm: d too large (max 2048 bf16 / 1024 fp32)");
  return DP_OK;
}

int launch_ln_fwd(const LnArgs& a, hipStream_t s) {
  if (a.rows <= 0 || !a.x || !a.y) return set_error(DP_EINVAL, "ln_fwd: bad arguments");
  if (int e = check_ln_dim(a.dtype, a.d)) return e;
  if ((a.gamma == nullptr) != (a.beta == nullptr) || (a.scale == nullptr) != (a.shift == nullptr))
    return set_error(DP_EINVAL, "ln_fwd: gamma/beta and scale/shift come in pairs");
  if (a.x32_out && ((a.x_f32 && a.dtype == BF16) || ((uintptr_t)a.x32_out % 16))) return set_error(DP_EINVAL, "ln_fwd: the fp32 copy goes with an input in the storage dtype and a 16-byte aligned destination");
  KScope ks(KK_LN_FWD, 0.0, a.rows * (double)a.d * (dtype_size(a.dtype) + (a.x_f32 ? 4 : dtype_size(a.dtype)) + (a.x32_out ? 4 : 0)) + 8.0 * a.rows, s, a.rows, a.d);
  if (a.dtype == BF16) return a.x_f32 ? ln_fwd_t<float, bf16>(a, s) : ln_fwd_t<bf16, bf16>(a, s);
  return ln_fwd_t<float, float>(a, s);
}

// ------------------------------------------------------------------ LayerNorm backward
// Rows per workgroup (a multiple of LNB_AT_ONCE): 16, fewer where that leaves few workgroups for the CUs; the lines are in 512 columns of a row, two waves of
// ln_bwd_kernel and one of gate_bwd_kernel in bf16.  1024 rows of 1152 on 64
// workgroups took 16.3 us, on 256 8.8; 8192 rows of 640 on 512 workgroups 26.8 us, on 1024 20.2 (with eight columns a thread).  A few dozen rows: two, one pass.
// (The partial sums to be added afterwards grow to the same number, a few MB.)
// Rows of more than 1024 columns are five to eight waves, and few such workgroups fit a CU: where those of the least rows do not run at once and those of
// up to 40 do, these are taken, instead of a second round that is nearly empty (us, 16 rows and as chosen: gated, 14336 x 1152 71.5 -> 55.5, 16384 83.1 -> 70.0, 24576 122 ->
// 106, 9216 x 1536 63.9 -> 52.3, 10240 x 1920 93.3 -> 75.2, 8 rows 6144 x 1536 29.9 -> 26.4; modulated alone, 14336 x 1600 71.8 -> 61.8; affine, 14336 x 1600 88.0 -> 80.8, 14336 x
// 1920 101 -> 95, but 24576 x 1152, where it is two rounds either way, 91 -> 101).  Narrower rows have workgroups enough to fill their last round.
static int ln_bwd_rows(int rows, int d, int rows_per_batch, bool modulated) {
  const long halves = (d + 511) / 512;
  const int least = rows * halves >= 1536 * 16 ? 16 : (rows * halves >= 1536 * 8 ? 8 : (rows * halves >= 512 ? 4 : 2));
  const int waves = (d / 4 + 63) / 64;
  if (least < 8 || waves < (modulated ? 5 : 6)) return least;
  const long at_once = 256 * (modulated ? (waves == 5 ? 3 : 2) : (waves == 6 ? 4 : 3));      // (modulated: of the gated kernel; as they were seen to run)
  for (const int r : {8, 10, 12, 14, 16, 20, 22, 24, 28, 32, 40})
    if (r >= least && (long)(rows / rows_per_batch) * ((rows_per_batch + r - 1) / r) <= at_once) return r;
  return least;
}

// Gated branch behind a result row: see ln_bwd_kernel.
struct GateBwd { const void* gate; int gate_ld; const void* branch; void* dbranch; float* partial; };
// A gated branch on its own (the last block's, whose result gradient comes from outside).  Rows and workgroups as in ln_bwd_kernel.
template <typename T>
__global__ void __launch_bounds__(256) gate_bwd_kernel(int d, int rows_per_batch, int wg_rows, const float* __restrict__ dres, const GateBwd gt) {
  constexpr int V = Vec<T>::N;
  const int b = blockIdx.y, col = threadIdx.x * V, r_begin = blockIdx.x * wg_rows, r_end = min(rows_per_batch, r_begin + wg_rows);
  if (col >= d) return;
  float hsum[V], gate[V];
#pragma unroll
  for (int i = 0; i < V; ++i) hsum[i] = 0.f;
  load_vec<T>((const T*)gt.gate + (size_t)b * gt.gate_ld + col, gate);
#pragma unroll 4
  for (int r = r_begin; r < r_end; ++r) {
    const size_t o = ((size_t)b * rows_per_batch + r) * d + col;
    float dr[V], br[V], ob[V];
    load_f32<V>(dres + o, dr);
    load_vec<T>((const T*)gt.branch + o, br);
#pragma unroll
    for (int i = 0; i < V; ++i) { hsum[i] = fmaf(dr[i], br[i], hsum[i]); ob[i] = dr[i] * gate[i]; }
    store_vec<T>((T*)gt.dbranch + o, ob);
  }
  store_f32<V>(gt.partial + ((size_t)b * gridDim.x + blockIdx.x) * 2 * d + col, hsum);
}

// grid = (chunks_per_batch, n_batches); a thread owns four columns of all rows of its workgroup (as many waves as a row has 64-lane
// chunks), so the column sums need no exchange; the rows' sums meet in LDS.  partial: [batch][chunk][2][d].
// The kernel moves ~16 bytes per element and is bound by how much of that is outstanding: LNB_AT_ONCE rows are loaded before the first is used.
// (With whole rows per wave a row of 1152 needed 242 registers; 1024 x 1152 8.8 us, 8192 x 1152 28.8 us; now 9.0 and 26 to 30 us, 32768 x 320 40.6 -> 31.6.
// With eight columns a thread, 80 of 128 lanes had any of 640: U-Net blocks 8 x 1024 x 640 1655 -> 1645 us, 8 x 4096 x 320 3266 -> 3255, and four rows ahead
// are no faster.  With a row's columns inside one wave, as in the forward, a workgroup has all its rows at once and nothing behind them: 8192 x 640 19.3 -> 26.5 us.)
//
// GATE: the result is also the gradient of a gated branch's sum, x_next = x + gate_b * branch: dbranch = result * gate_b, and per
// workgroup the column sums of result * branch (gate_partial, [batch][chunk][2][d], one of the two).  A kernel of its own for it reads the
// result again: 7.9 us at 1024 x 1152, 18.9 us at 8192 x 1152, against 2.5 and 14 to 18 here.
constexpr int LNB_AT_ONCE = 2;
template <typename T, bool GATE>
__global__ void __launch_bounds__(512, 2) ln_bwd_kernel(int d, int rows_per_batch, int wg_rows, const T* __restrict__ dy, const float* __restrict__ x,
                                                        const float* __restrict__ mean, const float* __restrict__ rstd,
                                                        const T* __restrict__ gamma, const T* __restrict__ scale, int mod_ld,
                                                        const float* __restrict__ dres, const T* __restrict__ dres_t,
                                                        T* __restrict__ dx, float* __restrict__ dx32, float* __restrict__ partial, const GateBwd gt) {
  constexpr int V = 4, R = LNB_AT_ONCE;
  using VT = typename Vec4<T>::type;
  __shared__ float red[2][8][2 * R];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6, b = blockIdx.y, col = tid * V;
  const bool on = col < d;
  const int r_begin = blockIdx.x * wg_rows, r_end = min(rows_per_batch, r_begin + wg_rows);
  auto widen = [](VT v, float (&out)[V]) {
#pragma unroll
    for (int i = 0; i < V; ++i) out[i] = to_f<T>(v[i]);
  };
  float gsum[V], bsum[V], gain[V], hsum[V], gate[V];
#pragma unroll
  for (int i = 0; i < V; ++i) { gsum[i] = 0.f; bsum[i] = 0.f; gain[i] = 1.f; hsum[i] = 0.f; gate[i] = 0.f; }
  if (on) {
    if (scale) {
      widen(load4(scale + (size_t)b * mod_ld + col), gain);
#pragma unroll
      for (int i = 0; i < V; ++i) gain[i] += 1.0f;
    } else if (gamma) {
      widen(load4(gamma + col), gain);
    }
    if constexpr (GATE) widen(load4((const T*)gt.gate + (size_t)b * gt.gate_ld + col), gate);
  }
  const float inv_d = 1.0f / d;
  int turn = 0;
  for (int r0 = r_begin; r0 < r_end; r0 += R, turn ^= 1) {
    VT dyr[R], drt[R], br[R];
    float xh[R][V], drf[R][V], g[R][V], mu[R], rs[R], s1[R], s2[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const size_t row = (size_t)b * rows_per_batch + min(r0 + k, r_end - 1);
      mu[k] = mean[row]; rs[k] = rstd[row];
      if (on) {
        const size_t o = row * d + col;
        dyr[k] = *reinterpret_cast<const VT*>(dy + o);
        load_f32<V>(x + o, xh[k]);
        if (dres) load_f32<V>(dres + o, drf[k]);
        else if (dres_t) drt[k] = *reinterpret_cast<const VT*>(dres_t + o);
        if constexpr (GATE) br[k] = *reinterpret_cast<const VT*>((const T*)gt.branch + o);
      }
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
      s1[k] = 0.f; s2[k] = 0.f;
      const bool live = r0 + k < r_end;      // a row past the last one is the last one again: taken out by choice, since 0 times an infinity is NaN
      if (on) {
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const float dyv = live ? to_f<T>(dyr[k][i]) : 0.f;
          xh[k][i] = live ? (xh[k][i] - mu[k]) * rs[k] : 0.f;
          gsum[i] += dyv * xh[k][i];
          bsum[i] += dyv;
          g[k][i] = dyv * gain[i];
          s1[k] += g[k][i];
          s2[k] += g[k][i] * xh[k][i];
        }
      }
      s1[k] = wave_sum(s1[k]); s2[k] = wave_sum(s2[k]);
    }
    if (waves > 1) {      // (two copies in turn: one barrier per pass)
      if (lane == 0) {
#pragma unroll
        for (int k = 0; k < R; ++k) { red[turn][wave][2 * k] = s1[k]; red[turn][wave][2 * k + 1] = s2[k]; }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < R; ++k) {
        s1[k] = red[turn][0][2 * k]; s2[k] = red[turn][0][2 * k + 1];
        for (int w = 1; w < waves; ++w) { s1[k] += red[turn][w][2 * k]; s2[k] += red[turn][w][2 * k + 1]; }
      }
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if (!on || r0 + k >= r_end) continue;
      const size_t o = ((size_t)b * rows_per_batch + r0 + k) * d + col;
      const float m1 = s1[k] * inv_d, m2 = s2[k] * inv_d;
      float v[V];
#pragma unroll
      for (int i = 0; i < V; ++i) v[i] = rs[k] * (g[k][i] - m1 - xh[k][i] * m2);
      if (dres) {
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] += drf[k][i];
      } else if (dres_t) {
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] += to_f<T>(drt[k][i]);
      }
      if constexpr (GATE) {
        float ob[V];
#pragma unroll
        for (int i = 0; i < V; ++i) { hsum[i] = fmaf(v[i], to_f<T>(br[k][i]), hsum[i]); ob[i] = v[i] * gate[i]; }
        store4((T*)gt.dbranch + o, ob);
      }
      if (dx32) store_f32<V>(dx32 + o, v);
      if (dx) store4(dx + o, v);
    }
  }
  if (!on) return;
  const size_t chunk = ((size_t)b * gridDim.x + blockIdx.x) * 2 * d;
  if (partial) { store_f32<V>(partial + chunk + col, gsum); store_f32<V>(partial + chunk + d + col, bsum); }
  if constexpr (GATE) store_f32<V>(gt.partial + chunk + col, hsum);
}

// out_k[b * ld + col] = (acc ? old : 0) + sum_chunks partial[b][chunk][k][col], k = 0 (gain grad), 1 (shift grad).
// grid = (ceil(2d / COLS), n_batches); a thread sums four columns of every GROUPS-th chunk in ascending order, then the groups are added in ascending
// order, in PARTS parts (fixed order; four for modulated LayerNorms, eight otherwise).  blockIdx.z: one of several LayerNorms of the same shape.  32 samples of 32 chunks of 1152, three
// LayerNorms: 6912 workgroups of 1024 threads that read a value each took 18.9 us, beside the main stream of a stage 140, now 12 and 27; 1024 chunks of 320 12 -> 6.
struct LnReduceSet { const float* partial[LN_REDUCE_MAX]; void* out0[LN_REDUCE_MAX]; void* out1[LN_REDUCE_MAX]; };
template <int THREADS, int COLS, typename Out>
__global__ void __launch_bounds__(THREADS) ln_bwd_reduce_kernel(const LnReduceSet set, int nchunk, int d, int ld, int accumulate) {
  const float* __restrict__ partial = set.partial[blockIdx.z];
  Out* out0 = (Out*)set.out0[blockIdx.z];
  Out* out1 = (Out*)set.out1[blockIdx.z];
  constexpr int GROUPS = THREADS / (COLS / 4), PARTS = THREADS / COLS < 8 ? THREADS / COLS : 8, PER = GROUPS / PARTS;
  static_assert(GROUPS % PARTS == 0 && THREADS % COLS == 0, "reduction shape");
  __shared__ __attribute__((aligned(16))) float red[GROUPS][COLS + 4];
  __shared__ float part[PARTS][COLS];
  const int tid = threadIdx.x, lc = tid % (COLS / 4) * 4, grp = tid / (COLS / 4), b = blockIdx.y, col = blockIdx.x * COLS + lc;     // col indexes the [2][d] row of a chunk
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if (col < 2 * d) {
    const float* p = partial + (size_t)b * nchunk * 2 * d + col;
#pragma unroll 8
    for (int c = grp; c < nchunk; c += GROUPS) s += *reinterpret_cast<const f32x4*>(p + (size_t)c * 2 * d);
  }
  *reinterpret_cast<f32x4*>(&red[grp][lc]) = s;
  __syncthreads();
  if (tid < COLS * PARTS) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < PER; ++g) t += red[tid / COLS * PER + g][tid % COLS];
    part[tid / COLS][tid % COLS] = t;
  }
  __syncthreads();
  const int oc = blockIdx.x * COLS + tid;
  if (tid < COLS && oc < 2 * d) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < PARTS; ++g) t += part[g][tid];
    Out* o = (oc < d ? out0 + oc : out1 + (oc - d)) + (size_t)b * ld;
    *o = from_f<Out>(accumulate ? to_f<Out>(*o) + t : t);
  }
}

size_t ln_bwd_partial_bytes(int rows, int d, int rows_per_batch, bool modulated) {
  const int nb = rows / rows_per_batch, wg_rows = ln_bwd_rows(rows, d, rows_per_batch, modulated), nchunk = (rows_per_batch + wg_rows - 1) / wg_rows;
  return (size_t)nb * nchunk * 2 * d * sizeof(float);
}

static GateBwd gate_of(const LnBwdArgs& a) { return GateBwd{a.gate, a.gate_ld, a.branch, a.dbranch, a.gate_partial}; }
static int ln_bwd_threads(const LnBwdArgs& a) { return (a.d / (a.dtype == BF16 ? 8 : 4) + 63) / 64 * 64; }      // at most 256: check_ln_dim
template <typename T>
static int ln_bwd_t(const LnBwdArgs& a, int rpb, int nb, int nchunk, float* partial, hipStream_t s) {
  auto kern = a.gate ? ln_bwd_kernel<T, true> : ln_bwd_kernel<T, false>;
  hipLaunchKernelGGL(kern, dim3(nchunk, nb), dim3((a.d / 4 + 63) / 64 * 64), 0, s, a.d, rpb, ln_bwd_rows(a.rows, a.d, rpb, a.scale != nullptr), (const T*)a.dy,
                     (const float*)a.x, a.mean, a.rstd, (const T*)a.gamma, (const T*)a.scale, a.mod_ld,
                     a.dres_storage ? nullptr : (const float*)a.dres, a.dres_storage ? (const T*)a.dres : nullptr, (T*)a.dx, a.dx32, partial, gate_of(a));
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "ln_bwd launch failed");
}

int launch_ln_bwd(const LnBwdArgs& a, hipStream_t s) {
  if (a.rows <= 0 || !a.dy || !a.x || !a.mean || !a.rstd || (!a.dx && !a.dx32)) return set_error(DP_EINVAL, "ln_bwd: bad arguments");
  if (int e = check_ln_dim(a.dtype, a.d)) return e;
  const bool modulated = a.scale != nullptr;
  const int rpb = modulated ? a.rows_per_batch : a.rows;
  if (rpb <= 0 || a.rows % rpb) return set_error(DP_EINVAL, "ln_bwd: rows must be a multiple of rows_per_batch");
  const int nb = a.rows / rpb, wg_rows = ln_bwd_rows(a.rows, a.d, rpb, modulated), nchunk = (rpb + wg_rows - 1) / wg_rows;
  if (a.gate && (!modulated || !a.branch || !a.dbranch || !a.gate_partial || !a.partial || a.gate_ld % 8)) return set_error(DP_EINVAL, "ln_bwd: a gated branch needs modulated rows, its operands and partial buffers");
  const bool want_cols = modulated ? (a.dscale && a.dshift) : (a.dgamma && a.dbeta);
  float* partial = nullptr;
  if (want_cols) {
    if (!a.partial || a.partial_bytes < ln_bwd_partial_bytes(a.rows, a.d, rpb, modulated)) return set_error(DP_EWORKSPACE, "ln_bwd: partial buffer too small");
    partial = a.partial;
  }
  int e;
  {
    KScope ks(KK_LN_BWD, 0.0, a.rows * (double)a.d * (dtype_size(a.dtype) + 4.0 + (a.dres ? (a.dres_storage ? dtype_size(a.dtype) : 4.0) : 0.0) + (a.dx ? dtype_size(a.dtype) : 0.0) + (a.dx32 ? 4.0 : 0.0) + (a.gate ? 2.0 * dtype_size(a.dtype) : 0.0)) + 8.0 * a.rows, s, a.rows, a.d);
    e = a.dtype == BF16 ? ln_bwd_t<bf16>(a, rpb, nb, nchunk, partial, s) : ln_bwd_t<float>(a, rpb, nb, nchunk, partial, s);
  }
  if (e || !want_cols || a.defer_reduce) return e;
  return launch_ln_bwd_reduce(&a, 1, s);
}

int launch_gate_bwd(const LnBwdArgs& a, hipStream_t s) {
  if (a.rows <= 0 || a.rows_per_batch <= 0 || a.rows % a.rows_per_batch || a.gate_ld % 8) return set_error(DP_EINVAL, "gate_bwd: bad sizes");
  if (int e = check_ln_dim(a.dtype, a.d)) return e;
  const void* ptrs[] = {a.dres, a.branch, a.gate, a.dbranch, a.gate_partial};
  for (const void* q : ptrs) if (!q || ((uintptr_t)q % 16)) return set_error(DP_EALIGN, "gate_bwd: operands must be non-null and 16-byte aligned");
  const int wg_rows = ln_bwd_rows(a.rows, a.d, a.rows_per_batch, true), nchunk = (a.rows_per_batch + wg_rows - 1) / wg_rows;
  auto kern = a.dtype == BF16 ? gate_bwd_kernel<bf16> : gate_bwd_kernel<float>;
  KScope ks(KK_OTHER, 0.0, a.rows * (double)a.d * (4.0 + 2.0 * dtype_size(a.dtype)), s, a.rows, a.d);
  hipLaunchKernelGGL(kern, dim3(nchunk, a.rows / a.rows_per_batch), dim3(ln_bwd_threads(a)), 0, s, a.d, a.rows_per_batch, wg_rows, (const float*)a.dres, gate_of(a));
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "gate_bwd launch failed");
}

// Second half of launch_ln_bwd for n LayerNorms of the same shape: fixed-order sum of the per-workgroup column partials
// into the parameter (or modulation) gradients.  Separate so that a caller can do it for a whole block at once (defer_reduce).
int launch_ln_bwd_reduce(const LnBwdArgs* a, int n, hipStream_t s) {
  if (n < 1 || n > LN_REDUCE_MAX) return set_error(DP_EINVAL, "ln_bwd_reduce: bad count");
  const bool modulated = a[0].scale != nullptr;
  const int d = a[0].d, rpb = modulated ? a[0].rows_per_batch : a[0].rows;
  LnReduceSet set;
  for (int i = 0; i < n; ++i) {
    if (rpb <= 0 || a[i].rows % rpb || !a[i].partial) return set_error(DP_EINVAL, "ln_bwd_reduce: bad arguments");
    if (a[i].rows != a[0].rows || a[i].d != d || (a[i].scale != nullptr) != modulated || (modulated && a[i].rows_per_batch != rpb) ||
        a[i].dmod_ld != a[0].dmod_ld || a[i].accumulate != a[0].accumulate)
      return set_error(DP_EINVAL, "ln_bwd_reduce: the LayerNorms differ in shape");
    set.partial[i] = a[i].partial;
    set.out0[i] = modulated ? a[i].dscale : (void*)a[i].dgamma;
    set.out1[i] = modulated ? a[i].dshift : (void*)a[i].dbeta;
  }
  const int nb = a[0].rows / rpb, wg_rows = ln_bwd_rows(a[0].rows, d, rpb, modulated), nchunk = (rpb + wg_rows - 1) / wg_rows;
  KScope ks(KK_REDUCE, 0.0, (double)n * nb * nchunk * 2 * d * 4, s, nchunk, 2 * d);
  if (modulated)
    hipLaunchKernelGGL((a[0].dtype == BF16 ? ln_bwd_reduce_kernel<256, 64, bf16> : ln_bwd_reduce_kernel<256, 64, float>), dim3((2 * d + 63) / 64, nb, n), dim3(256), 0, s, set, nchunk, d, a[0].dmod_ld, 0);
  else
    hipLaunchKernelGGL((ln_bwd_reduce_kernel<1024, 32, float>), dim3((2 * d + 31) / 32, 1, n), dim3(1024), 0, s, set, nchunk, d, d, a[0].accumulate);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "ln_bwd_reduce launch failed");
}

// ------------------------------------------------------------------ GeGLU
template <typename T>
__global__ void geglu_fwd_kernel(const T* __restrict__ u, T* __restrict__ g, size_t rows, int inner) {
  constexpr int V = Vec<T>::N;
  const int per_row = inner / V;
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= rows * per_row) return;
  const size_t r = i / per_row; const int c = (int)(i % per_row) * V;
  float a[V], b[V], o[V];
  load_vec<T>(u + r * 2 * inner + c, a);
  load_vec<T>(u + r * 2 * inner + inner + c, b);
#pragma unroll
  for (int k = 0; k < V; ++k) o[k] = a[k] * gelu_erf_f(b[k]);
  store_vec<T>(g + r * inner + c, o);
}
template <typename T>
__global__ void geglu_bwd_kernel(const T* __restrict__ dg, const T* __restrict__ u, T* __restrict__ du, size_t rows, int inner) {
  constexpr int V = Vec<T>::N;
  const int per_row = inner / V;
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= rows * per_row) return;
  const size_t r = i / per_row; const int c = (int)(i % per_row) * V;
  float a[V], b[V], dgo[V], o1[V], o2[V];
  load_vec<T>(u + r * 2 * inner + c, a);
  load_vec<T>(u + r * 2 * inner + inner + c, b);
  load_vec<T>(dg + r * inner + c, dgo);
#pragma unroll
  for (int k = 0; k < V; ++k) { o1[k] = dgo[k] * gelu_erf_f(b[k]); o2[k] = dgo[k] * a[k] * gelu_erf_grad_f(b[k]); }
  store_vec<T>(du + r * 2 * inner + c, o1);
  store_vec<T>(du + r * 2 * inner + inner + c, o2);
}

static int check_vec(int dtype, int n, const char* what) {
  const int V = dtype == BF16 ? 8 : 4;
  if (n <= 0 || n % V) return set_errorf(DP_EUNSUPPORTED, "%s: width must be a positive multiple of %d", what, V);
  return DP_OK;
}

int launch_geglu_fwd(int dtype, const void* u, void* g, int rows, int inner, hipStream_t s) {
  if (int e = check_vec(dtype, inner, "geglu")) return e;
  const int V = dtype == BF16 ? 8 : 4;
  const size_t n = (size_t)rows * (inner / V);
  KScope ks(KK_GEGLU_FWD, 0.0, 3.0 * rows * (double)inner * dtype_size(dtype), s, rows, inner);
  if (dtype == BF16) hipLaunchKernelGGL(geglu_fwd_kernel<bf16>, dim3((n + 255) / 256), dim3(256), 0, s, (const bf16*)u, (bf16*)g, (size_t)rows, inner);
  else hipLaunchKernelGGL(geglu_fwd_kernel<float>, dim3((n + 255) / 256), dim3(256), 0, s, (const float*)u, (float*)g, (size_t)rows, inner);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "geglu_fwd launch failed");
}
int launch_geglu_bwd(int dtype, const void* dg, const void* u, void* du, int rows, int inner, hipStream_t s) {
  if (int e = check_vec(dtype, inner, "geglu")) return e;
  const int V = dtype == BF16 ? 8 : 4;
  const size_t n = (size_t)rows * (inner / V);
  KScope ks(KK_GEGLU_BWD, 0.0, 5.0 * rows * (double)inner * dtype_size(dtype), s, rows, inner);
  if (dtype == BF16) hipLaunchKernelGGL(geglu_bwd_kernel<bf16>, dim3((n + 255) / 256), dim3(256), 0, s, (const bf16*)dg, (const bf16*)u, (bf16*)du, (size_t)rows, inner);
  else hipLaunchKernelGGL(geglu_bwd_kernel<float>, dim3((n + 255) / 256), dim3(256), 0, s, (const float*)dg, (const float*)u, (float*)du, (size_t)rows, inner);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "geglu_bwd launch failed");
}

// ------------------------------------------------------------------ column sums
constexpr int CS_ROWS = 64;    // rows per workgroup (16 per wave)

// Stage 1: partial[chunk][col] = sum of x over the chunk's rows.  A lane owns Vec::N consecutive
// columns (16-byte loads); the four waves of a workgroup take rows round-robin and are added
// in a fixed order.
template <typename T>
__global__ void __launch_bounds__(256) colsum_kernel(const T* __restrict__ x, int ldx, int rows, int cols, float* __restrict__ partial) {
  constexpr int V = Vec<T>::N;
  __shared__ float red[4][64 * V];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = (blockIdx.x * 64 + lane) * V;
  const int r0 = blockIdx.y * CS_ROWS, r1 = min(rows, r0 + CS_ROWS);
  float s[V];
#pragma unroll
  for (int i = 0; i < V; ++i) s[i] = 0.f;
  if (col < cols) {
    for (int r = r0 + wave; r < r1; r += 4) {
      float v[V];
      load_vec<T>(x + (size_t)r * ldx + col, v);
#pragma unroll
      for (int i = 0; i < V; ++i) s[i] += v[i];
    }
  }
#pragma unroll
  for (int i = 0; i < V; ++i) red[wave][lane * V + i] = s[i];
  __syncthreads();
  for (int t = threadIdx.x; t < 64 * V; t += 256) {
    const int c = blockIdx.x * 64 * V + t;
    if (c < cols) partial[(size_t)blockIdx.y * cols + c] = ((red[0][t] + red[1][t]) + red[2][t]) + red[3][t];
  }
}

// Stage 2: out[c] = (accumulate ? out[c] : 0) + sum_r partial[r][c]; 32 columns x 32 row groups per
// workgroup, each thread sums its rows in ascending order, the 32 group sums are added in ascending order.
__global__ void __launch_bounds__(1024) rows_reduce_kernel(const float* __restrict__ partial, int nrows, int ncols,
                                                           float* __restrict__ out, int accumulate) {
  __shared__ float red[32][33];
  const int lc = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int col = blockIdx.x * 32 + lc;
  float s = 0.f;
  if (col < ncols)
    for (int r = grp; r < nrows; r += 32) s += partial[(size_t)r * ncols + col];
  red[grp][lc] = s;
  __syncthreads();
  if (grp == 0 && col < ncols) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 32; ++g) t += red[g][lc];
    out[col] = accumulate ? out[col] + t : t;
  }
}

size_t colsum_partial_bytes(int rows, int cols) { return (size_t)((rows + CS_ROWS - 1) / CS_ROWS) * cols * sizeof(float); }

int launch_colsum(int dtype, const void* x, int ldx, int rows, int cols, float* out, int accumulate, float* partial,
                  size_t partial_bytes, hipStream_t s) {
  const int V = dtype == BF16 ? 8 : 4;
  if (rows <= 0 || cols <= 0 || cols % V || ldx % V || !x || !out) return set_error(DP_EINVAL, "colsum: bad arguments (cols must be a multiple of 8 (bf16) / 4 (fp32))");
  if (!partial || partial_bytes < colsum_partial_bytes(rows, cols)) return set_error(DP_EWORKSPACE, "colsum: partial buffer too small");
  dim3 grid((cols + 64 * V - 1) / (64 * V), (rows + CS_ROWS - 1) / CS_ROWS);
  KScope ks(KK_REDUCE, 0.0, (double)rows * cols * dtype_size(dtype), s, rows, cols);
  if (dtype == BF16) hipLaunchKernelGGL(colsum_kernel<bf16>, grid, dim3(256), 0, s, (const bf16*)x, ldx, rows, cols, partial);
  else hipLaunchKernelGGL(colsum_kernel<float>, grid, dim3(256), 0, s, (const float*)x, ldx, rows, cols, partial);
  if (hipGetLastError() != hipSuccess) return set_error(DP_EHIP, "colsum launch failed");
  hipLaunchKernelGGL(rows_reduce_kernel, dim3((cols + 31) / 32), dim3(1024), 0, s, partial, (int)grid.y, cols, out, accumulate);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "rows_reduce launch failed");
}

// out[i] = (accumulate ? out[i] : 0) + sum_z partial[z * n + i], four elements per thread (n % 4 == 0)
__global__ void reduce_partials_kernel(const float* __restrict__ partial, int nz, size_t n4, float* __restrict__ out, int accumulate) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= n4) return;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  for (int z = 0; z < nz; ++z) s += reinterpret_cast<const f32x4*>(partial)[(size_t)z * n4 + i];
  f32x4* o = reinterpret_cast<f32x4*>(out) + i;
  *o = accumulate ? *o + s : s;
}
int launch_reduce_partials(const float* partial, int nz, size_t n, float* out, int accumulate, hipStream_t s) {
  if (n % 4) return set_error(DP_EUNSUPPORTED, "reduce_partials: element count must be a multiple of 4");
  hipLaunchKernelGGL(reduce_partials_kernel, dim3((n / 4 + 255) / 256), dim3(256), 0, s, partial, nz, n / 4, out, accumulate);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "reduce_partials launch failed");
}

// Two tensors in one launch: out (n4 vectors of 4) and out_b (nb4 vectors), each summed over nz planes in plane order.
__global__ void reduce_partials2_kernel(const float* __restrict__ partial, int nz, size_t n4, float* __restrict__ out,
                                        const float* __restrict__ partial_b, size_t nb4, float* __restrict__ out_b, int accumulate) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  const float* src = partial; float* dst = out; size_t plane = n4;
  if (i >= n4) {
    i -= n4;
    if (i >= nb4) return;
    src = partial_b; dst = out_b; plane = nb4;
  }
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  for (int z = 0; z < nz; ++z) s += reinterpret_cast<const f32x4*>(src)[(size_t)z * plane + i];
  f32x4* o = reinterpret_cast<f32x4*>(dst) + i;
  *o = accumulate ? *o + s : s;
}
int launch_reduce_partials2(const float* partial, int nz, size_t n, float* out, const float* partial_b, size_t n_b, float* out_b,
                            int accumulate, hipStream_t s) {
  if (n % 4 || n_b % 4) return set_error(DP_EUNSUPPORTED, "reduce_partials: element counts must be multiples of 4");
  if (n_b && (!partial_b || !out_b)) return set_error(DP_EINVAL, "reduce_partials: second tensor missing");
  const size_t total = n / 4 + n_b / 4;
  hipLaunchKernelGGL(reduce_partials2_kernel, dim3((total + 255) / 256), dim3(256), 0, s, partial, nz, n / 4, out, partial_b, n_b / 4, out_b, accumulate);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "reduce_partials launch failed");
}

// ------------------------------------------------------------------ SiLU and its backward
template <typename T>
__global__ void silu_kernel(const T* __restrict__ x, T* __restrict__ y, size_t n) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < n) y[i] = from_f<T>(silu_f(to_f<T>(x[i])));
}
template <typename T>
__global__ void silu_bwd_kernel(const float* __restrict__ dz, const T* __restrict__ c, float* __restrict__ dc, int accumulate, size_t n) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float v = dz[i] * silu_grad_f(to_f<T>(c[i]));
  dc[i] = accumulate ? dc[i] + v : v;
}
int launch_silu(int dtype, const void* x, void* y, size_t n, hipStream_t s) {
  if (dtype == BF16) hipLaunchKernelGGL(silu_kernel<bf16>, dim3((n + 255) / 256), dim3(256), 0, s, (const bf16*)x, (bf16*)y, n);
  else hipLaunchKernelGGL(silu_kernel<float>, dim3((n + 255) / 256), dim3(256), 0, s, (const float*)x, (float*)y, n);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "silu launch failed");
}
int launch_silu_bwd(int dtype, const float* dz, const void* c, float* dc, int accumulate, size_t n, hipStream_t s) {
  if (dtype == BF16) hipLaunchKernelGGL(silu_bwd_kernel<bf16>, dim3((n + 255) / 256), dim3(256), 0, s, dz, (const bf16*)c, dc, accumulate, n);
  else hipLaunchKernelGGL(silu_bwd_kernel<float>, dim3((n + 255) / 256), dim3(256), 0, s, dz, (const float*)c, dc, accumulate, n);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "silu_bwd launch failed");
}

// ------------------------------------------------------------------ cast, embedding
template <typename T>
__global__ void cast_kernel(const float* __restrict__ in, T* __restrict__ out, size_t n) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < n) out[i] = from_f<T>(in[i]);
}
int launch_cast_from_f32(int dtype, const float* in, void* out, size_t n, hipStream_t s) {
  if (dtype == BF16) hipLaunchKernelGGL(cast_kernel<bf16>, dim3((n + 255) / 256), dim3(256), 0, s, in, (bf16*)out, n);
  else hipLaunchKernelGGL(cast_kernel<float>, dim3((n + 255) / 256), dim3(256), 0, s, in, (float*)out, n);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "cast launch failed");
}

template <typename T>
__global__ void cast_to_f32_kernel(const T* __restrict__ in, float* __restrict__ out, size_t n) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < n) out[i] = to_f<T>(in[i]);
}
int launch_cast_to_f32(int dtype, const void* in, float* out, size_t n, hipStream_t s) {
  if (dtype == BF16) hipLaunchKernelGGL(cast_to_f32_kernel<bf16>, dim3((n + 255) / 256), dim3(256), 0, s, (const bf16*)in, out, n);
  else hipLaunchKernelGGL(cast_to_f32_kernel<float>, dim3((n + 255) / 256), dim3(256), 0, s, (const float*)in, out, n);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "cast launch failed");
}

// bf16 -> OCP E4M3 with a per-tensor scale: the product with 1 / scale is formed in fp32, clamped to the format's
// largest finite value (+-448) and converted by the hardware's round-to-nearest-even conversion; 8 values per thread.
__global__ void __launch_bounds__(256) quantize_fp8_kernel(const bf16* __restrict__ x, int ldx, unsigned char* __restrict__ q, int ldq,
                                                           int rows, int cols, float inv_scale) {
  const size_t i = blockIdx.x * (size_t)256 + threadIdx.x;
  const int per_row = cols / 8;
  if (i >= (size_t)rows * per_row) return;
  const size_t r = i / per_row; const int c = (int)(i % per_row) * 8;
  const bf16x8 v = *reinterpret_cast<const bf16x8*>(x + r * ldx + c);
  float f[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) f[t] = fminf(fmaxf((float)v[t] * inv_scale, -448.0f), 448.0f);
  int lo = 0, hi = 0;
  lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[0], f[1], lo, false);
  lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[2], f[3], lo, true);
  hi = __builtin_amdgcn_cvt_pk_fp8_f32(f[4], f[5], hi, false);
  hi = __builtin_amdgcn_cvt_pk_fp8_f32(f[6], f[7], hi, true);
  u32x2 o = {(uint32_t)lo, (uint32_t)hi};
  *reinterpret_cast<u32x2*>(q + r * ldq + c) = o;
}
int launch_quantize_fp8(const void* x, int ldx, void* q, int ldq, int rows, int cols, float inv_scale, hipStream_t s) {
  if (rows <= 0 || cols <= 0 || !x || !q) return set_error(DP_EINVAL, "quantize_fp8: bad arguments");
  if (cols % 8 || ldx % 8 || ldq % 8 || ldx < cols || ldq < cols) return set_error(DP_EUNSUPPORTED, "quantize_fp8: cols and leading dims must be multiples of 8");
  if (((uintptr_t)x % 16) || ((uintptr_t)q % 8)) return set_error(DP_EALIGN, "quantize_fp8: operands must be 16- / 8-byte aligned");
  if (!(inv_scale > 0.f) || !(inv_scale < INFINITY)) return set_error(DP_EINVAL, "quantize_fp8: the scale must be positive and finite");
  const size_t n = (size_t)rows * (cols / 8);
  if ((n + 255) / 256 > 0x7fffffffull) return set_error(DP_EUNSUPPORTED, "quantize_fp8: tensor too large");
  KScope ks(KK_OTHER, 0.0, 3.0 * (double)rows * cols, s, rows, cols, 0);
  hipLaunchKernelGGL(quantize_fp8_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const bf16*)x, ldx, (unsigned char*)q, ldq, rows, cols, inv_scale);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "quantize_fp8 launch failed");
}

// One wave per token row.  Token ids outside [0, vocab) are clamped (ids live on the device
// and cannot be validated on the host); the sum is rounded once to the storage type.
template <typename T>
__global__ void __launch_bounds__(256) embed_kernel(const int32_t* __restrict__ ids, const T* __restrict__ tok, const T* __restrict__ pos,
                                                    T* __restrict__ x, float* __restrict__ x32, int rows, int seq, int d, int vocab) {
  constexpr int V = Vec<T>::N;
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  int id = ids[row];
  id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
  const T* t = tok + (size_t)id * d;
  const T* p = pos + (size_t)(row % seq) * d;
  for (int col = lane * V; col < d; col += 64 * V) {
    float a[V], b[V];
    load_vec<T>(t + col, a);
    load_vec<T>(p + col, b);
#pragma unroll
    for (int i = 0; i < V; ++i) a[i] = to_f<T>(from_f<T>(a[i] + b[i]));
    if (x32) store_f32<V>(x32 + (size_t)row * d + col, a);
    else store_vec<T>(x + (size_t)row * d + col, a);
  }
}
int launch_embed(int dtype, const int32_t* ids, const void* tok, const void* pos, void* x, float* x32, int rows, int seq, int d, int vocab,
                 hipStream_t s) {
  if (int e = check_vec(dtype, d, "embed")) return e;
  if (rows <= 0 || seq <= 0 || vocab <= 0) return set_error(DP_EINVAL, "embed: bad sizes");
  if (dtype == BF16) hipLaunchKernelGGL(embed_kernel<bf16>, dim3((rows + 3) / 4), dim3(256), 0, s, ids, (const bf16*)tok, (const bf16*)pos, (bf16*)x, x32, rows, seq, d, vocab);
  else hipLaunchKernelGGL(embed_kernel<float>, dim3((rows + 3) / 4), dim3(256), 0, s, ids, (const float*)tok, (const float*)pos, (float*)x, x32, rows, seq, d, vocab);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "embed launch failed");
}

// ---------------------------------------------------------------- batched 16-bit transpose
// dst[c, r] = src[r, c] for up to kTransposeMax dense row-major matrices in one launch (the weight
// matrices of a block, transposed once per backward pass so that dx = dy W runs as y = x W'^T on
// contraction-contiguous operands).  One workgroup moves a 64 x 64 tile through LDS.
__global__ void __launch_bounds__(256) transpose16_batch_kernel(const TransposeBatch tb) {
  __shared__ uint16_t tile[64][66];
  int mi = 0;
  while (mi + 1 < tb.n && (int)blockIdx.x >= tb.tile_start[mi + 1]) ++mi;
  const uint16_t* src = (const uint16_t*)tb.src[mi];
  uint16_t* dst = (uint16_t*)tb.dst[mi];
  const int R = tb.rows[mi], C = tb.cols[mi];
  const int tcols = (C + 63) / 64;
  const int t = blockIdx.x - tb.tile_start[mi];
  const int r0 = (t / tcols) * 64, c0 = (t % tcols) * 64;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int id = threadIdx.x + i * 256, r = id >> 3, c = (id & 7) * 8;
    if (r0 + r < R && c0 + c < C) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(src + (size_t)(r0 + r) * C + c0 + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) { tile[r][c + 2 * e] = (uint16_t)(v[e] & 0xffff); tile[r][c + 2 * e + 1] = (uint16_t)(v[e] >> 16); }
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int id = threadIdx.x + i * 256, c = id >> 3, r = (id & 7) * 8;   // output row c0 + c, output columns r0 + r .. + 7
    if (c0 + c < C && r0 + r < R) {
      u32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (uint32_t)tile[r + 2 * e][c] | ((uint32_t)tile[r + 2 * e + 1][c] << 16);
      *reinterpret_cast<u32x4*>(dst + (size_t)(c0 + c) * R + r0 + r) = v;
    }
  }
}
int launch_transpose16_batch(const TransposeBatch& tb, hipStream_t s) {
  if (tb.n <= 0 || tb.n > kTransposeMax) return set_error(DP_EINVAL, "transpose: bad matrix count");
  for (int i = 0; i < tb.n; ++i) {
    if (!tb.src[i] || !tb.dst[i] || tb.rows[i] <= 0 || tb.cols[i] <= 0) return set_error(DP_EINVAL, "transpose: bad matrix");
    if ((tb.rows[i] % 8) || (tb.cols[i] % 8)) return set_error(DP_EUNSUPPORTED, "transpose: dims must be multiples of 8");
    if (((uintptr_t)tb.src[i] % 16) || ((uintptr_t)tb.dst[i] % 16)) return set_error(DP_EALIGN, "transpose: operands must be 16-byte aligned");
    const int tiles = ((tb.rows[i] + 63) / 64) * ((tb.cols[i] + 63) / 64);
    if (tb.tile_start[i + 1] - tb.tile_start[i] != tiles || (i == 0 && tb.tile_start[0] != 0))
      return set_error(DP_EINVAL, "transpose: tile table does not match the shapes");
  }
  double bytes = 0.0;
  for (int i = 0; i < tb.n; ++i) bytes += 4.0 * tb.rows[i] * tb.cols[i];
  KScope ks(KK_OTHER, 0.0, bytes, s, tb.n, 0, 0);
  hipLaunchKernelGGL(transpose16_batch_kernel, dim3(tb.tile_start[tb.n]), dim3(256), 0, s, tb);
  return hipGetLastError() == hipSuccess ? DP_OK : set_error(DP_EHIP, "transpose launch failed");
}

}  // namespace dp
