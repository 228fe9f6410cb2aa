// Host side of the C ABI: descriptor validation, workspace planning, and the launch
// sequences of stage_fwd / stage_bwd / encoder_fwd_partial and of the per-layer timing
// export.  No allocation or synchronisation happens in the compute entry points.
#include "../../include/dpipe.h"
#include "dp_kernels.h"
#include "dp_errors.h"
#include "dp_host.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

namespace dp {

// Optional event recording: entries 0 .. blocks at the blocks' boundaries, then the start and (backward) the end of the pass.
struct ProfileHooks {
  std::vector<hipEvent_t>* ev = nullptr;
};

// Timing events of the profile entry points, destroyed on every way out.
struct EventSet {
  std::vector<hipEvent_t> ev;
  int create(size_t n) {
    ev.reserve(n);
    for (size_t i = 0; i < n; ++i) {
      hipEvent_t e;
      if (hipEventCreate(&e) != hipSuccess) return set_error(DP_EHIP, "hipEventCreate failed");
      ev.push_back(e);
    }
    return DP_OK;
  }
  ~EventSet() { for (auto& e : ev) (void)hipEventDestroy(e); }
};

}  // namespace dp

using namespace dp;

struct dp_stage {
  dp_stage_desc d;
  std::vector<ParamInfo> params;
  int per_block;
  size_t es;      // element size of the storage dtype
  int T, Tc;      // token rows, context rows
  // The backward runs the weight-gradient GEMMs and bias-gradient reductions (off the critical
  // path) on a second stream, forked from and joined to the caller's stream with events.  Created
  // lazily on the first stage_bwd (host objects only; no device memory).
  hipStream_t side = nullptr;
  std::vector<hipEvent_t> events;
  bool overlap = true;
  DwGroupPlan dw_plan{-1, 0, 1, 0};     // how a block's weight gradients are cut into workgroups (bf16)
  int fuse = 3;   // bit 0: GeGLU forward in the projection GEMM's epilogue; bit 1: its backward in the dx GEMM's
};

struct dp_encoder {
  dp_encoder_desc d;
  std::vector<ParamInfo> params;
  size_t es;
  // scratch of the split projections for up to (i + 1) * SPLITK_STEP rows, in every call of fewer rows too (mode 0; constant beyond the last entry)
  std::vector<size_t> splitk_bytes;
  int batch_invariant = 0;   // 1: split-K factors chosen for one sample's rows; 2: no split-K, 32x32x16 tiles only
};

namespace dp {

// ============================================================ U-Net block plan
enum { U_LN1_G, U_LN1_B, U_WQKV, U_WO1, U_BO1, U_LN2_G, U_LN2_B, U_WQ2, U_WKV2, U_WO2, U_BO2, U_LN3_G, U_LN3_B, U_W1, U_B1, U_W2, U_B2, U_COUNT };
enum { D_ADA_W, D_ADA_B, D_WQKV, D_BQKV, D_WO, D_BO, D_FC1_W, D_FC1_B, D_FC2_W, D_FC2_B, D_COUNT };

struct UnetBuf {
  void *xin, *h1, *qkv, *a1, *x1, *h2, *q2, *kv2, *a2, *x2, *h3, *u, *g;
  float *mean1, *rstd1, *lse1, *mean2, *rstd2, *lse2, *mean3, *rstd3;
};
struct DitBuf {
  void *xin, *m, *h1, *qkv, *a, *o, *x1, *h2, *f1, *f, *f2;
  float *mean1, *rstd1, *lse, *mean2, *rstd2;
};
constexpr int SIDE_MIN_BLOCKS = 3;      // stages that use the side stream: see use_side_stream
// A residual-stream gradient lives twice: fp32 (f) for the running sum and in the storage dtype (h) as a GEMM
// operand (U-Net only).  For fp32 storage both point at the same buffer.
struct GradPair { float* f; void* h; };
// What the weight-gradient work of a block reads.  It is done for the whole block at once, after (bf16 stages: possibly
// beside) the activation-gradient chain, so these buffers alternate between consecutive blocks.
struct BwdSet {
  void *dqkv, *dq2, *dkv2, *du, *dg, *dg2, *h[2];      // dg, dg2: DiT gated-branch gradients; h: storage copies of dx2, dx1
  float* ln_partial[3];                                  // column partials of the LayerNorm backward kernels; DiT: [2] of the gated branches
  float* dcond_pre;                                      // DiT: gradient of SiLU(cond) (where not all blocks' are formed together)
};
struct BwdScratch {
  float* f[2];
  void* out_h[3];                         // storage copies of the blocks' dx, taken in turn (read by the weight gradients of the next block)
  BwdSet set[2];
  void *dh, *da, *dg_raw;                 // dg_raw: unfused GeGLU backward
  float *delta, *partial; size_t partial_bytes;
  float* dkv_ws; size_t dkv_ws_bytes;     // query-split partials of the cross-attention dK/dV kernel
  void* wt;                               // transposed copies of every block's weight matrices (bf16 stages only)
  size_t ln_partial_bytes;
  void* dm;                               // DiT: every block's modulation gradients [batch, 6 d]
  float* cond_ws;                         // ... and the parts of the conditioning gradient; nullptr: block by block
};

static void plan_unet_block(Plan& p, const dp_stage& s, UnetBuf& u, bool with_xin) {
  const size_t T = s.T, Tc = s.Tc, d = s.d.d_model, inner = s.d.ff_inner, es = s.es;
  const size_t stat = (size_t)s.d.batch * s.d.n_heads * s.d.tokens * sizeof(float);
  // xin, x1, x2: the residual stream, kept in fp32 inside the stage
  u.xin = with_xin ? p.take(T * d * 4) : nullptr;
  u.h1 = p.take(T * d * es); u.qkv = p.take(T * 3 * d * es); u.a1 = p.take(T * d * es); u.x1 = p.take(T * d * 4);
  u.h2 = p.take(T * d * es); u.q2 = p.take(T * d * es); u.kv2 = p.take(Tc * 2 * d * es); u.a2 = p.take(T * d * es);
  u.x2 = p.take(T * d * 4); u.h3 = p.take(T * d * es); u.u = p.take(T * 2 * inner * es); u.g = p.take(T * inner * es);
  u.mean1 = (float*)p.take(T * 4); u.rstd1 = (float*)p.take(T * 4); u.lse1 = (float*)p.take(stat);
  u.mean2 = (float*)p.take(T * 4); u.rstd2 = (float*)p.take(T * 4); u.lse2 = (float*)p.take(stat);
  u.mean3 = (float*)p.take(T * 4); u.rstd3 = (float*)p.take(T * 4);
}
static void plan_dit_block(Plan& p, const dp_stage& s, DitBuf& u, bool with_xin) {
  const size_t T = s.T, d = s.d.d_model, ff = s.d.ff_inner, es = s.es, B = s.d.batch;
  const size_t stat = (size_t)s.d.batch * s.d.n_heads * s.d.tokens * sizeof(float);
  u.xin = with_xin ? p.take(T * d * 4) : nullptr;
  u.m = p.take(B * 6 * d * es);
  u.h1 = p.take(T * d * es); u.qkv = p.take(T * 3 * d * es); u.a = p.take(T * d * es); u.o = p.take(T * d * es);
  u.x1 = p.take(T * d * 4); u.h2 = p.take(T * d * es); u.f1 = p.take(T * ff * es); u.f = p.take(T * ff * es);
  u.f2 = p.take(T * d * es);
  u.mean1 = (float*)p.take(T * 4); u.rstd1 = (float*)p.take(T * 4); u.lse = (float*)p.take(stat);
  u.mean2 = (float*)p.take(T * 4); u.rstd2 = (float*)p.take(T * 4);
}

static GemmArgs gemm_dw(int dtype, const void* dy, int M, int N, const void* x, int K, float* dW, int accumulate, float* partial, size_t partial_bytes);

// Shapes of a block's weight gradients in the order in which they are collected: out features, in features, rows.
struct DwShape { int out, in, rows; };
static int dw_shapes(const dp_stage& s, DwShape* e) {
  const int T = s.T, d = s.d.d_model, ff = s.d.ff_inner;
  if (s.d.kind == DP_BLOCK_UNET_XATTN_GEGLU) {
    const DwShape t[] = {{d, ff, T}, {2 * ff, d, T}, {d, d, T}, {d, d, T}, {d, d, T}, {3 * d, d, T}, {2 * d, s.d.ctx_dim, s.Tc}};
    memcpy(e, t, sizeof(t));
    return 7;
  }
  const DwShape t[] = {{d, ff, T}, {ff, d, T}, {d, d, T}, {3 * d, d, T}, {6 * d, d, s.d.batch}};
  memcpy(e, t, sizeof(t));
  return 5;
}

static DwGroupPlan plan_dw(const dp_stage& s) {
  DwShape e[8];
  GemmArgs g[8];
  const int n = dw_shapes(s, e);
  for (int i = 0; i < n; ++i) g[i] = gemm_dw(s.d.dtype, nullptr, e[i].rows, e[i].out, nullptr, e[i].in, nullptr, 0, nullptr, 0);
  return gemm_dw_group_plan(g, n, 0, (size_t)-1);
}

static size_t partial_need(const dp_stage& s) {
  const int T = s.T, d = s.d.d_model, ff = s.d.ff_inner;
  size_t n = 0;
  auto mx = [&](size_t v) { n = std::max(n, v); };
  const bool unet = s.d.kind == DP_BLOCK_UNET_XATTN_GEGLU;
  DwShape e[8];
  const int ne = dw_shapes(s, e);
  for (int i = 0; i < ne; ++i) mx(gemm_splitk_ws_bytes(e[i].out, e[i].in, e[i].rows));        // where the group is not available
  if (s.es == 2) mx(s.dw_plan.ws_bytes);
  if (!unet) mx(gemm_splitk_ws_bytes(s.d.batch, d, 6 * d));
  mx(colsum_partial_bytes(T, std::max(3 * d, unet ? 2 * ff : ff)));
  mx(colsum_partial_bytes(s.d.batch, 6 * d));
  return n;
}

// Weight matrices whose activation-gradient GEMM (dx = dy W) reads a transposed copy unless reads_stored_weight() says otherwise: for each, the
// index in the block's parameter list and its shape [out features, in features].
struct WtEntry { int param, rows, cols; };
static int wt_entries(const dp_stage& s, WtEntry* e) {
  const int d = s.d.d_model, ff = s.d.ff_inner;
  if (s.d.kind == DP_BLOCK_UNET_XATTN_GEGLU) {
    const WtEntry t[] = {{U_WQKV, 3 * d, d}, {U_WO1, d, d}, {U_WQ2, d, d}, {U_WO2, d, d}, {U_W1, 2 * ff, d}, {U_W2, d, ff}};
    memcpy(e, t, sizeof(t));
    return 6;
  }
  const WtEntry t[] = {{D_WQKV, 3 * d, d}, {D_WO, d, d}, {D_FC1_W, ff, d}, {D_FC2_W, d, ff}};
  memcpy(e, t, sizeof(t));
  return 4;
}
static size_t wt_block_elems(const dp_stage& s) {
  WtEntry e[8];
  const int n = wt_entries(s, e);
  size_t t = 0;
  for (int i = 0; i < n; ++i) t += ((size_t)e[i].rows * e[i].cols + 127) / 128 * 128;
  return t;
}

static void plan_bwd_scratch(Plan& p, const dp_stage& s, BwdScratch& b) {
  const size_t T = s.T, Tc = s.Tc, d = s.d.d_model, ff = s.d.ff_inner, es = s.es, B = s.d.batch;
  const bool unet = s.d.kind == DP_BLOCK_UNET_XATTN_GEGLU;
  b = BwdScratch();
  for (int i = 0; i < 2; ++i) b.f[i] = (float*)p.take(T * d * 4);
  const bool copies = unet && es == 2;
  if (copies) for (int i = 0; i < 3 && i + 1 < s.d.n_blocks; ++i) b.out_h[i] = p.take(T * d * es);
  b.dh = p.take(T * d * es); b.da = p.take(T * d * es);
  b.delta = (float*)p.take((size_t)s.d.batch * s.d.n_heads * s.d.tokens * sizeof(float));
  b.ln_partial_bytes = ln_bwd_partial_bytes((int)T, (int)d, unet ? (int)T : s.d.tokens, !unet);
  for (int i = 0; i < 2; ++i) {
    BwdSet& t = b.set[i];
    if (i && (s.d.n_blocks < SIDE_MIN_BLOCKS || es == 4)) {
      // one stream: a block's work is done before the next block's begins, but for what a DiT block prepares for the one after it
      t = b.set[0];
      if (!unet && s.d.n_blocks > 1) {
        t.ln_partial[2] = (float*)p.take(b.ln_partial_bytes);
        if (es == 2) t.dg = p.take(T * d * es);      // (fp32: used up by then)
      }
      continue;
    }
    t.dqkv = p.take(T * 3 * d * es);
    if (copies) for (int k = 0; k < 2; ++k) t.h[k] = p.take(T * d * es);
    for (int k = 0; k < 3; ++k) t.ln_partial[k] = (float*)p.take(b.ln_partial_bytes);
    if (unet) {
      t.dq2 = p.take(T * d * es); t.dkv2 = p.take(Tc * 2 * d * es); t.du = p.take(T * 2 * ff * es);
    } else {
      t.dg = p.take(T * d * es); t.dg2 = p.take(T * d * es); t.du = p.take(T * ff * es);
      t.dcond_pre = (float*)p.take(B * d * 4);
    }
  }
  if (unet) {
    b.dkv_ws_bytes = attn_dkv_ws_bytes(s.d.batch, s.d.n_heads, s.d.ctx_tokens, s.d.d_head);
    b.dkv_ws = (float*)p.take(b.dkv_ws_bytes);
    b.dg_raw = p.take(T * ff * es);
  }
  if (!unet) {
    b.dm = p.take((size_t)s.d.n_blocks * B * 6 * d * es);
    if (cond_grad_supported(s.d.dtype, s.d.batch, s.d.d_model)) b.cond_ws = (float*)p.take(cond_grad_ws_bytes(s.d.n_blocks, s.d.batch, s.d.d_model));
  }
  b.wt = s.es == 2 ? p.take((size_t)s.d.n_blocks * wt_block_elems(s) * s.es) : nullptr;
  b.partial_bytes = partial_need(s);
  b.partial = (float*)p.take(b.partial_bytes);
}

struct StagePlan {
  std::vector<UnetBuf> ub; std::vector<DitBuf> db;
  void *pp0 = nullptr, *pp1 = nullptr, *pp2 = nullptr, *sc_in = nullptr;   // pp*: fp32 block inputs of a no-save forward
  std::vector<void*> mods;   // DiT, no-save forward: one modulation buffer per block (they are all computed up front)
  BwdScratch bs{};
  float* splitk = nullptr; size_t splitk_bytes = 0;   // partial sums of the projections that are split along the contraction (small batches)
  float* splitk_kv = nullptr; size_t splitk_kv_bytes = 0;   // ... of the context projections on the side stream, beside the others
  size_t bytes = 0;
};

// Scratch of the forward's and, with save, the backward's activation projections: enough for the split of every one of them, so that a
// projection is cut alike (and gives the same bits) whichever pass or stream it runs on.
static size_t kv_splitk_need(const dp_stage& s) { return s.es == 2 && s.Tc ? gemm_epi_splitk_ws_bytes(s.Tc, 2 * s.d.d_model, s.d.ctx_dim) : 0; }
static size_t splitk_need(const dp_stage& s, bool save) {
  if (s.es != 2) return 0;
  const int T = s.T, d = s.d.d_model, ff = s.d.ff_inner;
  const bool unet = s.d.kind == DP_BLOCK_UNET_XATTN_GEGLU;
  size_t n = kv_splitk_need(s);
  auto mx = [&](int rows, int out, int in) { n = std::max(n, gemm_epi_splitk_ws_bytes(rows, out, in)); };
  mx(T, 3 * d, d); mx(T, d, d); mx(T, unet ? 2 * ff : ff, d); mx(T, d, ff);
  if (!unet) mx(s.d.batch, 6 * d, d);
  if (save) { mx(T, d, 3 * d); mx(T, d, unet ? 2 * ff : ff); mx(T, ff, d); }
  return n;
}

static void make_plan(const dp_stage& s, void* base, bool save, StagePlan& sp) {
  Plan p(base);
  const bool unet = s.d.kind == DP_BLOCK_UNET_XATTN_GEGLU;
  const int nb = save ? s.d.n_blocks : 1;
  if (!unet) sp.sc_in = p.take((size_t)s.d.batch * s.d.d_model * s.es);
  if (unet) { sp.ub.resize(nb); for (int i = 0; i < nb; ++i) plan_unet_block(p, s, sp.ub[i], save); }
  else { sp.db.resize(nb); for (int i = 0; i < nb; ++i) plan_dit_block(p, s, sp.db[i], save); }
  sp.splitk_bytes = splitk_need(s, save);
  sp.splitk = sp.splitk_bytes ? (float*)p.take(sp.splitk_bytes) : nullptr;
  if (save && s.d.n_blocks >= SIDE_MIN_BLOCKS) sp.splitk_kv_bytes = kv_splitk_need(s);
  sp.splitk_kv = sp.splitk_kv_bytes ? (float*)p.take(sp.splitk_kv_bytes) : nullptr;
  if (save) plan_bwd_scratch(p, s, sp.bs);
  else {
    const size_t rb = (size_t)s.T * s.d.d_model * 4;
    sp.pp0 = p.take(rb); sp.pp1 = p.take(rb); sp.pp2 = p.take(rb);
    if (!unet) {
      sp.mods.resize(s.d.n_blocks);
      for (int i = 0; i < s.d.n_blocks; ++i) sp.mods[i] = p.take((size_t)s.d.batch * 6 * s.d.d_model * s.es);
    }
  }
  sp.bytes = p.off;
}

// ============================================================ small GEMM builders
static GemmArgs gemm_base(int dtype) {
  GemmArgs g;
  memset(&g, 0, sizeof(g));
  g.dtype = dtype;
  return g;
}
// y[M,N] = x[M,K] W[N,K]^T (+ bias)
static GemmArgs gemm_fwd(int dtype, const void* x, int M, int K, const void* W, int N, const void* bias, void* y) {
  GemmArgs g = gemm_base(dtype);
  g.A = x; g.B = W; g.M = M; g.N = N; g.K = K; g.lda = K; g.ldb = K; g.out = y; g.ldo = N; g.bias = bias;
  return g;
}
// dx[M,K] = dy[M,N] W[N,K]; when a transposed copy Wt[K,N] exists the product runs on it, with both operands contraction-contiguous, which the
// tiles of 256 rows need
static GemmArgs gemm_dx(int dtype, const void* dy, int M, int N, const void* W, const void* Wt, int K, void* dx) {
  GemmArgs g = gemm_base(dtype);
  g.A = dy; g.M = M; g.N = K; g.K = N; g.lda = N; g.out = dx; g.ldo = K;
  if (Wt) { g.B = Wt; g.ldb = N; g.b_mc = 0; }
  else { g.B = W; g.ldb = K; g.b_mc = 1; }
  return g;
}
// dW[N,K] (+)= dy[M,N]^T x[M,K]   (fp32)
static GemmArgs gemm_dw(int dtype, const void* dy, int M, int N, const void* x, int K, float* dW, int accumulate,
                        float* partial, size_t partial_bytes) {
  GemmArgs g = gemm_base(dtype);
  g.A = dy; g.B = x; g.M = N; g.N = K; g.K = M; g.lda = N; g.ldb = K; g.a_mc = 1; g.b_mc = 1;
  g.out_f32 = dW; g.ldo32 = K; g.accumulate = accumulate; g.splitk_ws = partial; g.splitk_ws_bytes = partial_bytes;
  return g;
}

// Fork/join bookkeeping between the caller's stream and the stage's side stream.  A "batch" is a
// group of launches on the side stream that starts after the main stream's current position
// (fork) and ends with an event; before the main stream overwrites a buffer that a batch reads,
// it waits for that batch (the side stream runs in order, so this also covers earlier batches).
struct Side {
  hipStream_t main, side;
  std::vector<hipEvent_t>* ev;
  size_t next_ev = 0;
  int issued = 0, waited = 0;
  std::vector<hipEvent_t> done;
  bool on;
  int err = DP_OK;

  hipEvent_t take() { return (*ev)[next_ev++ % ev->size()]; }
  hipStream_t begin() {                       // returns the stream the batch is launched on
    if (!on) return main;
    hipEvent_t e = take();
    if (hipEventRecord(e, main) != hipSuccess || hipStreamWaitEvent(side, e, 0) != hipSuccess) err = set_error(DP_EHIP, "stream fork failed");
    return side;
  }
  int end() {                                 // returns the batch id
    if (!on) return 0;
    hipEvent_t e = take();
    if (hipEventRecord(e, side) != hipSuccess) err = set_error(DP_EHIP, "hipEventRecord failed");
    done.push_back(e);
    return ++issued;
  }
  void wait(int batch) {                      // main stream waits for batch (and all before it)
    if (!on || batch <= waited) return;
    if (hipStreamWaitEvent(main, done[batch - 1], 0) != hipSuccess) err = set_error(DP_EHIP, "stream join failed");
    waited = batch;
  }
};

// Weight- and bias-gradient work of one block, collected and launched together (flush); where a bf16 problem does not fit the grouped kernel, every
// piece by itself.
struct BlockGrads {
  const dp_stage& s; BwdScratch& b; hipStream_t st; int acc;
  GemmArgs dw[DW_GROUP_MAX]; int n_dw = 0;
  LnBwdArgs ln[LN_REDUCE_MAX]; int n_ln = 0;
  BlockGrads(const dp_stage& s_, BwdScratch& b_, hipStream_t st_, int acc_) : s(s_), b(b_), st(st_), acc(acc_) {}

  // dW[N, K] = gy[M, N]^T x[M, K], and db[N] = column sums of gy
  int weight(const void* gy, int M, int N, const void* x, int K, float* dW, float* db) {
    GemmArgs g = gemm_dw(s.d.dtype, gy, M, N, x, K, dW, acc, b.partial, b.partial_bytes);
    g.colsum_out = db;
    dw[n_dw++] = g;
    return DP_OK;
  }
  int one(GemmArgs g, hipStream_t q) {
    float* db = g.colsum_out;
    if (db && !gemm_colsum_supported(g)) g.colsum_out = nullptr;
    DP_TRY(launch_gemm(g, q));
    return db && !g.colsum_out ? launch_colsum(s.d.dtype, g.A, g.lda, g.K, g.M, db, acc, b.partial, b.partial_bytes, q) : DP_OK;
  }
  // LayerNorm backward on the main stream; the sums of its column partials are left for later
  int layer_norm(LnBwdArgs& lb, float* partial) {
    lb.partial = partial; lb.partial_bytes = b.ln_partial_bytes; lb.defer_reduce = 1;
    DP_TRY(launch_ln_bwd(lb, st));
    ln[n_ln++] = lb;
    return DP_OK;
  }
  int flush_ln(hipStream_t q) {
    if (n_ln) DP_TRY(launch_ln_bwd_reduce(ln, n_ln, q));
    n_ln = 0;
    return DP_OK;
  }
  int flush_dw(hipStream_t q) {
    if (s.es == 4) {
      DP_TRY(launch_gemm_f32_group(dw, n_dw, q));
      n_dw = 0;
      return DP_OK;
    }
    bool group = n_dw > 0;
    for (int i = 0; i < n_dw; ++i) group = group && gemm_dw_group_supported(dw[i]);
    if (group) DP_TRY(launch_gemm_dw_group(dw, n_dw, s.dw_plan, q));
    else for (int i = 0; i < n_dw; ++i) DP_TRY(one(dw[i], q));
    n_dw = 0;
    return DP_OK;
  }
};

static AttnArgs attn_base(const dp_stage& s) {
  AttnArgs a;
  memset(&a, 0, sizeof(a));
  a.dtype = s.d.dtype; a.B = s.d.batch; a.H = s.d.n_heads; a.Nq = s.d.tokens; a.d_head = s.d.d_head;
  a.scale = 1.0f / sqrtf((float)s.d.d_head);
  return a;
}

static inline char* at(void* p, size_t elems, size_t es) { return (char*)p + elems * es; }
static inline const char* at(const void* p, size_t elems, size_t es) { return (const char*)p + elems * es; }

static int record(ProfileHooks* ph, int idx, hipStream_t st) {
  if (ph && ph->ev) {
    if (hipEventRecord((*ph->ev)[idx], st) != hipSuccess) return set_error(DP_EHIP, "hipEventRecord failed");
  }
  return DP_OK;
}

// Scratch of the projections on the caller's stream that are split along the contraction (few rows, long contractions).
struct SplitK {
  float* ws; size_t bytes;
  int launch(GemmArgs g, hipStream_t st) const { g.splitk_ws = ws; g.splitk_ws_bytes = bytes; return launch_gemm(g, st); }
};

// Whether the activation-gradient product of a weight matrix runs on the matrix as it is stored, which then needs no transposed copy.  The product as
// the block's backward forms it, with its epilogue.
static bool reads_stored_weight(const dp_stage& s, const WtEntry& e, const SplitK& sk) {
  GemmArgs g = gemm_dx(s.d.dtype, nullptr, s.T, e.rows, nullptr, nullptr, e.cols, nullptr);
  g.splitk_ws = sk.ws; g.splitk_ws_bytes = sk.bytes;
  const bool unet = s.d.kind == DP_BLOCK_UNET_XATTN_GEGLU;
  if (unet && e.param == U_W2 && (s.fuse & 2)) g.geglu = 2;
  if (!unet && e.param == D_FC2_W) { g.dact_pre = &e; g.dact_kind = s.d.gelu_tanh ? 2 : 1; }      // (only that there is one)
  return gemm_takes_stored_weight(g);
}

// ============================================================ U-Net stage
// x: fp32 block input.  y: fp32 (next block's input) unless y_is_out (storage dtype, the stage output).
// kv_side: the context K/V projection of this block was issued on the side stream as batch kv_batch
// of *kv_side (it depends on the context and the weights only); otherwise it is computed here.
// x_storage (first block): the stage input in the storage dtype; the first LayerNorm reads it and writes its rows in fp32
// into x on the way, which saves a pass over the input.
static int unet_block_fwd(const dp_stage& s, const void* const* P, const float* x, const void* ctx, void* y, bool y_is_out,
                          UnetBuf& u, const SplitK& sk, hipStream_t st, Side* kv_side = nullptr, int kv_batch = 0, const void* x_storage = nullptr) {
  const int dt = s.d.dtype, T = s.T, Tc = s.Tc, d = s.d.d_model, inner = s.d.ff_inner, dc = s.d.ctx_dim;
  const size_t es = s.es;
  auto proj = [&](const GemmArgs& g) { return sk.launch(g, st); };
  LnArgs ln; memset(&ln, 0, sizeof(ln));
  ln.dtype = dt; ln.rows = T; ln.d = d; ln.eps = s.d.ln_eps; ln.x_f32 = 1;
  // self-attention
  ln.x = x; ln.y = u.h1; ln.gamma = P[U_LN1_G]; ln.beta = P[U_LN1_B]; ln.mean = u.mean1; ln.rstd = u.rstd1;
  if (x_storage) { ln.x = x_storage; ln.x_f32 = dt == F32; ln.x32_out = const_cast<float*>(x); }
  // the LayerNorm in front of a product: inside it, or as a launch of its own
  auto normalise = [&](GemmArgs& g) -> int {
    GemmArgs n = g;
    n.A = ln.x; n.norm_x = (const float*)ln.x; n.norm_gamma = ln.gamma; n.norm_beta = ln.beta; n.norm_eps = ln.eps;
    n.norm_out = (float*)ln.y; n.norm_mean = ln.mean; n.norm_rstd = ln.rstd; n.norm_copy = ln.x32_out;
    if (!gemm_f32_norm_supported(n)) return launch_ln_fwd(ln, st);
    g = n;
    return DP_OK;
  };
  GemmArgs first[] = {gemm_fwd(dt, u.h1, T, d, P[U_WQKV], 3 * d, nullptr, u.qkv), gemm_fwd(dt, ctx, Tc, dc, P[U_WKV2], 2 * d, nullptr, u.kv2)};
  DP_TRY(normalise(first[0]));
  ln.x_f32 = 1; ln.x32_out = nullptr;
  const bool both = dt == F32 && !kv_side;      // the context's projection depends on nothing before it
  if (both) DP_TRY(launch_gemm_f32_group(first, 2, st));
  else DP_TRY(proj(first[0]));
  AttnArgs a = attn_base(s);
  a.Nk = s.d.tokens; a.q = u.qkv; a.k = at(u.qkv, d, es); a.v = at(u.qkv, 2 * d, es); a.ldq = a.ldk = a.ldv = 3 * d;
  a.o = u.a1; a.ldo = d; a.lse = u.lse1;
  DP_TRY(launch_attn_fwd(a, st));
  GemmArgs g = gemm_fwd(dt, u.a1, T, d, P[U_WO1], d, P[U_BO1], u.x1);
  g.residual = x; g.ld_res = d; g.residual_f32 = 1; g.out_fused_f32 = 1;
  DP_TRY(proj(g));
  // cross-attention
  ln.x = u.x1; ln.y = u.h2; ln.gamma = P[U_LN2_G]; ln.beta = P[U_LN2_B]; ln.mean = u.mean2; ln.rstd = u.rstd2;
  g = gemm_fwd(dt, u.h2, T, d, P[U_WQ2], d, nullptr, u.q2);
  DP_TRY(normalise(g));
  DP_TRY(proj(g));
  if (kv_side) kv_side->wait(kv_batch);
  else if (!both) DP_TRY(proj(first[1]));
  a = attn_base(s);
  a.Nk = s.d.ctx_tokens; a.q = u.q2; a.ldq = d; a.k = u.kv2; a.v = at(u.kv2, d, es); a.ldk = a.ldv = 2 * d;
  a.o = u.a2; a.ldo = d; a.lse = u.lse2;
  DP_TRY(launch_attn_fwd(a, st));
  g = gemm_fwd(dt, u.a2, T, d, P[U_WO2], d, P[U_BO2], u.x2);
  g.residual = u.x1; g.ld_res = d; g.residual_f32 = 1; g.out_fused_f32 = 1;
  DP_TRY(proj(g));
  // GeGLU feed-forward
  ln.x = u.x2; ln.y = u.h3; ln.gamma = P[U_LN3_G]; ln.beta = P[U_LN3_B]; ln.mean = u.mean3; ln.rstd = u.rstd3;
  {
    // u = h3 W1^T + b1 and g = value * gelu(gate) in one kernel where the GEMM supports it
    GemmArgs f = gemm_fwd(dt, u.h3, T, d, P[U_W1], 2 * inner, P[U_B1], u.g);
    f.ldo = inner; f.pre_out = u.u; f.ld_pre = 2 * inner; f.geglu = 1; f.geglu_inner = inner;
    const bool can_fuse = gemm_geglu_fwd_supported(f);
    if ((s.fuse & 1) && (can_fuse || gemm_f32_geglu_supported(f))) {
      DP_TRY(normalise(f));
      DP_TRY(proj(f));
    } else {
      // switching the fusion off changes no bit: the LayerNorm goes where the fused kernel has it, which adds up a row in another order than a launch of its own
      GemmArgs v = gemm_fwd(dt, u.h3, T, d, P[U_W1], 2 * inner, P[U_B1], u.u);
      if (can_fuse) v.choice_rows = -1;      // the fused kernel's order of additions
      DP_TRY(normalise(v));
      DP_TRY(proj(v));
      DP_TRY(launch_geglu_fwd(dt, u.u, u.g, T, inner, st));
    }
  }
  g = gemm_fwd(dt, u.g, T, inner, P[U_W2], d, P[U_B2], y);
  g.residual = u.x2; g.ld_res = d; g.residual_f32 = 1; g.out_fused_f32 = y_is_out ? 0 : 1;
  DP_TRY(proj(g));
  return DP_OK;
}

// dy: gradient of the block output (fp32 running sum in f[c] + a storage-dtype copy).  The fp32 sums go from f[c] to
// f[c ^ 1] (dx2), f[c] (dx1) and f[c ^ 1] (the block's dx; not for the first block of the stage, whose dx goes to
// dx_final in the storage dtype only).  `t`: the block's buffers; out_h: storage copy of the block's dx.
// dy.f == nullptr: the upstream gradient exists in the storage dtype only (dy.h, the caller's tensor)
static int unet_block_bwd(const dp_stage& s, const void* const* P, const void* const* WT, void* const* G, int acc, const void* ctx, GradPair dy, int c,
                          void* dx_final, void* out_h, UnetBuf& u, BwdScratch& b, BwdSet& t, const SplitK& sk, Side& sd, int* batch) {
  const int dt = s.d.dtype, T = s.T, Tc = s.Tc, d = s.d.d_model, inner = s.d.ff_inner, dc = s.d.ctx_dim;
  const size_t es = s.es;
  hipStream_t st = sd.main;
  auto proj = [&](const GemmArgs& g) { return sk.launch(g, st); };
  const bool f32 = es == 4;
  const GradPair dx2{b.f[c ^ 1], f32 ? (void*)b.f[c ^ 1] : t.h[0]}, dx1{b.f[c], f32 ? (void*)b.f[c] : t.h[1]}, out{b.f[c ^ 1], out_h};
  auto gf = [&](int i) { return (float*)G[i]; };
  auto set_dx = [&](LnBwdArgs& lb, GradPair p) { lb.dx32 = p.f; lb.dx = f32 ? nullptr : p.h; };
  BlockGrads bg(s, b, st, acc);
  // ---- feed-forward
  DP_TRY(bg.weight(dy.h, T, d, u.g, inner, gf(U_W2), gf(U_B2)));
  // dg = dy W2 never reaches memory: the GEMM epilogue turns it into du = [dg gelu(gate) | dg value gelu'(gate)]
  GemmArgs dg = gemm_dx(dt, dy.h, T, d, P[U_W2], WT[U_W2], inner, t.du);
  dg.ldo = 2 * inner; dg.geglu = 2; dg.geglu_inner = inner; dg.geglu_u = u.u; dg.ld_geglu = 2 * inner;
  if ((s.fuse & 2) && (dt == BF16 || gemm_f32_geglu_supported(dg))) {
    DP_TRY(proj(dg));
  } else {
    DP_TRY(proj(gemm_dx(dt, dy.h, T, d, P[U_W2], WT[U_W2], inner, b.dg_raw)));
    DP_TRY(launch_geglu_bwd(dt, b.dg_raw, u.u, t.du, T, inner, st));
  }
  DP_TRY(bg.weight(t.du, T, 2 * inner, u.h3, d, gf(U_W1), gf(U_B1)));
  DP_TRY(proj(gemm_dx(dt, t.du, T, 2 * inner, P[U_W1], WT[U_W1], d, b.dh)));
  LnBwdArgs lb; memset(&lb, 0, sizeof(lb));
  lb.dtype = dt; lb.rows = T; lb.d = d; lb.accumulate = acc;
  lb.dy = b.dh; lb.x = u.x2; lb.mean = u.mean3; lb.rstd = u.rstd3; lb.gamma = P[U_LN3_G]; set_dx(lb, dx2);
  if (dy.f) lb.dres = dy.f; else { lb.dres = dy.h; lb.dres_storage = 1; }
  lb.dgamma = gf(U_LN3_G); lb.dbeta = gf(U_LN3_B);
  DP_TRY(bg.layer_norm(lb, t.ln_partial[2]));
  // ---- cross-attention
  DP_TRY(bg.weight(dx2.h, T, d, u.a2, d, gf(U_WO2), gf(U_BO2)));
  DP_TRY(proj(gemm_dx(dt, dx2.h, T, d, P[U_WO2], WT[U_WO2], d, b.da)));
  AttnArgs a = attn_base(s);
  a.Nk = s.d.ctx_tokens; a.q = u.q2; a.ldq = d; a.k = u.kv2; a.v = at(u.kv2, d, es); a.ldk = a.ldv = 2 * d;
  a.o = u.a2; a.ldo = d; a.lse = u.lse2; a.dout = b.da; a.lddo = d; a.delta = b.delta;
  a.dq = t.dq2; a.lddq = d; a.dk = t.dkv2; a.dv = at(t.dkv2, d, es); a.lddk = a.lddv = 2 * d;
  a.dkv_ws = b.dkv_ws; a.dkv_ws_bytes = b.dkv_ws_bytes;
  DP_TRY(launch_attn_bwd(a, st));
  DP_TRY(bg.weight(t.dq2, T, d, u.h2, d, gf(U_WQ2), nullptr));
  DP_TRY(proj(gemm_dx(dt, t.dq2, T, d, P[U_WQ2], WT[U_WQ2], d, b.dh)));
  if (f32) DP_TRY(bg.flush_dw(st));      // dx1 takes the place of dy, of which fp32 stages have no copy
  lb.dy = b.dh; lb.x = u.x1; lb.mean = u.mean2; lb.rstd = u.rstd2; lb.gamma = P[U_LN2_G]; lb.dres = dx2.f; lb.dres_storage = 0; set_dx(lb, dx1);
  lb.dgamma = gf(U_LN2_G); lb.dbeta = gf(U_LN2_B);
  DP_TRY(bg.layer_norm(lb, t.ln_partial[1]));
  // ---- self-attention
  DP_TRY(bg.weight(dx1.h, T, d, u.a1, d, gf(U_WO1), gf(U_BO1)));
  DP_TRY(proj(gemm_dx(dt, dx1.h, T, d, P[U_WO1], WT[U_WO1], d, b.da)));
  a = attn_base(s);
  a.Nk = s.d.tokens; a.q = u.qkv; a.k = at(u.qkv, d, es); a.v = at(u.qkv, 2 * d, es); a.ldq = a.ldk = a.ldv = 3 * d;
  a.o = u.a1; a.ldo = d; a.lse = u.lse1; a.dout = b.da; a.lddo = d; a.delta = b.delta;
  a.dq = t.dqkv; a.dk = at(t.dqkv, d, es); a.dv = at(t.dqkv, 2 * d, es); a.lddq = a.lddk = a.lddv = 3 * d;
  DP_TRY(launch_attn_bwd(a, st));
  DP_TRY(bg.weight(t.dqkv, T, 3 * d, u.h1, d, gf(U_WQKV), nullptr));
  DP_TRY(bg.weight(t.dkv2, Tc, 2 * d, ctx, dc, gf(U_WKV2), nullptr));      // last: its contraction is the short one
  DP_TRY(proj(gemm_dx(dt, t.dqkv, T, 3 * d, P[U_WQKV], WT[U_WQKV], d, b.dh)));
  lb.dy = b.dh; lb.x = u.xin; lb.mean = u.mean1; lb.rstd = u.rstd1; lb.gamma = P[U_LN1_G]; lb.dres = dx1.f;
  if (dx_final) { lb.dx = dx_final; lb.dx32 = nullptr; } else set_dx(lb, out);
  lb.dgamma = gf(U_LN1_G); lb.dbeta = gf(U_LN1_B);
  DP_TRY(bg.layer_norm(lb, t.ln_partial[0]));
  if (f32) DP_TRY(bg.flush_dw(st));      // (as above: the next block overwrites dx1)
  hipStream_t q = sd.begin();
  DP_TRY(bg.flush_dw(q));
  DP_TRY(bg.flush_ln(q));
  *batch = sd.end();
  return sd.err;
}

// ============================================================ DiT stage
// save = false (the self-conditioning pass) skips the tensors only the backward reads.
// have_mods: the modulation vectors of this block are there already.
static int dit_block_fwd(const dp_stage& s, const void* const* P, const float* x, const void* sc_in, void* y, bool y_is_out,
                         bool save, DitBuf& u, const SplitK& sk, hipStream_t st, bool have_mods, const void* x_storage) {
  const int dt = s.d.dtype, T = s.T, d = s.d.d_model, ff = s.d.ff_inner, B = s.d.batch, N = s.d.tokens;
  const size_t es = s.es;
  auto proj = [&](const GemmArgs& g) { return sk.launch(g, st); };
  if (!have_mods) DP_TRY(proj(gemm_fwd(dt, sc_in, B, d, P[D_ADA_W], 6 * d, P[D_ADA_B], u.m)));
  LnArgs ln; memset(&ln, 0, sizeof(ln));
  ln.dtype = dt; ln.rows = T; ln.d = d; ln.eps = s.d.ln_eps; ln.mod_ld = 6 * d; ln.rows_per_batch = N; ln.x_f32 = 1;
  ln.x = x; ln.y = u.h1; ln.shift = u.m; ln.scale = at(u.m, d, es); ln.mean = u.mean1; ln.rstd = u.rstd1;
  if (x_storage) { ln.x = x_storage; ln.x_f32 = dt == F32; ln.x32_out = const_cast<float*>(x); }     // see unet_block_fwd
  DP_TRY(launch_ln_fwd(ln, st));
  ln.x_f32 = 1; ln.x32_out = nullptr;
  DP_TRY(proj(gemm_fwd(dt, u.h1, T, d, P[D_WQKV], 3 * d, P[D_BQKV], u.qkv)));
  AttnArgs a = attn_base(s);
  a.Nk = N; a.q = u.qkv; a.k = at(u.qkv, d, es); a.v = at(u.qkv, 2 * d, es); a.ldq = a.ldk = a.ldv = 3 * d;
  a.o = u.a; a.ldo = d; a.lse = u.lse;
  DP_TRY(launch_attn_fwd(a, st));
  GemmArgs g = gemm_fwd(dt, u.a, T, d, P[D_WO], d, P[D_BO], u.x1);
  g.pre_out = save ? u.o : nullptr; g.ld_pre = d; g.gate = at(u.m, 2 * d, es); g.gate_ld = 6 * d; g.rows_per_batch = N;
  g.residual = x; g.ld_res = d; g.residual_f32 = 1; g.out_fused_f32 = 1;
  DP_TRY(proj(g));
  ln.x = u.x1; ln.y = u.h2; ln.shift = at(u.m, 3 * d, es); ln.scale = at(u.m, 4 * d, es); ln.mean = u.mean2; ln.rstd = u.rstd2;
  DP_TRY(launch_ln_fwd(ln, st));
  g = gemm_fwd(dt, u.h2, T, d, P[D_FC1_W], ff, P[D_FC1_B], u.f);
  g.pre_out = save ? u.f1 : nullptr; g.ld_pre = ff; g.act = s.d.gelu_tanh ? 2 : 1;
  DP_TRY(proj(g));
  g = gemm_fwd(dt, u.f, T, ff, P[D_FC2_W], d, P[D_FC2_B], y);
  g.pre_out = save ? u.f2 : nullptr; g.ld_pre = d; g.gate = at(u.m, 5 * d, es); g.gate_ld = 6 * d; g.rows_per_batch = N;
  g.residual = u.x1; g.ld_res = d; g.residual_f32 = 1; g.out_fused_f32 = y_is_out ? 0 : 1;
  DP_TRY(proj(g));
  return DP_OK;
}

// dy: fp32, f[c] or the caller's tensor; dx1 goes to f[c ^ 1] and the block's dx back to f[c] (or, in the storage dtype, to dx_final).
static int dit_block_bwd(const dp_stage& s, bool last, const void* const* P, const void* const* WT, void* const* G, int acc, const void* cond, const void* sc_in,
                         const float* dy, int c, void* dx_final, float* d_cond, int dcond_acc, void* dm, DitBuf& u, const DitBuf* prev, BwdScratch& b, BwdSet& t, BwdSet& t_prev,
                         const SplitK& sk, Side& sd, int* batch, int prev_batch) {
  const int dt = s.d.dtype, T = s.T, d = s.d.d_model, ff = s.d.ff_inner, B = s.d.batch, N = s.d.tokens;
  const size_t es = s.es;
  hipStream_t st = sd.main;
  auto proj = [&](const GemmArgs& g) { return sk.launch(g, st); };
  float* dx1 = b.f[c ^ 1];
  auto gf = [&](int i) { return (float*)G[i]; };
  BlockGrads bg(s, b, st, acc);
  // ---- MLP branch
  LnBwdArgs lb; memset(&lb, 0, sizeof(lb));
  lb.dtype = dt; lb.rows = T; lb.d = d;
  lb.mod_ld = 6 * d; lb.rows_per_batch = N; lb.dmod_ld = 6 * d;
  // a gated branch's backward rides in the kernel that forms the gradient of its sum: the attention branch's in this block's second
  // LayerNorm, the MLP branch's in the first LayerNorm of the block after it (the last block's gradient comes from outside)
  auto gated = [&](LnBwdArgs& l, const void* m, int k, const void* branch, void* dbranch, float* partial) {
    l.gate = at(m, (size_t)k * d, es); l.gate_ld = 6 * d; l.branch = branch; l.dbranch = dbranch; l.gate_partial = partial + (k == 2 ? 0 : d);
  };
  if (last) {
    lb.dres = dy;
    gated(lb, u.m, 5, u.f2, t.dg, t.ln_partial[2]);
    DP_TRY(launch_gate_bwd(lb, st));
  }
  DP_TRY(bg.weight(t.dg, T, d, u.f, ff, gf(D_FC2_W), gf(D_FC2_B)));
  GemmArgs g = gemm_dx(dt, t.dg, T, d, P[D_FC2_W], WT[D_FC2_W], ff, t.du);
  g.dact_pre = u.f1; g.ld_dact = ff; g.dact_kind = s.d.gelu_tanh ? 2 : 1;
  DP_TRY(proj(g));
  DP_TRY(bg.weight(t.du, T, ff, u.h2, d, gf(D_FC1_W), gf(D_FC1_B)));
  DP_TRY(proj(gemm_dx(dt, t.du, T, ff, P[D_FC1_W], WT[D_FC1_W], d, b.dh)));
  lb.dy = b.dh; lb.x = u.x1; lb.mean = u.mean2; lb.rstd = u.rstd2; lb.scale = at(u.m, 4 * d, es); lb.dres = dy; lb.dx32 = dx1;
  lb.dscale = at(dm, 4 * d, es); lb.dshift = at(dm, 3 * d, es);
  gated(lb, u.m, 2, u.o, t.dg2, t.ln_partial[2]);
  DP_TRY(bg.layer_norm(lb, t.ln_partial[1]));
  // ---- attention branch
  DP_TRY(bg.weight(t.dg2, T, d, u.a, d, gf(D_WO), gf(D_BO)));
  DP_TRY(proj(gemm_dx(dt, t.dg2, T, d, P[D_WO], WT[D_WO], d, b.da)));
  AttnArgs a = attn_base(s);
  a.Nk = N; a.q = u.qkv; a.k = at(u.qkv, d, es); a.v = at(u.qkv, 2 * d, es); a.ldq = a.ldk = a.ldv = 3 * d;
  a.o = u.a; a.ldo = d; a.lse = u.lse; a.dout = b.da; a.lddo = d; a.delta = b.delta;
  a.dq = t.dqkv; a.dk = at(t.dqkv, d, es); a.dv = at(t.dqkv, 2 * d, es); a.lddq = a.lddk = a.lddv = 3 * d;
  DP_TRY(launch_attn_bwd(a, st));
  DP_TRY(bg.weight(t.dqkv, T, 3 * d, u.h1, d, gf(D_WQKV), gf(D_BQKV)));
  DP_TRY(proj(gemm_dx(dt, t.dqkv, T, 3 * d, P[D_WQKV], WT[D_WQKV], d, b.dh)));
  if (es == 4) DP_TRY(bg.flush_dw(st));      // fp32 stages have one dg: what follows prepares the next block's there
  lb.dy = b.dh; lb.x = u.xin; lb.mean = u.mean1; lb.rstd = u.rstd1; lb.scale = at(u.m, d, es); lb.dres = dx1;
  if (dx_final) { lb.dx = dx_final; lb.dx32 = nullptr; } else lb.dx32 = b.f[c];
  lb.dscale = at(dm, d, es); lb.dshift = dm;
  lb.gate = nullptr;
  if (prev) {
    sd.wait(prev_batch);      // the last to read these buffers
    gated(lb, prev->m, 5, prev->f2, t_prev.dg, t_prev.ln_partial[2]);
  }
  DP_TRY(bg.layer_norm(lb, t.ln_partial[0]));
  lb.gate = nullptr; lb.partial = t.ln_partial[2]; lb.dscale = at(dm, 2 * d, es); lb.dshift = at(dm, 5 * d, es);
  bg.ln[bg.n_ln++] = lb;      // the gates' gradients are summed with the others
  // ---- weight gradients and the conditioning path (m = SiLU(cond) W_ada^T + b_ada: d W_ada, d b_ada and d cond, accumulated over
  // the blocks in issue order, or formed for all blocks after the last); nothing on the main stream reads their results
  hipStream_t q = sd.begin();
  DP_TRY(bg.flush_ln(q));
  DP_TRY(bg.weight(dm, B, 6 * d, sc_in, d, gf(D_ADA_W), gf(D_ADA_B)));
  DP_TRY(bg.flush_dw(q));
  if (!b.cond_ws) {
    g = gemm_base(dt);
    g.A = dm; g.B = P[D_ADA_W]; g.M = B; g.N = d; g.K = 6 * d; g.lda = 6 * d; g.ldb = d; g.b_mc = 1;
    g.out_f32 = t.dcond_pre; g.ldo32 = d; g.accumulate = 0; g.splitk_ws = b.partial; g.splitk_ws_bytes = b.partial_bytes;
    DP_TRY(launch_gemm(g, q));
    DP_TRY(launch_silu_bwd(dt, t.dcond_pre, cond, d_cond, dcond_acc, (size_t)B * d, q));
  }
  *batch = sd.end();
  return sd.err;
}

// ============================================================ stage drivers
static int check_stage_call(const dp_stage* s, const void* const* params, const void* a, const void* b, const void* c,
                            const void* ws, size_t ws_bytes, int save) {
  if (!s) return set_error(DP_EINVAL, "stage handle is NULL");
  if (!params) return set_error(DP_EINVAL, "params is NULL");
  for (size_t i = 0; i < s->params.size(); ++i)
    if (int e = check_ptr(params[i], s->params[i].name.c_str())) return e;
  DP_TRY(check_ptr(a, "input tensor")); DP_TRY(check_ptr(b, "ctx_or_cond")); DP_TRY(check_ptr(c, "output tensor"));
  DP_TRY(check_ptr(ws, "workspace", 256));
  const size_t need = dp_stage_workspace_bytes(s, save);
  if (ws_bytes < need) return set_errorf(DP_EWORKSPACE, "workspace too small: %zu bytes given, %zu needed", ws_bytes, need);
  return DP_OK;
}

// The side stream carries a block's weight gradients beside the next block's backward.  The first block's have nothing beside them, what does
// run together slows each other down, and events and waits weigh on short kernels.  Step time with it against without, in %, at 1 / 2 / 3 / 5 / 8
// blocks (batch x tokens x width): U-Net 8 x 4096 x 320 +1.3 / -0.4 / -0.9 / -1.2 / -1.4; 8 x 1024 x 640 +3.1 / +1.4 / +0.8 / +0.7 / +0.6;
// 2 x 513 x 1280 +6.1 / +3.4 / +3.5 / +3.3 / +3.3; 2 x 256 x 640 +20 / +14 / +10 / +7 / +8; DiT 32 x 256 x 1152 +2.5 / +0.7 / +0.1 / +0.1 / +0.1;
// 4 x 256 x 1152 +12 / +4.6 / +2.6 / +1.1 / +0.3.  So one and two blocks never use it.  From three on it pays for many rows and costs
// stages of few: dp_stage_set_overlap(0) is for those.
static bool use_side_stream(const dp_stage& s) { return s.overlap && s.es == 2 && s.d.n_blocks >= SIDE_MIN_BLOCKS; }

static int ensure_side_stream(dp_stage* s) {
  if (s->side) return DP_OK;
  if (hipStreamCreateWithFlags(&s->side, hipStreamNonBlocking) != hipSuccess) { s->side = nullptr; return set_error(DP_EHIP, "hipStreamCreate failed"); }
  s->events.resize((size_t)s->d.n_blocks * 32 + 8);
  for (auto& e : s->events)
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return set_error(DP_EHIP, "hipEventCreate failed");
  return DP_OK;
}

static int run_stage_fwd(dp_stage* s, const void* const* params, const void* x, const void* cc, void* y, void* ws, int save,
                         hipStream_t st, ProfileHooks* ph) {
  StagePlan sp;
  make_plan(*s, ws, save != 0, sp);
  const SplitK sk{sp.splitk, sp.splitk_bytes};
  const bool unet = s->d.kind == DP_BLOCK_UNET_XATTN_GEGLU;
  const int nb = s->d.n_blocks;
  DP_TRY(record(ph, nb + 1, st));
  if (!unet) DP_TRY(launch_silu(s->d.dtype, cc, sp.sc_in, (size_t)s->d.batch * s->d.d_model, st));
  // the residual stream runs in fp32 inside the stage: widen the stage input once
  float* cur = (float*)(save ? (unet ? sp.ub[0].xin : sp.db[0].xin) : sp.pp2);
  // U-Net, saving pass (one K/V buffer per block): the context projections of all blocks run on the
  // side stream while the main stream works through block 0's self-attention
  Side sd;
  sd.main = st; sd.on = use_side_stream(*s) && unet && save != 0;
  int kv_batch = 0;
  if (sd.on) {
    DP_TRY(ensure_side_stream(s));
    sd.side = s->side; sd.ev = &s->events;
    hipStream_t q = sd.begin();
    for (int b = 0; b < nb; ++b) {
      const void* const* P = params + (size_t)b * s->per_block;
      DP_TRY(SplitK({sp.splitk_kv, sp.splitk_kv_bytes}).launch(gemm_fwd(s->d.dtype, cc, s->Tc, s->d.ctx_dim, P[U_WKV2], 2 * s->d.d_model, nullptr, sp.ub[b].kv2), q));
    }
    kv_batch = sd.end();
  }
  // DiT: the modulation vectors m = SiLU(cond) W_ada^T + b_ada of all blocks are as many rows as the batch has samples: one launch
  // reads the blocks' weights together
  bool mods = false;
  if (!unet) {
    GemmArgs g = gemm_fwd(s->d.dtype, sp.sc_in, s->d.batch, s->d.d_model, nullptr, 6 * s->d.d_model, nullptr, nullptr);
    mods = gemm_few_rows_supported(g);
    for (int b0 = 0; mods && b0 < nb; b0 += GEMM_BATCH_MAX) {
      GemmBatch bt;
      bt.n = std::min(nb - b0, GEMM_BATCH_MAX);
      for (int i = 0; i < bt.n; ++i) {
        const void* const* P = params + (size_t)(b0 + i) * s->per_block;
        bt.B[i] = P[D_ADA_W]; bt.bias[i] = P[D_ADA_B]; bt.out[i] = save ? sp.db[b0 + i].m : sp.mods[b0 + i];
      }
      DP_TRY(launch_gemm_few_rows(g, bt, st));
    }
  }
  for (int b = 0; b < nb; ++b) {
    DP_TRY(record(ph, b, st));
    const void* const* P = params + (size_t)b * s->per_block;
    const bool last = b == nb - 1;
    void* out;
    if (last) out = y;
    else if (save) out = unet ? sp.ub[b + 1].xin : sp.db[b + 1].xin;
    else out = (b & 1) ? sp.pp1 : sp.pp0;
    const int slot = save ? b : 0;
    const void* xs = b == 0 ? x : nullptr;
    if (unet) DP_TRY(unet_block_fwd(*s, P, cur, cc, out, last, sp.ub[slot], sk, st, sd.on ? &sd : nullptr, kv_batch, xs));
    else {
      DitBuf ub = sp.db[slot];
      if (!save) ub.m = sp.mods[b];
      DP_TRY(dit_block_fwd(*s, P, cur, sp.sc_in, out, last, save != 0, ub, sk, st, mods, xs));
    }
    cur = (float*)out;
  }
  sd.wait(sd.issued);
  DP_TRY(record(ph, nb, st));
  return sd.err;
}

static int run_stage_bwd(dp_stage* s, const void* const* params, const void* dy, const void* cc, void* dx, void* d_cond,
                         void* const* dparams, int acc, void* ws, hipStream_t st, ProfileHooks* ph) {
  StagePlan sp;
  make_plan(*s, ws, true, sp);
  const SplitK sk{sp.splitk, sp.splitk_bytes};
  const bool unet = s->d.kind == DP_BLOCK_UNET_XATTN_GEGLU;
  const int nb = s->d.n_blocks;
  BwdScratch& bs = sp.bs;
  Side sd;
  sd.main = st; sd.on = use_side_stream(*s);
  if (sd.on) {
    DP_TRY(ensure_side_stream(s));
    sd.side = s->side; sd.ev = &s->events;
  }
  DP_TRY(record(ph, nb + 1, st));
  // Transposed weight copies of all blocks, in one launch (a few for a long stage).
  std::vector<const void*> wt_ptrs((size_t)nb * s->per_block, nullptr);
  if (bs.wt) {
    WtEntry we[8];
    int nw = 0;
    for (int i = 0, n = wt_entries(*s, we); i < n; ++i)
      if (!reads_stored_weight(*s, we[i], sk)) we[nw++] = we[i];
    TransposeBatch tb; tb.n = 0;
    size_t off = 0;
    for (int b = 0; b < nb; ++b) {
      for (int i = 0; i < nw; ++i) {
        void* dst = at(bs.wt, off, s->es);
        transpose_batch_add(tb, params[(size_t)b * s->per_block + we[i].param], dst, we[i].rows, we[i].cols);
        wt_ptrs[(size_t)b * s->per_block + we[i].param] = dst;
        off += ((size_t)we[i].rows * we[i].cols + 127) / 128 * 128;
      }
      if (tb.n && (tb.n + nw > kTransposeMax || b == nb - 1)) { DP_TRY(launch_transpose16_batch(tb, st)); tb.n = 0; }
    }
  }
  // dy as a gradient pair: the caller's tensor as GEMM operand and, in fp32 stages, as the running sum; a widened copy only
  // where a kernel of the last block wants one (the U-Net block reads dy in the storage dtype everywhere)
  if (!unet && s->es == 2) DP_TRY(launch_cast_to_f32(s->d.dtype, dy, bs.f[1], (size_t)s->T * s->d.d_model, st));
  GradPair cur{s->es == 4 ? (float*)const_cast<void*>(dy) : (unet ? nullptr : bs.f[1]), const_cast<void*>(dy)};
  int ci = 1;   // index of the fp32 buffer that holds cur
  std::vector<const void*> dm(nb), w_ada(nb);
  int batch[2] = {0, 0};      // last side batch that reads each of the two buffer sets
  for (int i = 0; i < nb; ++i) {
    const int b = nb - 1 - i;
    DP_TRY(record(ph, i, st));
    // the set's previous user, two blocks ago; its weight gradients also were the last to read out_h[i % 3]
    sd.wait(batch[i & 1]);
    const void* const* P = params + (size_t)b * s->per_block;
    const void* const* WT = wt_ptrs.data() + (size_t)b * s->per_block;
    void* const* G = dparams + (size_t)b * s->per_block;
    void* dx_final = b == 0 ? dx : nullptr;
    if (unet) {
      DP_TRY(unet_block_bwd(*s, P, WT, G, acc, cc, cur, ci, dx_final, bs.out_h[i % 3], sp.ub[b], bs, bs.set[i & 1], sk, sd, &batch[i & 1]));
      ci ^= 1;
      cur = GradPair{bs.f[ci], s->es == 4 ? (void*)bs.f[ci] : bs.out_h[i % 3]};
    } else {
      dm[b] = at(bs.dm, (size_t)b * s->d.batch * 6 * s->d.d_model, s->es);
      w_ada[b] = P[D_ADA_W];
      DP_TRY(dit_block_bwd(*s, i == 0, P, WT, G, acc, cc, sp.sc_in, i == 0 ? cur.f : bs.f[ci], ci, dx_final, (float*)d_cond, i != 0, const_cast<void*>(dm[b]), sp.db[b],
                           b ? &sp.db[b - 1] : nullptr, bs, bs.set[i & 1], bs.set[(i + 1) & 1], sk, sd, &batch[i & 1], batch[(i + 1) & 1]));
    }
    if (ph && ph->ev) sd.wait(sd.issued);      // per-block timing: charge a block's side work to that block
  }
  DP_TRY(record(ph, nb, st));
  if (bs.cond_ws) {      // DiT: d cond from all blocks together
    hipStream_t q = sd.begin();
    DP_TRY(launch_cond_grad(dm.data(), w_ada.data(), nb, s->d.batch, s->d.d_model, bs.cond_ws, cc, (float*)d_cond, q));
    sd.end();
  }
  sd.wait(sd.issued);                          // join: everything is ordered before later work on the caller's stream
  DP_TRY(record(ph, nb + 2, st));
  return sd.err;
}

// ============================================================ encoder
enum { E_LN1_G, E_LN1_B, E_WQKV, E_BQKV, E_WO, E_BO, E_LN2_G, E_LN2_B, E_FC1_W, E_FC1_B, E_FC2_W, E_FC2_B, E_PER_LAYER };

struct EncBuf { void *h, *qkv, *a, *f; float* res; float* splitk; size_t splitk_bytes; size_t bytes; };
// Scratch of the four projections on `rows` rows whose splits are chosen for `choice_rows` rows.
static size_t encoder_splitk(const dp_encoder& e, int rows, int choice_rows) {
  const int d = e.d.d_model, ff = e.d.ff_inner;
  auto need = [&](int N, int K) { return gemm_epi_splitk_ws_bytes_for(rows, N, K, choice_rows); };
  return std::max(std::max(need(3 * d, d), need(d, d)), std::max(need(ff, d), need(d, ff)));
}
// More rows are split into fewer parts, down to none, and a workspace has to serve every smaller call: the running maximum over the rows.  On more rows
// no kind of tile has fewer tiles (those of 32 rows one more half way to a multiple of 64), which bound the parts and make them dearer, and the
// reduction of the partial sums costs more, so the parts chosen for the first row of a step of 64 are the most in it.
constexpr size_t SPLITK_STEP = 64;
static void plan_encoder_splitk(dp_encoder& e) {
  if (e.es != 2) return;
  const int d = e.d.d_model, ff = e.d.ff_inner, last = std::max(std::max(gemm_epi_split_rows(3 * d, d), gemm_epi_split_rows(d, d)), std::max(gemm_epi_split_rows(ff, d), gemm_epi_split_rows(d, ff)));
  size_t most = 0;
  for (int hi = (int)SPLITK_STEP; hi - (int)SPLITK_STEP < last; hi += (int)SPLITK_STEP) {
    most = std::max(most, encoder_splitk(e, hi, hi - (int)SPLITK_STEP + 1));
    e.splitk_bytes.push_back(most);
  }
}
static void plan_encoder(const dp_encoder& e, void* base, int samples, EncBuf& b) {
  Plan p(base);
  const size_t R = (size_t)samples * e.d.seq, d = e.d.d_model, es = e.es;
  b.h = p.take(R * d * es); b.qkv = p.take(R * 3 * d * es); b.a = p.take(R * d * es); b.f = p.take(R * e.d.ff_inner * es);
  b.res = (float*)p.take(R * d * 4);
  // partial sums of the projections that are split along the contraction on small batches
  b.splitk_bytes = e.batch_invariant == 1 ? encoder_splitk(e, (int)R, e.d.seq) : (e.splitk_bytes.empty() ? 0 : e.splitk_bytes[std::min((R + SPLITK_STEP - 1) / SPLITK_STEP, e.splitk_bytes.size()) - 1]);
  b.splitk = b.splitk_bytes ? (float*)p.take(b.splitk_bytes) : nullptr;
  b.bytes = p.off;
}

// One transformer layer on the fp32 residual stream `x` [R, d] (updated in place).  h_ready: w.h already
// holds LN1(x) (written by the previous layer's last reduction pass).  When next_gamma is given, the LayerNorm
// that follows this layer (the next layer's first, or the final one) is handed to the last projection's
// split-K reduction pass with output next_out; *next_done tells whether that pass existed and did it.
static int encoder_block(const dp_encoder& e, const void* const* P, float* x, int n, EncBuf& w, hipStream_t st, bool h_ready,
                         const void* next_gamma, const void* next_beta, void* next_out, bool* next_done) {
  const int dt = e.d.dtype, d = e.d.d_model, seq = e.d.seq, ff = e.d.ff_inner, R = n * seq;
  const size_t es = e.es;
  const bool fuse_ln = dt == DP_BF16;
  LnArgs ln; memset(&ln, 0, sizeof(ln));
  ln.dtype = dt; ln.rows = R; ln.d = d; ln.eps = e.d.ln_eps; ln.x_f32 = 1; ln.row_invariant = 1;
  const int choice_rows = e.batch_invariant == 1 ? seq : (e.batch_invariant == 2 ? -1 : 0);
  // y = LN(x) W^T: the LayerNorm inside the product where that has it, else a launch of its own unless w.h is there
  auto norm_proj = [&](GemmArgs g, const void* gamma, const void* beta, bool ready) -> int {
    g.splitk_ws = w.splitk; g.splitk_ws_bytes = w.splitk_bytes; g.choice_rows = choice_rows;
    if (!ready && gemm_norm_supported(g)) {
      g.A = x; g.norm_x = x; g.norm_gamma = gamma; g.norm_beta = beta; g.norm_eps = e.d.ln_eps;
    } else if (!ready) {
      ln.x = x; ln.y = w.h; ln.gamma = gamma; ln.beta = beta;
      DP_TRY(launch_ln_fwd(ln, st));
    }
    return launch_gemm(g, st);
  };
  DP_TRY(norm_proj(gemm_fwd(dt, w.h, R, d, P[E_WQKV], 3 * d, P[E_BQKV], w.qkv), P[E_LN1_G], P[E_LN1_B], h_ready));
  GemmArgs fc1 = gemm_fwd(dt, w.h, R, d, P[E_FC1_W], ff, P[E_FC1_B], w.f), g;
  fc1.act = 3; fc1.choice_rows = choice_rows;
  AttnArgs a; memset(&a, 0, sizeof(a));
  a.dtype = dt; a.B = n; a.H = e.d.n_heads; a.Nq = seq; a.Nk = seq; a.d_head = e.d.d_head; a.causal = e.d.causal;
  a.scale = 1.0f / sqrtf((float)e.d.d_head);
  a.q = w.qkv; a.k = at(w.qkv, d, es); a.v = at(w.qkv, 2 * d, es); a.ldq = a.ldk = a.ldv = 3 * d; a.o = w.a; a.ldo = d;
  DP_TRY(launch_attn_fwd(a, st));
  int ln_applied = 0;
  g = gemm_fwd(dt, w.a, R, d, P[E_WO], d, P[E_BO], x);
  g.splitk_ws = w.splitk; g.splitk_ws_bytes = w.splitk_bytes; g.choice_rows = choice_rows;
  g.residual = x; g.ld_res = d; g.residual_f32 = 1; g.out_fused_f32 = 1;
  if (fuse_ln && !gemm_norm_supported(fc1)) { g.ln_gamma = P[E_LN2_G]; g.ln_beta = P[E_LN2_B]; g.ln_out = w.h; g.ln_eps = e.d.ln_eps; g.ln_applied = &ln_applied; }
  DP_TRY(launch_gemm(g, st));
  DP_TRY(norm_proj(fc1, P[E_LN2_G], P[E_LN2_B], ln_applied != 0));
  ln_applied = 0;
  g = gemm_fwd(dt, w.f, R, ff, P[E_FC2_W], d, P[E_FC2_B], x);
  g.splitk_ws = w.splitk; g.splitk_ws_bytes = w.splitk_bytes; g.choice_rows = choice_rows;
  g.residual = x; g.ld_res = d; g.residual_f32 = 1; g.out_fused_f32 = 1;
  if (fuse_ln && next_gamma) { g.ln_gamma = next_gamma; g.ln_beta = next_beta; g.ln_out = next_out; g.ln_eps = e.d.ln_eps; g.ln_applied = &ln_applied; }
  DP_TRY(launch_gemm(g, st));
  if (next_done) *next_done = ln_applied != 0;
  return DP_OK;
}

// Layers [lb, le) on samples [off, off + n).  `hidden` holds the state in the storage dtype between
// calls; inside a call the residual stream of consecutive transformer layers stays in fp32.
// When ev is given, ev[l - lb] is recorded before layer l and ev[le - lb] at the end.
static int encoder_run(const dp_encoder& e, const void* const* params, const int32_t* ids, void* hidden, int lb, int le, int off,
                       int n, EncBuf& w, hipStream_t st, std::vector<hipEvent_t>* ev) {
  const int dt = e.d.dtype, d = e.d.d_model, seq = e.d.seq, R = n * seq, nl = e.d.n_layers;
  void* x = at(hidden, (size_t)off * seq * d, e.es);
  auto mark = [&](int l) -> int {
    if (ev && hipEventRecord((*ev)[l - lb], st) != hipSuccess) return set_error(DP_EHIP, "hipEventRecord failed");
    return DP_OK;
  };
  int l = lb;
  const int tl_end = std::min(le, nl + 1);
  const bool embed = l == 0, blocks = std::max(l, 1) < tl_end;
  if (embed) {      // in fp32 at once where layers follow
    DP_TRY(mark(0));
    DP_TRY(launch_embed(dt, ids + (size_t)off * seq, params[0], params[1], x, blocks ? w.res : nullptr, R, seq, d, e.d.vocab, st));
    ++l;
  }
  const bool final_ln = le == nl + 2;
  bool final_done = false;
  if (blocks) {
    DP_TRY(mark(l));
    if (!embed) DP_TRY(launch_cast_to_f32(dt, x, w.res, (size_t)R * d, st));
    // A layer's last reduction pass may also compute the LayerNorm that follows it (the next layer's first, or
    // the final one straight into `hidden`), also while layers are being timed one by one: the cost profile
    // then describes the launch sequence of an ordinary call, with a folded LayerNorm charged to the layer
    // whose reduction pass computes it.
    bool h_ready = false;
    for (; l < tl_end; ++l) {
      if (l != (lb == 0 ? 1 : lb)) DP_TRY(mark(l));
      const void* const* P = params + 2 + (size_t)(l - 1) * E_PER_LAYER;
      const void *ng = nullptr, *nb = nullptr;
      void* nout = nullptr;
      if (l + 1 < tl_end) { ng = P[E_PER_LAYER + E_LN1_G]; nb = P[E_PER_LAYER + E_LN1_B]; nout = w.h; }
      else if (l == nl && final_ln) { ng = params[2 + (size_t)nl * E_PER_LAYER]; nb = params[2 + (size_t)nl * E_PER_LAYER + 1]; nout = x; }
      bool done = false;
      DP_TRY(encoder_block(e, P, w.res, n, w, st, h_ready, ng, nb, nout, &done));
      h_ready = done && l + 1 < tl_end;
      final_done = done && l == nl && final_ln;
    }
    if (!final_ln) DP_TRY(launch_cast_from_f32(dt, w.res, x, (size_t)R * d, st));
  }
  if (final_ln && final_done) DP_TRY(mark(nl + 1));     // folded into the last layer's reduction pass: its own span is empty
  if (final_ln && !final_done) {
    DP_TRY(mark(nl + 1));
    const void* const* P = params + 2 + (size_t)nl * E_PER_LAYER;
    LnArgs ln; memset(&ln, 0, sizeof(ln));
    ln.dtype = dt; ln.rows = R; ln.d = d; ln.eps = e.d.ln_eps; ln.row_invariant = 1;
    ln.x = blocks ? (const void*)w.res : (const void*)x; ln.x_f32 = blocks ? 1 : 0; ln.y = x; ln.gamma = P[0]; ln.beta = P[1];
    DP_TRY(launch_ln_fwd(ln, st));
  }
  if (ev && hipEventRecord((*ev)[le - lb], st) != hipSuccess) return set_error(DP_EHIP, "hipEventRecord failed");
  return DP_OK;
}

static int check_encoder_call(const dp_encoder* e, const void* const* params, const int32_t* ids, const void* hidden,
                              int global_batch, int lb, int le, int off, int n, const void* ws, size_t ws_bytes) {
  if (!e) return set_error(DP_EINVAL, "encoder handle is NULL");
  if (!params) return set_error(DP_EINVAL, "params is NULL");
  for (size_t i = 0; i < e->params.size(); ++i)
    if (int err = check_ptr(params[i], e->params[i].name.c_str())) return err;
  DP_TRY(check_ptr(ids, "ids", 4)); DP_TRY(check_ptr(hidden, "hidden")); DP_TRY(check_ptr(ws, "workspace", 256));
  if (global_batch <= 0 || off < 0 || n < 0 || (long)off + n > global_batch)
    return set_errorf(DP_EINVAL, "sample range [%d, %d) outside the global batch of %d", off, off + n, global_batch);
  if (lb < 0 || le > e->d.n_layers + 2 || lb >= le) return set_errorf(DP_EINVAL, "layer range [%d, %d) invalid (0..%d)", lb, le, e->d.n_layers + 2);
  if ((long)n * e->d.n_heads > 65535) return set_error(DP_EUNSUPPORTED, "num_samples * n_heads exceeds 65535");
  const size_t need = dp_encoder_workspace_bytes(e, n);
  if (ws_bytes < need) return set_errorf(DP_EWORKSPACE, "workspace too small: %zu bytes given, %zu needed", ws_bytes, need);
  return DP_OK;
}

}  // namespace dp

// ============================================================ extern "C"
extern "C" {


int dp_stage_create(const dp_stage_desc* desc, dp_stage** out) {
  if (!desc || !out) return set_error(DP_EINVAL, "dp_stage_create: NULL argument");
  const dp_stage_desc& d = *desc;
  if (d.kind != DP_BLOCK_UNET_XATTN_GEGLU && d.kind != DP_BLOCK_DIT_ADALN_ZERO) return set_error(DP_EINVAL, "unknown block kind");
  if (d.dtype != DP_F32 && d.dtype != DP_BF16) return set_error(DP_EINVAL, "unknown dtype");
  if (d.n_blocks <= 0 || d.batch <= 0 || d.tokens <= 0 || d.d_model <= 0 || d.n_heads <= 0 || d.d_head <= 0 || d.ff_inner <= 0)
    return set_error(DP_EINVAL, "sizes must be positive");
  if ((long)d.n_heads * d.d_head != d.d_model) return set_error(DP_EINVAL, "d_model must equal n_heads * d_head");
  if (!(d.ln_eps > 0.f)) return set_error(DP_EINVAL, "ln_eps must be positive");
  const bool unet = d.kind == DP_BLOCK_UNET_XATTN_GEGLU;
  if (unet && (d.ctx_tokens <= 0 || d.ctx_dim <= 0)) return set_error(DP_EINVAL, "ctx_tokens and ctx_dim must be positive");
  if ((long)d.batch * d.tokens > (1L << 30) || (long)d.batch * d.n_heads > 65535)
    return set_error(DP_EUNSUPPORTED, "batch * tokens or batch * heads too large");
  if (d.n_blocks > 4096) return set_error(DP_EUNSUPPORTED, "too many blocks");
  const int V = d.dtype == DP_BF16 ? 8 : 4;
  if (d.d_model % V || d.ff_inner % V || d.d_head % (d.dtype == DP_BF16 ? 8 : 1) || (unet && d.ctx_dim % V))
    return set_errorf(DP_EUNSUPPORTED, "d_model, ff_inner, ctx_dim (and d_head for bf16) must be multiples of %d", V);
  if (d.dtype == DP_BF16 && (d.d_head > 96 || d.d_model > 2048)) return set_error(DP_EUNSUPPORTED, "bf16 path: d_head <= 96, d_model <= 2048");
  if (d.dtype == DP_F32 && (d.d_head > 256 || d.d_model > 1024 || d.tokens > 7500 || (unet && d.ctx_tokens > 7500)))
    return set_error(DP_EUNSUPPORTED, "fp32 path: d_head <= 256, d_model <= 1024, tokens <= 7500");
  dp_stage* s = new (std::nothrow) dp_stage();
  if (!s) return set_error(DP_EINVAL, "out of host memory");
  s->d = d;
  s->es = dtype_size(d.dtype);
  s->T = d.batch * d.tokens;
  s->Tc = unet ? d.batch * d.ctx_tokens : 0;
  const int64_t dm = d.d_model, inner = d.ff_inner, dc = d.ctx_dim;
  struct Spec { const char* n; int64_t r, c; };
  std::vector<Spec> per;
  if (unet) {
    per = {{"ln1_g", dm, 0}, {"ln1_b", dm, 0}, {"attn1_wqkv", 3 * dm, dm}, {"attn1_wo", dm, dm}, {"attn1_bo", dm, 0},
           {"ln2_g", dm, 0}, {"ln2_b", dm, 0}, {"attn2_wq", dm, dm}, {"attn2_wkv", 2 * dm, dc}, {"attn2_wo", dm, dm},
           {"attn2_bo", dm, 0}, {"ln3_g", dm, 0}, {"ln3_b", dm, 0}, {"ff_w1", 2 * inner, dm}, {"ff_b1", 2 * inner, 0},
           {"ff_w2", dm, inner}, {"ff_b2", dm, 0}};
  } else {
    per = {{"ada_w", 6 * dm, dm}, {"ada_b", 6 * dm, 0}, {"attn_wqkv", 3 * dm, dm}, {"attn_bqkv", 3 * dm, 0}, {"attn_wo", dm, dm},
           {"attn_bo", dm, 0}, {"fc1_w", inner, dm}, {"fc1_b", inner, 0}, {"fc2_w", dm, inner}, {"fc2_b", dm, 0}};
  }
  s->per_block = (int)per.size();
  if (s->es == 2) s->dw_plan = plan_dw(*s);
  for (int b = 0; b < d.n_blocks; ++b)
    for (auto& sp : per) s->params.push_back({"block" + std::to_string(b) + "." + sp.n, sp.r, sp.c});
  *out = s;
  return DP_OK;
}

void dp_stage_destroy(dp_stage* st) {
  if (!st) return;
  for (auto& e : st->events) (void)hipEventDestroy(e);
  if (st->side) (void)hipStreamDestroy(st->side);
  delete st;
}

int dp_stage_set_overlap(dp_stage* st, int enabled) {
  if (!st) return set_error(DP_EINVAL, "stage handle is NULL");
  st->overlap = enabled != 0;
  return DP_OK;
}

int dp_encoder_set_batch_invariant(dp_encoder* enc, int mode) {
  if (!enc) return set_error(DP_EINVAL, "encoder handle is NULL");
  if (mode < 0 || mode > 2) return set_error(DP_EINVAL, "batch-invariant mode must be 0, 1 or 2");
  enc->batch_invariant = mode;
  return DP_OK;
}

int dp_stage_set_fusion(dp_stage* st, int mask) {
  if (!st) return set_error(DP_EINVAL, "stage handle is NULL");
  if (mask < 0 || mask > 3) return set_error(DP_EINVAL, "fusion mask out of range");
  st->fuse = mask;
  return DP_OK;
}

int dp_stage_param_count(const dp_stage* st) { return st ? (int)st->params.size() : set_error(DP_EINVAL, "stage handle is NULL"); }

int dp_stage_param_shape(const dp_stage* st, int idx, int64_t shape[2], const char** name) {
  if (!st || !shape) return set_error(DP_EINVAL, "dp_stage_param_shape: NULL argument");
  if (idx < 0 || idx >= (int)st->params.size()) return set_error(DP_EINVAL, "parameter index out of range");
  shape[0] = st->params[idx].rows; shape[1] = st->params[idx].cols;
  if (name) *name = st->params[idx].name.c_str();
  return DP_OK;
}

size_t dp_stage_workspace_bytes(const dp_stage* st, int save_for_bwd) {
  if (!st) return 0;
  StagePlan sp;
  make_plan(*st, nullptr, save_for_bwd != 0, sp);
  return sp.bytes;
}

int stage_fwd(dp_stage* st, const void* const* params, const void* x, const void* ctx_or_cond, void* y, void* workspace,
              size_t workspace_bytes, int save_for_bwd, void* hip_stream) {
  DP_TRY(check_stage_call(st, params, x, ctx_or_cond, y, workspace, workspace_bytes, save_for_bwd != 0));
  return run_stage_fwd(st, params, x, ctx_or_cond, y, workspace, save_for_bwd != 0, (hipStream_t)hip_stream, nullptr);
}

int stage_bwd(dp_stage* st, const void* const* params, const void* dy, const void* ctx_or_cond, void* dx, void* d_cond,
              void* const* dparams, int accumulate, void* workspace, size_t workspace_bytes, void* hip_stream) {
  DP_TRY(check_stage_call(st, params, dy, ctx_or_cond, dx, workspace, workspace_bytes, 1));
  if (!dparams) return set_error(DP_EINVAL, "dparams is NULL");
  for (size_t i = 0; i < st->params.size(); ++i)
    if (int e = check_ptr(dparams[i], "parameter gradient")) return e;
  if (st->d.kind == DP_BLOCK_DIT_ADALN_ZERO) DP_TRY(check_ptr(d_cond, "d_cond"));
  return run_stage_bwd(st, params, dy, ctx_or_cond, dx, d_cond, dparams, accumulate != 0, workspace, (hipStream_t)hip_stream, nullptr);
}

int dp_encoder_create(const dp_encoder_desc* desc, dp_encoder** out) {
  if (!desc || !out) return set_error(DP_EINVAL, "dp_encoder_create: NULL argument");
  const dp_encoder_desc& d = *desc;
  if (d.dtype != DP_F32 && d.dtype != DP_BF16) return set_error(DP_EINVAL, "unknown dtype");
  if (d.n_layers <= 0 || d.d_model <= 0 || d.n_heads <= 0 || d.d_head <= 0 || d.seq <= 0 || d.vocab <= 0 || d.ff_inner <= 0)
    return set_error(DP_EINVAL, "sizes must be positive");
  if ((long)d.n_heads * d.d_head != d.d_model) return set_error(DP_EINVAL, "d_model must equal n_heads * d_head");
  if (!(d.ln_eps > 0.f)) return set_error(DP_EINVAL, "ln_eps must be positive");
  if (d.causal != 0 && d.causal != 1) return set_error(DP_EINVAL, "causal must be 0 or 1");
  const int V = d.dtype == DP_BF16 ? 8 : 4;
  if (d.d_model % V || d.ff_inner % V || d.d_head % (d.dtype == DP_BF16 ? 8 : 1))
    return set_errorf(DP_EUNSUPPORTED, "d_model, ff_inner (and d_head for bf16) must be multiples of %d", V);
  if (d.dtype == DP_BF16 && (d.d_head > 96 || d.d_model > 2048)) return set_error(DP_EUNSUPPORTED, "bf16 path: d_head <= 96, d_model <= 2048");
  if (d.dtype == DP_F32 && (d.d_head > 256 || d.d_model > 1024 || d.seq > 7500)) return set_error(DP_EUNSUPPORTED, "fp32 path: d_head <= 256, d_model <= 1024, seq <= 7500");
  if (d.n_layers > 4096) return set_error(DP_EUNSUPPORTED, "too many layers");
  dp_encoder* e = new (std::nothrow) dp_encoder();
  if (!e) return set_error(DP_EINVAL, "out of host memory");
  e->d = d;
  e->es = dtype_size(d.dtype);
  const int64_t dm = d.d_model, ff = d.ff_inner;
  e->params.push_back({"tok_emb", d.vocab, dm});
  e->params.push_back({"pos_emb", d.seq, dm});
  struct Spec { const char* n; int64_t r, c; };
  const Spec per[] = {{"ln1_g", dm, 0}, {"ln1_b", dm, 0}, {"wqkv", 3 * dm, dm}, {"bqkv", 3 * dm, 0}, {"wo", dm, dm}, {"bo", dm, 0},
                      {"ln2_g", dm, 0}, {"ln2_b", dm, 0}, {"fc1_w", ff, dm}, {"fc1_b", ff, 0}, {"fc2_w", dm, ff}, {"fc2_b", dm, 0}};
  for (int l = 0; l < d.n_layers; ++l)
    for (auto& sp : per) e->params.push_back({"layer" + std::to_string(l) + "." + sp.n, sp.r, sp.c});
  e->params.push_back({"lnf_g", dm, 0});
  e->params.push_back({"lnf_b", dm, 0});
  try { plan_encoder_splitk(*e); }
  catch (...) { delete e; return set_error(DP_EINVAL, "out of host memory"); }
  *out = e;
  return DP_OK;
}

void dp_encoder_destroy(dp_encoder* enc) { delete enc; }
int dp_encoder_param_count(const dp_encoder* enc) { return enc ? (int)enc->params.size() : set_error(DP_EINVAL, "encoder handle is NULL"); }
int dp_encoder_param_shape(const dp_encoder* enc, int idx, int64_t shape[2], const char** name) {
  if (!enc || !shape) return set_error(DP_EINVAL, "dp_encoder_param_shape: NULL argument");
  if (idx < 0 || idx >= (int)enc->params.size()) return set_error(DP_EINVAL, "parameter index out of range");
  shape[0] = enc->params[idx].rows; shape[1] = enc->params[idx].cols;
  if (name) *name = enc->params[idx].name.c_str();
  return DP_OK;
}
size_t dp_encoder_workspace_bytes(const dp_encoder* enc, int max_samples) {
  if (!enc || max_samples <= 0) return 0;
  EncBuf b;
  plan_encoder(*enc, nullptr, max_samples, b);
  return b.bytes;
}

int encoder_fwd_partial(dp_encoder* enc, const void* const* params, const int32_t* ids, void* hidden, int global_batch,
                        int layer_begin, int layer_end, int sample_offset, int num_samples, void* workspace,
                        size_t workspace_bytes, void* hip_stream) {
  DP_TRY(check_encoder_call(enc, params, ids, hidden, global_batch, layer_begin, layer_end, sample_offset, num_samples, workspace, workspace_bytes));
  if (num_samples == 0) return DP_OK;   // an empty slice is valid and touches nothing
  EncBuf w;
  plan_encoder(*enc, workspace, num_samples, w);
  return encoder_run(*enc, params, ids, hidden, layer_begin, layer_end, sample_offset, num_samples, w, (hipStream_t)hip_stream, nullptr);
}

int dp_stage_profile(dp_stage* st, const void* const* params, const void* x, const void* ctx_or_cond, void* y, const void* dy,
                     void* dx, void* d_cond, void* const* dparams, void* workspace, size_t workspace_bytes, int reps,
                     dp_layer_cost* rows, int max_rows, int* n_rows, void* hip_stream) {
  DP_TRY(check_stage_call(st, params, x, ctx_or_cond, y, workspace, workspace_bytes, 1));
  DP_TRY(check_ptr(dy, "dy")); DP_TRY(check_ptr(dx, "dx"));
  if (!dparams || !rows || !n_rows) return set_error(DP_EINVAL, "dp_stage_profile: NULL argument");
  for (size_t i = 0; i < st->params.size(); ++i)
    if (int e = check_ptr(dparams[i], "parameter gradient")) return e;
  if (st->d.kind == DP_BLOCK_DIT_ADALN_ZERO) DP_TRY(check_ptr(d_cond, "d_cond"));
  const int nb = st->d.n_blocks;
  if (reps < 1 || max_rows < nb) return set_error(DP_EINVAL, "dp_stage_profile: reps < 1 or too few rows");
  hipStream_t s = (hipStream_t)hip_stream;
  EventSet esf, esb;
  DP_TRY(esf.create(nb + 3)); DP_TRY(esb.create(nb + 3));
  std::vector<hipEvent_t>& ef = esf.ev;
  std::vector<hipEvent_t>& eb = esb.ev;
  std::vector<std::vector<float>> tf(nb), tb(nb);
  int rc = DP_OK;
  for (int r = 0; r < reps && rc == DP_OK; ++r) {
    ProfileHooks hf, hb;
    hf.ev = &ef; hb.ev = &eb;
    rc = run_stage_fwd(st, params, x, ctx_or_cond, y, workspace, 1, s, &hf);
    if (rc == DP_OK) rc = run_stage_bwd(st, params, dy, ctx_or_cond, dx, d_cond, dparams, 0, workspace, s, &hb);
    if (rc == DP_OK && hipStreamSynchronize(s) != hipSuccess) rc = set_error(DP_EHIP, "hipStreamSynchronize failed");
    auto ms = [&](const std::vector<hipEvent_t>& e, int from, int to) {
      float v = 0.f;
      if (rc == DP_OK && hipEventElapsedTime(&v, e[from], e[to]) != hipSuccess) rc = set_error(DP_EHIP, "hipEventElapsedTime failed");
      return v;
    };
    // what is done for all blocks together, before the first and after the last of them, goes to each in equal parts
    const float f_all = ms(ef, nb + 1, 0) / (float)nb, b_all = (ms(eb, nb + 1, 0) + ms(eb, nb, nb + 2)) / (float)nb;
    for (int b = 0; b < nb && rc == DP_OK; ++b) {
      tf[b].push_back(ms(ef, b, b + 1) + f_all);
      tb[b].push_back(ms(eb, nb - 1 - b, nb - b) + b_all);      // backward runs blocks in reverse: event i brackets block nb-1-i
    }
  }
  if (rc != DP_OK) return rc;
  const int64_t act = (int64_t)st->T * st->d.d_model * st->es;
  for (int b = 0; b < nb; ++b) {
    int64_t gbytes = 0;
    for (int i = 0; i < st->per_block; ++i) {
      const ParamInfo& pi = st->params[(size_t)b * st->per_block + i];
      gbytes += pi.rows * (pi.cols ? pi.cols : 1) * 4;
    }
    rows[b] = dp_layer_cost{0, b, st->d.batch, median(tf[b]), median(tb[b]), act, act, act, gbytes};
  }
  *n_rows = nb;
  return DP_OK;
}

int dp_encoder_profile(dp_encoder* enc, const void* const* params, const int32_t* ids, void* hidden, int global_batch,
                       const int* batches, int n_batches, int reps, void* workspace, size_t workspace_bytes,
                       dp_layer_cost* rows, int max_rows, int* n_rows, void* hip_stream) {
  if (!enc || !batches || !rows || !n_rows || n_batches <= 0 || reps < 1) return set_error(DP_EINVAL, "dp_encoder_profile: bad argument");
  const int nl = enc->d.n_layers + 2;
  if (max_rows < nl * n_batches) return set_error(DP_EINVAL, "dp_encoder_profile: too few rows");
  for (int i = 0; i < n_batches; ++i) {
    if (batches[i] < 1) return set_error(DP_EINVAL, "dp_encoder_profile: batch sizes must be positive");
    DP_TRY(check_encoder_call(enc, params, ids, hidden, global_batch, 0, nl, 0, batches[i], workspace, workspace_bytes));
  }
  hipStream_t s = (hipStream_t)hip_stream;
  EventSet es;
  DP_TRY(es.create(nl + 1));
  std::vector<hipEvent_t>& ev = es.ev;
  int rc = DP_OK, out = 0;
  for (int bi = 0; bi < n_batches && rc == DP_OK; ++bi) {
    const int n = batches[bi];
    EncBuf w;
    plan_encoder(*enc, workspace, n, w);
    std::vector<std::vector<float>> t(nl);
    for (int r = 0; r < reps && rc == DP_OK; ++r) {
      rc = encoder_run(*enc, params, ids, hidden, 0, nl, 0, n, w, s, &ev);
      if (rc == DP_OK && hipStreamSynchronize(s) != hipSuccess) rc = set_error(DP_EHIP, "hipStreamSynchronize failed");
      for (int l = 0; l < nl && rc == DP_OK; ++l) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, ev[l], ev[l + 1]) != hipSuccess) rc = set_error(DP_EHIP, "hipEventElapsedTime failed");
        t[l].push_back(ms);
      }
    }
    const int64_t act = (int64_t)n * enc->d.seq * enc->d.d_model * enc->es;
    for (int l = 0; l < nl && rc == DP_OK; ++l) rows[out++] = dp_layer_cost{1, l, n, median(t[l]), 0.f, act, act, 0, 0};
  }
  if (rc != DP_OK) return rc;
  *n_rows = out;
  return DP_OK;
}

size_t dp_op_gemm_workspace_bytes(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0) return 0;
  return std::max(gemm_splitk_ws_bytes(M, N, K), gemm_epi_splitk_ws_bytes(M, N, K));
}

int dp_op_gemm(int dtype, const void* A, int lda, int a_kmajor, const void* B, int ldb, int b_kmajor, int M, int N, int K,
               const void* bias, void* C, int ldc, int out_is_f32, int accumulate, void* workspace, size_t workspace_bytes,
               int tile_cfg, void* hip_stream) {
  if (dtype != DP_F32 && dtype != DP_BF16) return set_error(DP_EINVAL, "unknown dtype");
  DP_TRY(check_ptr(A, "A")); DP_TRY(check_ptr(B, "B")); DP_TRY(check_ptr(C, "C"));
  GemmArgs g;
  memset(&g, 0, sizeof(g));
  g.dtype = dtype; g.A = A; g.B = B; g.M = M; g.N = N; g.K = K; g.lda = lda; g.ldb = ldb; g.a_mc = a_kmajor != 0; g.b_mc = b_kmajor != 0;
  if (out_is_f32) {
    if (bias) return set_error(DP_EUNSUPPORTED, "dp_op_gemm: bias with fp32 output is not supported");
    g.out_f32 = (float*)C; g.ldo32 = ldc; g.accumulate = accumulate != 0;
  } else {
    g.out = C; g.ldo = ldc; g.bias = bias;
  }
  g.splitk_ws = (float*)workspace; g.splitk_ws_bytes = workspace ? workspace_bytes : 0;
  g.force_cfg = tile_cfg;
  return launch_gemm(g, (hipStream_t)hip_stream);
}

int dp_op_quantize_fp8(const void* x, int ldx, void* q, int ldq, int rows, int cols, float scale, void* hip_stream) {
  if (!(scale > 0.f) || !(scale < INFINITY)) return set_error(DP_EINVAL, "dp_op_quantize_fp8: the scale must be positive and finite");
  return launch_quantize_fp8(x, ldx, q, ldq, rows, cols, 1.0f / scale, (hipStream_t)hip_stream);
}

int dp_op_gemm_fp8(const void* A, int lda, const void* B, int ldb, int M, int N, int K, float out_scale, const void* bias, void* C,
                   int ldc, void* hip_stream) {
  Fp8GemmArgs a{A, lda, B, ldb, M, N, K, out_scale, bias, C, ldc};
  return launch_gemm_fp8(a, (hipStream_t)hip_stream);
}

int dp_op_attention_fwd(int dtype, int B, int H, int Nq, int Nk, int d_head, int causal, float scale, const void* q, int ldq,
                        const void* k, int ldk, const void* v, int ldv, void* o, int ldo, float* lse, void* hip_stream) {
  if (dtype != DP_F32 && dtype != DP_BF16) return set_error(DP_EINVAL, "unknown dtype");
  AttnArgs a;
  memset(&a, 0, sizeof(a));
  a.dtype = dtype; a.B = B; a.H = H; a.Nq = Nq; a.Nk = Nk; a.d_head = d_head; a.causal = causal != 0; a.scale = scale;
  a.q = q; a.ldq = ldq; a.k = k; a.ldk = ldk; a.v = v; a.ldv = ldv; a.o = o; a.ldo = ldo; a.lse = lse;
  return launch_attn_fwd(a, (hipStream_t)hip_stream);
}

int dp_op_attention_bwd(int dtype, int B, int H, int Nq, int Nk, int d_head, float scale, const void* q, int ldq, const void* k,
                        int ldk, const void* v, int ldv, const void* o, int ldo, const float* lse, const void* d_o, int lddo,
                        float* delta, void* dq, int lddq, void* dk, int lddk, void* dv, int lddv, void* hip_stream) {
  if (dtype != DP_F32 && dtype != DP_BF16) return set_error(DP_EINVAL, "unknown dtype");
  AttnArgs a;
  memset(&a, 0, sizeof(a));
  a.dtype = dtype; a.B = B; a.H = H; a.Nq = Nq; a.Nk = Nk; a.d_head = d_head; a.scale = scale;
  a.q = q; a.ldq = ldq; a.k = k; a.ldk = ldk; a.v = v; a.ldv = ldv; a.o = const_cast<void*>(o); a.ldo = ldo;
  a.lse = const_cast<float*>(lse); a.dout = d_o; a.lddo = lddo; a.delta = delta;
  a.dq = dq; a.lddq = lddq; a.dk = dk; a.lddk = lddk; a.dv = dv; a.lddv = lddv;
  return launch_attn_bwd(a, (hipStream_t)hip_stream);
}

}  // extern "C"
