// Context, arena carve-up and the orchestration of the hot path: a worker's local round
// (inner loop of Alg. 1: forward, backward, AdamW) on that worker's stream, and the server's
// sync() step (pseudo-gradient, Delayed Nesterov of Alg. 3, restart of Alg. 2) ordered
// against the workers with events.
#include "common.h"
#include <algorithm>
#include <atomic>
#include <math.h>
#include <stdio.h>
#include <string.h>
#include <mutex>
#include <new>
#include <vector>

using namespace als;

namespace {

struct Worker {
  float *theta, *start, *adam_m, *adam_v, *grad;
  bf16* lp;
  std::vector<float*> x, xm, rstd1, rstd2, lse;
  std::vector<void*> a, qkv, o, b, u, gl;
  void* xf; float* rstdf; float* logits; void* dlogits; float* loss_row;  // logits: fp32 mode only
  float *dxa, *dxb, *dtmp, *Dbuf, *partial;
  void *dx_lp, *dff, *d_o, *dqkv;
  // pinned; a step writes its loss there itself: a copy per call cost the host as much as several launches
  float* losses_host; float* losses_dev;   // losses_dev: its address on the device
  int32_t *sort_offset, *sort_rank, *sort_pos;
  float* splitk_ws; size_t splitk_bytes;
  float* head_ws; size_t head_ws_bytes;   // split-K scratch of the output matrix's input gradient
  // Output gradients that the weight-gradient products read (dY), per layer: of the block output
  // (for W2), of the FFN pre-activation (W1), of the attention block output (Wo), of q/k/v (Wqkv).
  // With the grouped launch every layer keeps its own until the end of the backward pass; otherwise
  // all layers point at the same four buffers.
  std::vector<void*> dy2, dy1, dyo, dyqkv;
  DwProblem* dw_probs_dev; DwItem* dw_items_dev; DwSplitTile* dw_split_dev; float* dw_partial;
  std::vector<DwProblem> dw_probs; std::vector<DwItem> dw_items; std::vector<DwSplitTile> dw_split;
  DwPlan dw_plan;
  int64_t adam_n; int last_n;
  int64_t t_restart;  // server event count when this replica last (re)started
  hipStream_t stream; hipEvent_t done_ev, ready_ev;
  hipStream_t done_st, ready_st;   // where these were last recorded
  StepState* state;            // of the steps that are replayed, in the arena
  hipGraphExec_t step_graph;   // one local step with its arguments in *state; null: launched kernel by kernel
  int64_t replayed;            // steps that ran as that graph
};

}  // namespace

struct als_ctx {
  als_config cfg;
  Layout L;
  char* arena; size_t arena_bytes;
  float *theta, *m, *delta;
  int64_t t;
  std::vector<Worker> w;
  char capture_error[512];   // why a step could not be captured, empty if none failed
  hipEvent_t server_ev; hipStream_t server_st;
  bool bf; bool allow_mfma;
  bool grouped_dw;   // the layers' weight gradients run as one grouped launch at the end of the backward pass
  bool list_dw;      // the same, the output matrix's too, where they have no aligned kernel
  int T;
};

namespace {

// Walks the arena handing out 256-byte aligned blocks; with base == nullptr it only counts.
struct Carver {
  char* base; size_t off;
  void* take(size_t bytes) {
    size_t a = (off + 255) & ~(size_t)255;
    off = a + bytes;
    return base ? (void*)(base + a) : nullptr;
  }
  float* f32(int64_t n) { return (float*)take((size_t)n * 4); }
  void* act(int64_t n, bool bf) { return take((size_t)n * (bf ? 2 : 4)); }
};

void carve(als_ctx* c, Carver& cv) {
  const als_config& g = c->cfg;
  bool bf = g.dtype == ALS_DTYPE_BF16;
  int64_t P = c->L.P, T = (int64_t)g.batch * g.seq_len, d = g.d_model, ff = g.d_ff, V = g.vocab;
  int64_t da = (int64_t)g.n_heads * head_width(g);  // attention width
  int64_t BhS = (int64_t)g.batch * g.n_heads * g.seq_len;
  c->theta = cv.f32(P); c->m = cv.f32(P); c->delta = cv.f32(P);
  c->w.resize(g.n_workers);
  const bool groupable = bf && !(g.flags & 1) && dw_group_supported((int)d, (int)(3 * da), (int)T, d, 3 * da) &&
                  dw_group_supported((int)da, (int)d, (int)T, da, d) && dw_group_supported((int)d, (int)ff, (int)T, d, ff);
  int64_t tiles = gemm_tiles((int)d, (int)V, 256, 256);
  tiles += g.n_layers * (gemm_tiles((int)d, (int)(3 * da), 256, 256) + gemm_tiles((int)da, (int)d, 256, 256) + 2 * gemm_tiles((int)d, (int)ff, 256, 256));
  const bool few = groupable && T <= 2048 && tiles <= 128;   // see below
  c->grouped_dw = groupable && !(g.flags & 2) && !few;
  // Scratch of the output matrix's input gradient: 64 MiB hold the partials of a round of 256 x 256 tiles.  The same with and
  // without the grouped launch, so that the product is split, and rounds, the same way.
  const size_t head_bytes = std::min((size_t)g.n_layers * T * (2 * d + ff + 3 * da) * 2, (size_t)64 << 20);
  // Products without an aligned kernel: each fills a part of the chip (600 tokens, 320 x 1280: 100 tiles of 64 x 64) and costs
  // a launch.  17 products of four layers and the head took 199 us in fp32 mode (1024 tokens, d = 256, V = 2000) and 137 in bf16
  // (600 tokens, d = 320, V = 5003); as one list 107 and 50.  Every layer keeps its four dY for it, and the line is drawn at the
  // memory: 256 MiB more in a worker's arena.  It is no line of speed: near it the list still gains (a round of 12 layers, d = 128, 4096
  // tokens in fp32, 216 MiB: 2880 us, 4190 with a launch per product; 4 layers, d = 320, 8000 tokens in bf16, 175 MiB: 2490 and 3220).
  // Aligned products of few 256 x 256 tiles and a short K too: grouped, they are split 5 to 8 times along K and their partials are most of
  // the traffic (2048 tokens, d = 256, 4 layers, V = 4096: 28 us, 18 for the partials' sum and 19 for the output matrix; as a list 41).
  // Rounds of one worker, grouped / list: 64 tiles, 2048 tokens: 557 / 531; 128, 1024: 506 / 482; 28, 512: 253 / 240; above the line 148, 1024:
  // 1109 / 1115; 208, 2048: 915 / 921; 64, 8192: 1035 / 1055; 197, 8192: 2232 / 2294.  Inside the lines, d = 128 to 1024, one and two workers: 64 tokens,
  // 6 tiles 212 / 201, 128 tiles 483 / 471; 128 tokens, 7 tiles 228 / 206, 104 tiles 1074 / 1061; 512 tokens, d = 1024, 128 tiles 639 / 595; 2048 tokens,
  // 6 tiles 306 / 267, 128 tiles (V = 24576) 1432 / 1328.
  {
    const bool aligned = bf && T % 64 == 0 && d % 128 == 0 && (da % 128 == 0 || ff % 128 == 0);
    c->list_dw = !(g.flags & 3) && (!aligned || few) && (int64_t)g.n_layers * T * (2 * d + ff + 3 * da) * (bf ? 2 : 4) <= (int64_t)256 << 20;
  }
  for (Worker& w : c->w) {
    w.theta = cv.f32(P); w.start = cv.f32(P); w.adam_m = cv.f32(P); w.adam_v = cv.f32(P);
    w.grad = cv.f32(P);
    w.state = (StepState*)cv.take(sizeof(StepState));
    w.lp = bf ? (bf16*)cv.take((size_t)P * 2) : nullptr;
    int L = g.n_layers;
    w.x.resize(L + 1); w.xm.resize(L); w.rstd1.resize(L); w.rstd2.resize(L); w.lse.resize(L);
    w.a.resize(L); w.qkv.resize(L); w.o.resize(L); w.b.resize(L); w.u.resize(L); w.gl.resize(L);
    for (int l = 0; l <= L; l++) w.x[l] = cv.f32(T * d);
    for (int l = 0; l < L; l++) {
      w.xm[l] = cv.f32(T * d); w.rstd1[l] = cv.f32(T); w.rstd2[l] = cv.f32(T); w.lse[l] = cv.f32(BhS);
      w.a[l] = cv.act(T * d, bf); w.qkv[l] = cv.act(T * 3 * da, bf); w.o[l] = cv.act(T * da, bf);
      w.b[l] = cv.act(T * d, bf); w.u[l] = cv.act(T * ff, bf); w.gl[l] = cv.act(T * ff, bf);
    }
    w.xf = cv.act(T * d, bf); w.rstdf = cv.f32(T);
    // bf16 mode: the output GEMM writes bf16 logits into dlogits and the cross-entropy runs in place
    w.logits = bf ? nullptr : cv.f32(T * V); w.dlogits = cv.act(T * V, bf); w.loss_row = cv.f32(T);
    w.dxa = cv.f32(T * d); w.dxb = cv.f32(T * d); w.dtmp = cv.f32(T * d); w.Dbuf = cv.f32(BhS);
    // one set of gain-gradient partials per norm, in the layout order of the gains (g1, g2 per layer, gf)
    w.partial = cv.f32((int64_t)(2 * g.n_layers + 1) * rmsnorm_bwd_blocks((int)T) * d);
    w.dx_lp = cv.act(T * d, bf); w.dff = cv.act(T * ff, bf); w.d_o = cv.act(T * da, bf);
    w.dqkv = cv.act(T * 3 * da, bf);
    w.sort_offset = (int32_t*)cv.take((size_t)g.max_local_steps * (V + 1) * 4);
    w.sort_rank = (int32_t*)cv.take((size_t)g.max_local_steps * T * 4);
    w.sort_pos = (int32_t*)cv.take((size_t)g.max_local_steps * T * 4);
    // split-K partials of the weight-gradient GEMMs: up to 16 copies of the largest layer
    // matrix, capped at 64 MiB
    {
      int64_t big = d * (ff > 3 * da ? ff : 3 * da);
      size_t want = (size_t)big * 4 * 16;
      w.splitk_bytes = bf ? (want < ((size_t)64 << 20) ? want : ((size_t)64 << 20)) : 0;
      w.splitk_ws = w.splitk_bytes ? (float*)cv.take(w.splitk_bytes) : nullptr;
    }
    w.dy2.assign(L, w.dx_lp); w.dy1.assign(L, w.dff); w.dyo.assign(L, w.dx_lp); w.dyqkv.assign(L, w.dqkv);
    w.dw_probs_dev = nullptr; w.dw_items_dev = nullptr; w.dw_split_dev = nullptr; w.dw_partial = nullptr;
    w.dw_plan = DwPlan{0, 0, 0, 0.0};
    w.head_ws = w.splitk_ws; w.head_ws_bytes = w.splitk_bytes;
    if (groupable && !c->grouped_dw && !c->list_dw) { w.head_ws = (float*)cv.take(head_bytes); w.head_ws_bytes = head_bytes; }
    w.dw_probs.clear();
    if (c->grouped_dw || c->list_dw)
      for (int l = 0; l < L; l++) {
        w.dy2[l] = cv.act(T * d, bf); w.dy1[l] = cv.act(T * ff, bf); w.dyo[l] = cv.act(T * d, bf);
        w.dyqkv[l] = cv.act(T * 3 * da, bf);
      }
    int n_tiles = 0;
    auto add = [&](const void* X, int64_t M, const void* dY, int64_t N, int64_t off) {
      w.dw_probs.push_back(DwProblem{(const bf16*)X, (const bf16*)dY, w.grad ? w.grad + off : nullptr, (int)M, (int)N, (int)M, (int)N, {0, 0}});
      n_tiles += (int)(((M + 255) / 256) * ((N + 255) / 256));
    };
    // the products, in the order of the flat parameter layout (pointers are null while only counting)
    if (c->grouped_dw || c->list_dw)
      for (int l = 0; l < L; l++) {
        add(w.a[l], d, w.dyqkv[l], 3 * da, c->L.Wqkv[l]);
        add(w.o[l], da, w.dyo[l], d, c->L.Wo[l]);
        add(w.b[l], d, w.dy1[l], ff, c->L.W1[l]);
        add(w.gl[l], ff, w.dy2[l], d, c->L.W2[l]);
      }
    if (c->list_dw) add(w.xf, d, w.dlogits, V, c->L.Wout);
    // The input gradient of the output matrix runs before anything is written to these: until then they are its
    // split-K scratch, one block from the first to the last.
    if (groupable && (c->grouped_dw || c->list_dw)) { w.head_ws = (float*)w.dy2[0]; w.head_ws_bytes = head_bytes; }
    if (c->grouped_dw) {
      w.dw_items.resize(dw_plan_max_items(n_tiles));
      w.dw_split.resize(dw_plan_max_split(n_tiles) + 1);
      w.dw_plan = dw_group_plan(w.dw_probs.data(), (int)w.dw_probs.size(), (int)T, w.dw_items.data(), w.dw_split.data());
      w.dw_probs_dev = (DwProblem*)cv.take(w.dw_probs.size() * sizeof(DwProblem));
      w.dw_items_dev = (DwItem*)cv.take((size_t)w.dw_plan.n_items * sizeof(DwItem));
      w.dw_split_dev = (DwSplitTile*)cv.take((size_t)(w.dw_plan.n_split + 1) * sizeof(DwSplitTile));
      w.dw_partial = cv.f32((int64_t)w.dw_plan.n_partial_tiles * 65536);
    }
  }
}

GemmDesc desc(const als_ctx* c, const void* A, int a_layout, int64_t lda, const void* B, int b_layout,
              int64_t ldb, int M, int N, int K, void* C, int64_t ldc, bool c_act) {
  GemmDesc g;
  memset(&g, 0, sizeof g);
  g.A = A; g.B = B; g.M = M; g.N = N; g.K = K; g.a_layout = a_layout; g.b_layout = b_layout;
  g.lda = lda; g.ldb = ldb; g.in_bf16 = c->bf; g.C = C; g.ldc = ldc; g.c_bf16 = c_act && c->bf;
  g.epi = EPI_STORE;
  return g;
}

// weight-gradient GEMM: X^T dY into the flat fp32 gradient, with the worker's split-K scratch
GemmDesc desc_dw(const als_ctx* c, const Worker& w, const void* X, int64_t ldx, const void* dY, int64_t ldy,
                 int M, int N, int K, float* out) {
  GemmDesc g = desc(c, X, 1, ldx, dY, 0, ldy, M, N, K, out, N, false);
  g.ws = w.splitk_ws; g.ws_bytes = w.splitk_bytes;
  return g;
}

#define RUN(expr) do { int rc_ = (expr); if (rc_) return rc_; } while (0)

// Weight operand of a GEMM: the bf16 working copy in bf16 mode, the fp32 master otherwise.
inline const void* wptr(const als_ctx* c, const Worker& w, int64_t off) {
  return c->bf ? (const void*)(w.lp + off) : (const void*)(w.theta + off);
}

// ss (forward, backward): take the tokens and what depends on them from there
int forward(als_ctx* c, Worker& w, const int32_t* tok, hipStream_t st, StepState* ss) {
  const als_config& g = c->cfg;
  const Layout& L = c->L;
  int T = c->T, d = g.d_model, ff = g.d_ff, V = g.vocab, B = g.batch, S = g.seq_len, h = g.n_heads;
  const int dh = head_width(g), da = h * dh;
  const int ln = g.norm_kind == ALS_NORM_LAYER;  // LayerNorm (gain, no bias) instead of RMSNorm
  bool mf = c->allow_mfma;
  float eps = (float)g.norm_eps;
  RUN(embed_rmsnorm_fwd(tok, w.theta + L.E, w.theta + L.Ppos, w.x[0], w.theta + L.g1[0], w.a[0], w.rstd1[0], B, S, d, V, eps, c->bf, ln, st, ss));
  for (int l = 0; l < g.n_layers; l++) {
    if (l) RUN(rmsnorm_fwd(w.x[l], w.theta + L.g1[l], w.a[l], w.rstd1[l], T, d, eps, c->bf, ln, st));
    RUN(gemm(desc(c, w.a[l], 0, d, wptr(c, w, L.Wqkv[l]), 0, 3 * da, T, 3 * da, d, w.qkv[l], 3 * da, true), mf, st));
    RUN(attention_fwd(w.qkv[l], w.o[l], w.lse[l], B, S, h, dh, c->bf, mf, st));
    GemmDesc po = desc(c, w.o[l], 0, da, wptr(c, w, L.Wo[l]), 0, d, T, d, da, w.xm[l], d, false);
    po.epi = EPI_RESID; po.R = w.x[l]; po.ldr = d;
    RUN(gemm(po, mf, st));
    RUN(rmsnorm_fwd(w.xm[l], w.theta + L.g2[l], w.b[l], w.rstd2[l], T, d, eps, c->bf, ln, st));
    GemmDesc f1 = desc(c, w.b[l], 0, d, wptr(c, w, L.W1[l]), 0, ff, T, ff, d, w.u[l], ff, true);
    f1.epi = EPI_GELU; f1.C2 = w.gl[l];
    RUN(gemm(f1, mf, st));
    GemmDesc f2 = desc(c, w.gl[l], 0, ff, wptr(c, w, L.W2[l]), 0, d, T, d, ff, w.x[l + 1], d, false);
    f2.epi = EPI_RESID; f2.R = w.xm[l]; f2.ldr = d;
    RUN(gemm(f2, mf, st));
  }
  RUN(rmsnorm_fwd(w.x[g.n_layers], w.theta + L.gf, w.xf, w.rstdf, T, d, eps, c->bf, ln, st));
  void* logits = c->bf ? w.dlogits : (void*)w.logits;
  RUN(gemm(desc(c, w.xf, 0, d, wptr(c, w, L.Wout), 0, V, T, V, d, logits, V, true), mf, st));
  RUN(cross_entropy(logits, tok, w.loss_row, w.dlogits, c->bf, B, S, V, st, ss));
  return ALS_OK;
}

// also writes the mean of the losses that forward() left per row
int backward(als_ctx* c, Worker& w, const int32_t* tok, int slot, float* loss_out, hipStream_t st, StepState* ss) {
  const als_config& g = c->cfg;
  const Layout& L = c->L;
  int T = c->T, d = g.d_model, ff = g.d_ff, V = g.vocab, B = g.batch, S = g.seq_len, h = g.n_heads;
  const int dh = head_width(g), da = h * dh;
  const int ln = g.norm_kind == ALS_NORM_LAYER;  // LayerNorm (gain, no bias) instead of RMSNorm
  bool mf = c->allow_mfma;
  int nl = g.n_layers;
  // output matrix and final norm
  if (!c->list_dw) RUN(gemm(desc_dw(c, w, w.xf, d, w.dlogits, V, d, V, T, w.grad + L.Wout), mf, st));
  GemmDesc dxf = desc(c, w.dlogits, 0, V, wptr(c, w, L.Wout), 1, V, T, d, V, w.dtmp, d, false);
  dxf.ws = w.head_ws; dxf.ws_bytes = w.head_ws_bytes;
  RUN(gemm(dxf, mf, st));
  // the norms leave their gain-gradient partials, which are added after the last layer
  const int64_t pset = (int64_t)rmsnorm_bwd_blocks(T) * d;
  RUN(rmsnorm_bwd(w.dtmp, w.x[nl], w.rstdf, w.theta + L.gf, nullptr, w.dxa, nl ? w.dy2[nl - 1] : w.dx_lp, c->bf,
                  w.partial + 2 * nl * pset, T, d, ln, st));
  // The weight gradient of every matrix is X^T dY.  Either each is a product of its own, issued
  // here next to the input gradient that reads the same dY, or (grouped) every layer keeps its four
  // dY until the loop is over and all of them run as one launch.
  const bool each = !c->grouped_dw && !c->list_dw;
  for (int l = nl - 1; l >= 0; l--) {
    // feed-forward block: x_next = xm + gelu(b W1) W2
    if (each) RUN(gemm(desc_dw(c, w, w.gl[l], ff, w.dy2[l], d, ff, d, T, w.grad + L.W2[l]), mf, st));
    GemmDesc du = desc(c, w.dy2[l], 0, d, wptr(c, w, L.W2[l]), 1, d, T, ff, d, w.dy1[l], ff, true);
    du.epi = EPI_DGELU; du.U = w.u[l];
    RUN(gemm(du, mf, st));
    if (each) RUN(gemm(desc_dw(c, w, w.b[l], d, w.dy1[l], ff, d, ff, T, w.grad + L.W1[l]), mf, st));
    RUN(gemm(desc(c, w.dy1[l], 0, ff, wptr(c, w, L.W1[l]), 1, ff, T, d, ff, w.dtmp, d, false), mf, st));
    RUN(rmsnorm_bwd(w.dtmp, w.xm[l], w.rstd2[l], w.theta + L.g2[l], w.dxa, w.dxb, w.dyo[l], c->bf,
                    w.partial + (2 * l + 1) * pset, T, d, ln, st));
    // attention block: xm = x + attn(a Wqkv) Wo
    if (each) RUN(gemm(desc_dw(c, w, w.o[l], da, w.dyo[l], d, da, d, T, w.grad + L.Wo[l]), mf, st));
    RUN(gemm(desc(c, w.dyo[l], 0, d, wptr(c, w, L.Wo[l]), 1, d, T, da, d, w.d_o, da, true), mf, st));
    RUN(attention_bwd(w.qkv[l], w.o[l], w.d_o, w.lse[l], w.Dbuf, w.dyqkv[l], B, S, h, dh, c->bf, mf, st));
    if (each) RUN(gemm(desc_dw(c, w, w.a[l], d, w.dyqkv[l], 3 * da, d, 3 * da, T, w.grad + L.Wqkv[l]), mf, st));
    RUN(gemm(desc(c, w.dyqkv[l], 0, 3 * da, wptr(c, w, L.Wqkv[l]), 1, 3 * da, T, d, 3 * da, w.dtmp, d, false), mf, st));
    RUN(rmsnorm_bwd(w.dtmp, w.x[l], w.rstd1[l], w.theta + L.g1[l], w.dxb, w.dxa, l ? w.dy2[l - 1] : w.dx_lp, c->bf,
                    w.partial + 2 * l * pset, T, d, ln, st));
  }
  if (c->grouped_dw) RUN(dw_group_launch(w.dw_probs_dev, w.dw_items_dev, w.dw_split_dev, w.dw_plan, w.dw_partial, st));
  if (c->list_dw)
    RUN(c->bf ? gemm_mfma_any_dw_list(w.dw_probs.data(), (int)w.dw_probs.size(), T, st)
              : gemm_mfma_f32_dw_list(w.dw_probs.data(), (int)w.dw_probs.size(), T, st));
  // w.dtmp (T x d floats) is free again here: scratch for the embedding gradient's chunk partials
  RUN(embed_bwd(tok, w.sort_offset + (int64_t)slot * (V + 1), w.sort_pos + (int64_t)slot * T, w.dxa,
                w.grad + L.E, w.grad + L.Ppos, w.dtmp, w.loss_row, loss_out, B, S, d, V,
                NormPartials{w.partial, w.grad + L.g1[0], rmsnorm_bwd_blocks(T), 2 * nl + 1}, st, ss));
  return ALS_OK;
}

int check_ctx_worker(als_ctx* ctx, int worker) {
  if (!ctx) return set_error(ALS_ERR_INVALID, "context is null");
  if (worker < 0 || worker >= (int)ctx->w.size()) return set_error(ALS_ERR_INVALID, "worker %d out of range", worker);
  return ALS_OK;
}

std::atomic<bool> g_fail_capture{false};

// The step of one worker as a graph, captured on a stream of its own (nothing runs there).  On any failure the context goes on
// without: a step is then launched kernel by kernel, and the reason is kept for als_replay_info; the calling thread's last error stays what it was.
void capture_step(als_ctx* ctx, Worker& w, hipStream_t cs) {
  char last[sizeof ctx->capture_error];
  snprintf(last, sizeof last, "%s", als_last_error());
  hipGraph_t graph = nullptr;
  int rc = ALS_OK;
  hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeRelaxed);
  if (e == hipSuccess) {
    rc = forward(ctx, w, nullptr, cs, w.state);
    if (!rc) rc = backward(ctx, w, nullptr, 0, nullptr, cs, w.state);
    if (!rc) rc = adamw(w.theta, w.grad, w.adam_m, w.adam_v, w.lp, ctx->L.P, ctx->L.P_decay, AdamArgs{}, cs, w.state);
    if (!rc && g_fail_capture.load()) rc = set_error(ALS_ERR_HIP, "capture made to fail");
    e = hipStreamEndCapture(cs, &graph);
  }
  if (e == hipSuccess && !rc) e = hipGraphInstantiate(&w.step_graph, graph, nullptr, nullptr, 0);
  if (e != hipSuccess || rc) {
    w.step_graph = nullptr;
    snprintf(ctx->capture_error, sizeof ctx->capture_error, "%s", rc ? als_last_error() : hipGetErrorString(e));
    set_error(rc, "%s", last);
  }
  if (graph) (void)hipGraphDestroy(graph);
  (void)hipGetLastError();
}

// Whether the launches of the workers' steps hold the host longer than the chip (streams: different ones that the workers run on).  A launch
// takes the host 1.3 to 2.4 us, a node of a graph 0.4 to 1.2; of the workers that run side by side each advances by one kernel in about 5 us
// where the kernels are small.  Side by side are four at most: a process has four hardware queues, further streams share them.  Where
// the chip is the slower side a graph's start costs more than it saves, so with one or two streams steps are always launched.  Rounds of 2
// steps in us, kernel by kernel / as graphs, on a box whose host takes 1.3 us for a launch (workers on streams):
//                                     1 on 1       2 on 2       3 on 3        4 on 4        8 on 4        8 on 8        16 on 16      16 on 4
//   T 64, d 64, 2 layers              338 / 335    697 / 378    957 / 443     1315 / 843    2444 / 1644   1946 / 1323   3765 / 2249   4023 / 3180
//   T 256, d 64, 2 layers, fp32       347 / 344    445 / 406    653 / 466     892 / 903     1693 / 1754   1583 / 1388   3202 / 2239   3283 / 3483
//   T 512, d 256, 2 layers            398 / 411    480 / 485    665 / 574     1036 / 1048   2056 / 2092   1637 / 1727   3212 / 2997   4063 / 4193
//   T 512, d 256, 6 layers            953 / 964    1128 / 1124  1585 / 1315   2509 / 2472   5014 / 5035   5588 / 4147   8728 / 7158   11482 / 10029
//   T 2048, d 128, V 32000, 12 layers 2283 / 2296  3384 / 3215  4839 / 4187   6677 / 6695   13317 / 13296 11783 / 11813 21847 / 21708 26033 / 26448
//   T 4096, d 256, 2 layers           757 / 773    1048 / 1058  1379 / 1383   2187 / 2225   4331 / 4350   3851 / 3866   7156 / 7134   8652 / 8699
// and on one whose host takes 2.4 us: 4 on 4 of the second 1191 / 647, of the third 1274 / 922.  Beyond the line nothing is gained on any number
// of streams: T 4096, d 256, V 8192: 2553 / 2564, 5021 / 5008 (8 on 8), 9940 / 9880 (16 on 16); T 1024, d 896, 4 layers: 6536 / 6519, 12767 / 12787, 25322 / 25340.
constexpr int HW_QUEUES = 4;
bool replay_pays(const als_config& c, int streams) {
  const double T = (double)c.batch * c.seq_len, da = (double)c.n_heads * head_width(c), d = c.d_model;
  const double flops = 6.0 * T * (c.n_layers * (4.0 * d * da + 2.0 * d * c.d_ff + c.seq_len * da) + d * c.vocab);
  const int launches = 15 * c.n_layers + 12, side_by_side = std::min(std::min(c.n_workers, streams), HW_QUEUES);
  return side_by_side * 2.4 > 5.0 + flops / launches / 250e6;
}
int used_streams(const als_config& c, void* const* streams, int n_streams) {   // worker i runs on streams[i % n_streams]
  const int n = std::min(c.n_workers, n_streams);
  int different = 0;
  for (int i = 0; i < n; i++) different += std::find(streams, streams + i, streams[i]) == streams + i;
  return different;
}

// A wait costs the host 4 to 6 us: none where the stream's own order gives it.  (The handle of the per-thread default stream stands
// for another stream in every thread.)
int wait_event(hipStream_t st, hipEvent_t ev, hipStream_t recorded_on) {
  if (st != recorded_on || st == hipStreamPerThread) ALS_HIP(hipStreamWaitEvent(st, ev, 0));
  return ALS_OK;
}

// Calls that advance a worker or the server (step counts, the order of events, losses in host memory) are no work that a graph could replay:
// a stream under capture is refused, before anything is enqueued or changed.
int check_not_captured(hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess) (void)hipGetLastError();   // the launches report what is wrong with the stream, if anything is
  if (cap != hipStreamCaptureStatusNone) return set_error(ALS_ERR_HIP, "the worker's stream is being captured");
  return ALS_OK;
}

int sync_all(als_ctx* ctx) {
  for (Worker& w : ctx->w) ALS_HIP(hipStreamSynchronize(w.stream));
  return ALS_OK;
}

}  // namespace

extern "C" size_t als_arena_bytes(const als_config* cfg) {
  if (validate_config(cfg)) return 0;
  als_ctx tmp;
  tmp.cfg = *cfg;
  make_layout(*cfg, &tmp.L);
  Carver cv{nullptr, 0};
  carve(&tmp, cv);
  return cv.off + 256;
}

extern "C" int als_init(const als_config* cfg, void* arena, size_t arena_bytes, const float* theta0,
                        void* const* streams, int n_streams, als_ctx** out) {
  int rc = validate_config(cfg);
  if (rc) return rc;
  if (!arena || !theta0 || !out || !streams || n_streams < 1)
    return set_error(ALS_ERR_INVALID, "als_init: null argument or no stream");
  if ((uintptr_t)arena % 256) return set_error(ALS_ERR_ARENA, "arena must be 256-byte aligned");
  size_t need = als_arena_bytes(cfg);
  if (arena_bytes < need) return set_error(ALS_ERR_ARENA, "arena too small: %zu bytes given, %zu needed", arena_bytes, need);
  als_ctx* c = new (std::nothrow) als_ctx();
  if (!c) return set_error(ALS_ERR_INVALID, "out of host memory");
  c->cfg = *cfg;
  make_layout(*cfg, &c->L);
  c->arena = (char*)arena; c->arena_bytes = arena_bytes;
  c->bf = cfg->dtype == ALS_DTYPE_BF16;
  c->allow_mfma = !(cfg->flags & 1);
  c->T = cfg->batch * cfg->seq_len;
  c->t = 0;
  c->capture_error[0] = 0;
  Carver cv{(char*)arena, 0};
  carve(c, cv);
  if (c->grouped_dw)
    for (Worker& w : c->w) {
      if (hipMemcpy(w.dw_probs_dev, w.dw_probs.data(), w.dw_probs.size() * sizeof(DwProblem), hipMemcpyHostToDevice) != hipSuccess ||
          hipMemcpy(w.dw_items_dev, w.dw_items.data(), (size_t)w.dw_plan.n_items * sizeof(DwItem), hipMemcpyHostToDevice) != hipSuccess ||
          (w.dw_plan.n_split && hipMemcpy(w.dw_split_dev, w.dw_split.data(), (size_t)w.dw_plan.n_split * sizeof(DwSplitTile), hipMemcpyHostToDevice) != hipSuccess)) {
        int code = set_error(ALS_ERR_HIP, "als_init: uploading the weight-gradient work list failed: %s", hipGetErrorString(hipGetLastError()));
        delete c;
        return code;
      }
    }
  int64_t P = c->L.P;
  hipStream_t s0 = (hipStream_t)streams[0];
  c->server_ev = nullptr;
  for (Worker& w : c->w) { w.done_ev = nullptr; w.ready_ev = nullptr; w.losses_host = nullptr; w.step_graph = nullptr; w.replayed = 0; }
  auto fail = [&](int code) { als_destroy(c); return code; };
  if (hipEventCreateWithFlags(&c->server_ev, hipEventDisableTiming) != hipSuccess)
    return fail(set_error(ALS_ERR_HIP, "hipEventCreate failed"));
  if (hipMemcpyAsync(c->theta, theta0, (size_t)P * 4, hipMemcpyHostToDevice, s0) != hipSuccess ||
      hipMemsetAsync(c->m, 0, (size_t)P * 4, s0) != hipSuccess ||
      hipMemsetAsync(c->delta, 0, (size_t)P * 4, s0) != hipSuccess ||
      hipStreamSynchronize(s0) != hipSuccess)
    return fail(set_error(ALS_ERR_HIP, "als_init: copying theta0 failed: %s", hipGetErrorString(hipGetLastError())));
  for (size_t i = 0; i < c->w.size(); i++) {
    Worker& w = c->w[i];
    w.stream = (hipStream_t)streams[i % n_streams];
    w.adam_n = 0; w.last_n = 0; w.t_restart = 0;
    w.ready_st = w.done_st = w.stream;
    if (hipEventCreateWithFlags(&w.done_ev, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&w.ready_ev, hipEventDisableTiming) != hipSuccess ||
        hipHostMalloc((void**)&w.losses_host, (size_t)cfg->max_local_steps * 4, hipHostMallocDefault) != hipSuccess ||
        hipHostGetDevicePointer((void**)&w.losses_dev, w.losses_host, 0) != hipSuccess)
      return fail(set_error(ALS_ERR_HIP, "als_init: event or pinned-buffer creation failed"));
    if (hipMemsetAsync(w.adam_m, 0, (size_t)P * 4, w.stream) != hipSuccess ||
        hipMemsetAsync(w.adam_v, 0, (size_t)P * 4, w.stream) != hipSuccess ||
        hipMemsetAsync(w.grad, 0, (size_t)P * 4, w.stream) != hipSuccess)
      return fail(set_error(ALS_ERR_HIP, "als_init: clearing optimiser state failed"));
    rc = restart_copy(c->theta, w.theta, w.start, w.lp, P, w.stream);
    if (rc) return fail(rc);
    if (hipEventRecord(w.ready_ev, w.stream) != hipSuccess || hipEventRecord(w.done_ev, w.stream) != hipSuccess)
      return fail(set_error(ALS_ERR_HIP, "als_init: hipEventRecord failed"));
  }
  c->server_st = s0;
  if (hipEventRecord(c->server_ev, s0) != hipSuccess) return fail(set_error(ALS_ERR_HIP, "hipEventRecord failed"));
  rc = sync_all(c);
  if (rc) return fail(rc);
  if (replay_pays(*cfg, used_streams(*cfg, streams, n_streams)) && !gemm_hooks_active()) {
    hipStream_t cs = nullptr;
    if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) == hipSuccess) {
      for (Worker& w : c->w) capture_step(c, w, cs);
      (void)hipStreamDestroy(cs);
    } else {
      snprintf(c->capture_error, sizeof c->capture_error, "%s", hipGetErrorString(hipGetLastError()));
    }
  }
  *out = c;
  return ALS_OK;
}

extern "C" int als_destroy(als_ctx* c) {
  if (!c) return ALS_OK;
  for (Worker& w : c->w) {
    if (w.stream) (void)hipStreamSynchronize(w.stream);
    // on the per-thread default stream the last steps may be another thread's, and their graph has to outlive them
    if (w.step_graph) (void)hipEventSynchronize(w.done_ev);
    if (w.done_ev) (void)hipEventDestroy(w.done_ev);
    if (w.ready_ev) (void)hipEventDestroy(w.ready_ev);
    if (w.losses_host) (void)hipHostFree(w.losses_host);
    if (w.step_graph) (void)hipGraphExecDestroy(w.step_graph);
  }
  if (c->server_ev) (void)hipEventDestroy(c->server_ev);
  delete c;
  return ALS_OK;
}

extern "C" int als_worker_local_steps(als_ctx* ctx, int worker, int n_steps, const int32_t* tokens,
                                      const float* lr_host, float* loss_host) {
  int rc = check_ctx_worker(ctx, worker);
  if (rc) return rc;
  const als_config& g = ctx->cfg;
  if (n_steps < 0 || n_steps > g.max_local_steps)
    return set_error(ALS_ERR_INVALID, "n_steps %d outside 0..max_local_steps=%d", n_steps, g.max_local_steps);
  if (n_steps > 0 && (!tokens || !lr_host)) return set_error(ALS_ERR_INVALID, "tokens_dev and lr_host must be non-null");
  Worker& w = ctx->w[worker];
  RUN(check_not_captured(w.stream));
  RUN(wait_event(w.stream, w.ready_ev, w.ready_st));
  int64_t per = (int64_t)g.batch * (g.seq_len + 1);
  const bool replay = w.step_graph && !gemm_hooks_active();   // the measurement hooks of the GEMM kernels have to see the launches
  auto adam_args = [&](int s, int64_t n) {   // of step s, the worker's n-th
    AdamArgs a;
    a.lr = lr_host[s];
    a.beta1 = (float)g.adam_beta1; a.beta2 = (float)g.adam_beta2; a.eps = (float)g.adam_eps;
    a.wd = (float)g.weight_decay;
    a.bc1 = (float)(1.0 - pow(g.adam_beta1, (double)n));
    a.bc2 = (float)(1.0 - pow(g.adam_beta2, (double)n));
    return a;
  };
  StepState state;
  auto state_from = [&](int s) {   // of the steps from s on
    memset(&state, 0, sizeof state);
    state.tok = tokens + (int64_t)s * per;
    state.offset = w.sort_offset + (int64_t)s * (g.vocab + 1);
    state.pos = w.sort_pos + (int64_t)s * ctx->T;
    state.loss_out = w.losses_dev + s;
    state.tok_step = per; state.offset_step = g.vocab + 1; state.pos_step = ctx->T;
    for (int i = 0; i < ALS_STATE_STEPS && s + i < n_steps; i++) {
      state.adam = adam_args(s + i, w.adam_n + 1 + i);
      state.scalars[i].lr = state.adam.lr; state.scalars[i].bc1 = state.adam.bc1; state.scalars[i].bc2 = state.adam.bc2;
    }
  };
  if (replay && n_steps) state_from(0);
  RUN(embed_sort(tokens, n_steps, g.batch, g.seq_len, g.vocab, w.sort_offset, w.sort_rank, w.sort_pos, w.stream,
                 replay ? w.state : nullptr, &state));
  for (int s = 0; s < n_steps; s++) {
    if (replay) {
      if (s && s % ALS_STATE_STEPS == 0) {
        state_from(s);
        RUN(set_step_state(w.state, state, w.stream));
      }
      ALS_HIP(hipGraphLaunch(w.step_graph, w.stream));
      w.adam_n += 1;
      w.replayed += 1;
      continue;
    }
    const int32_t* tok = tokens + (int64_t)s * per;
    RUN(forward(ctx, w, tok, w.stream, nullptr));
    RUN(backward(ctx, w, tok, s, w.losses_dev + s, w.stream, nullptr));
    w.adam_n += 1;
    RUN(adamw(w.theta, w.grad, w.adam_m, w.adam_v, w.lp, ctx->L.P, ctx->L.P_decay, adam_args(s, w.adam_n), w.stream));
  }
  w.last_n = n_steps;
  ALS_HIP(hipEventRecord(w.done_ev, w.stream));
  w.done_st = w.stream;
  if (loss_host) {
    ALS_HIP(hipStreamSynchronize(w.stream));
    memcpy(loss_host, w.losses_host, (size_t)n_steps * 4);
  }
  return ALS_OK;
}

extern "C" int als_worker_loss_grad(als_ctx* ctx, int worker, const int32_t* tokens, float* loss_host) {
  int rc = check_ctx_worker(ctx, worker);
  if (rc) return rc;
  if (!tokens || !loss_host) return set_error(ALS_ERR_INVALID, "tokens_dev and loss_host must be non-null");
  Worker& w = ctx->w[worker];
  RUN(check_not_captured(w.stream));
  RUN(wait_event(w.stream, w.ready_ev, w.ready_st));
  RUN(embed_sort(tokens, 1, ctx->cfg.batch, ctx->cfg.seq_len, ctx->cfg.vocab, w.sort_offset, w.sort_rank,
                 w.sort_pos, w.stream));
  RUN(forward(ctx, w, tokens, w.stream, nullptr));
  RUN(backward(ctx, w, tokens, 0, w.losses_dev, w.stream, nullptr));
  ALS_HIP(hipEventRecord(w.done_ev, w.stream));
  w.done_st = w.stream;
  ALS_HIP(hipStreamSynchronize(w.stream));
  *loss_host = w.losses_host[0];
  return ALS_OK;
}

static int outer_apply(als_ctx* ctx, const int32_t* workers, int n_group, int restart_flag, const als_outer_rule& rule) {
  if (!ctx || !workers) return set_error(ALS_ERR_INVALID, "null argument");
  int k = (int)ctx->w.size();
  if (n_group < 1 || n_group > k) return set_error(ALS_ERR_INVALID, "n_group %d outside 1..k", n_group);
  if (rule.kind != ALS_RULE_DN && rule.kind != ALS_RULE_BUFFER) return set_error(ALS_ERR_INVALID, "unknown outer rule %d", rule.kind);
  if (!(rule.poly_exponent >= 0) || !isfinite(rule.poly_exponent) || !isfinite(rule.dc_lambda) || rule.dc_lambda < 0)
    return set_error(ALS_ERR_INVALID, "outer rule: poly_exponent and dc_lambda must be finite and >= 0");
  unsigned long long seen = 0;
  for (int j = 0; j < n_group; j++) {
    if (workers[j] < 0 || workers[j] >= k) return set_error(ALS_ERR_INVALID, "worker %d out of range", workers[j]);
    if (seen >> workers[j] & 1ull) return set_error(ALS_ERR_INVALID, "worker %d listed twice", workers[j]);
    seen |= 1ull << workers[j];
  }
  const als_config& g = ctx->cfg;
  hipStream_t st = ctx->w[workers[0]].stream;
  RUN(check_not_captured(st));
  RUN(wait_event(st, ctx->server_ev, ctx->server_st));
  for (int j = 0; j < n_group; j++) RUN(wait_event(st, ctx->w[workers[j]].done_ev, ctx->w[workers[j]].done_st));
  int64_t P = ctx->L.P;
  // Which events are applied: a worker whose staleness (server events since it started)
  // exceeds the threshold is discarded -- no server change, no event counted -- but still restarts.
  std::vector<int> applied;
  std::vector<float> weight;
  {
    int64_t t = ctx->t;
    for (int j = 0; j < n_group; j++) {
      int64_t stale = t - ctx->w[workers[j]].t_restart;
      if (rule.staleness_threshold >= 0 && stale > rule.staleness_threshold) continue;
      applied.push_back(workers[j]);
      weight.push_back(rule.poly_exponent > 0 ? (float)pow(1.0 + (double)stale, -rule.poly_exponent) : 1.0f);
      t++;
    }
  }
  int n_app = (int)applied.size();
  bool fused_restart = restart_flag && n_app == n_group && n_group <= ALS_DN_MAX_GROUP;
  for (int j0 = 0; j0 < n_app; j0 += ALS_DN_MAX_GROUP) {
    DnGroup dg;
    memset(&dg, 0, sizeof dg);
    dg.G = n_app - j0 < ALS_DN_MAX_GROUP ? n_app - j0 : ALS_DN_MAX_GROUP;
    dg.restart = fused_restart ? 1 : 0;
    for (int j = 0; j < ALS_DN_MAX_GROUP; j++) dg.weight[j] = 1.0f;
    for (int j = 0; j < dg.G; j++) {
      Worker& w = ctx->w[applied[j0 + j]];
      dg.theta_start[j] = w.start; dg.theta_worker[j] = w.theta; dg.start_out[j] = w.start;
      dg.lp_out[j] = w.lp;
      dg.weight[j] = weight[j0 + j];
      if ((ctx->t + j + 1) % g.dn_N == 0) dg.boundary_mask |= 1u << j;
    }
    dg.lr = (float)g.outer_lr; dg.beta = (float)g.outer_beta;
    dg.c_beta = (float)(g.dn_c * g.outer_beta);
    dg.cb_boundary = (float)((1.0 - g.dn_c * g.dn_N + g.dn_c) * g.outer_beta);
    dg.Nf = (float)g.dn_N;
    dg.dc_lambda = (float)rule.dc_lambda;
    dg.buffered = rule.kind == ALS_RULE_BUFFER;
    RUN(dn_group(ctx->theta, ctx->m, ctx->delta, dg, P, st));
    ctx->t += dg.G;
  }
  if (restart_flag && !fused_restart)
    for (int j = 0; j < n_group; j++) {
      Worker& w = ctx->w[workers[j]];
      RUN(restart_copy(ctx->theta, w.theta, w.start, w.lp, P, st));
    }
  if (restart_flag)
    for (int j = 0; j < n_group; j++) ctx->w[workers[j]].t_restart = ctx->t;
  ALS_HIP(hipEventRecord(ctx->server_ev, st));
  ctx->server_st = st;
  // Whatever touches these replicas next (their local steps, or a later sync) is ordered
  // after this call.
  for (int j = 0; j < n_group; j++) {
    ALS_HIP(hipEventRecord(ctx->w[workers[j]].ready_ev, st));
    ALS_HIP(hipEventRecord(ctx->w[workers[j]].done_ev, st));
    ctx->w[workers[j]].ready_st = ctx->w[workers[j]].done_st = st;
  }
  return ALS_OK;
}

extern "C" int als_outer_apply_dn(als_ctx* ctx, const int32_t* workers, int n_group, int restart_flag) {
  als_outer_rule rule;
  memset(&rule, 0, sizeof rule);
  rule.kind = ALS_RULE_DN; rule.staleness_threshold = -1;
  return outer_apply(ctx, workers, n_group, restart_flag, rule);
}

extern "C" int als_outer_apply_rule(als_ctx* ctx, const int32_t* workers, int n_group, int restart_flag,
                                    const als_outer_rule* rule) {
  if (!rule) return set_error(ALS_ERR_INVALID, "rule is null");
  return outer_apply(ctx, workers, n_group, restart_flag, *rule);
}

extern "C" int64_t als_worker_staleness(als_ctx* ctx, int worker) {
  if (check_ctx_worker(ctx, worker)) return -1;
  return ctx->t - ctx->w[worker].t_restart;
}

extern "C" int als_sync(als_ctx* ctx, int worker) {
  if (!ctx) return set_error(ALS_ERR_INVALID, "context is null");
  if (worker < 0) return sync_all(ctx);
  int rc = check_ctx_worker(ctx, worker);
  if (rc) return rc;
  ALS_HIP(hipStreamSynchronize(ctx->w[worker].stream));
  return ALS_OK;
}

static float* vector_ptr(als_ctx* ctx, int which, int worker) {
  switch (which) {
    case ALS_VEC_THETA: return ctx->theta;
    case ALS_VEC_MOMENTUM: return ctx->m;
    case ALS_VEC_DELTA: return ctx->delta;
    default: break;
  }
  if (worker < 0 || worker >= (int)ctx->w.size()) return nullptr;
  Worker& w = ctx->w[worker];
  switch (which) {
    case ALS_VEC_WORKER_THETA: return w.theta;
    case ALS_VEC_WORKER_START: return w.start;
    case ALS_VEC_ADAM_M: return w.adam_m;
    case ALS_VEC_ADAM_V: return w.adam_v;
    case ALS_VEC_GRAD: return w.grad;
    default: return nullptr;
  }
}

extern "C" int als_get_vector(als_ctx* ctx, int which, int worker, float* host_out) {
  if (!ctx || !host_out) return set_error(ALS_ERR_INVALID, "null argument");
  float* p = vector_ptr(ctx, which, worker);
  if (!p) return set_error(ALS_ERR_INVALID, "unknown vector %d / worker %d", which, worker);
  RUN(sync_all(ctx));
  ALS_HIP(hipMemcpy(host_out, p, (size_t)ctx->L.P * 4, hipMemcpyDeviceToHost));
  return ALS_OK;
}

extern "C" int als_set_vector(als_ctx* ctx, int which, int worker, const float* host_in) {
  if (!ctx || !host_in) return set_error(ALS_ERR_INVALID, "null argument");
  float* p = vector_ptr(ctx, which, worker);
  if (!p) return set_error(ALS_ERR_INVALID, "unknown vector %d / worker %d", which, worker);
  RUN(sync_all(ctx));
  ALS_HIP(hipMemcpy(p, host_in, (size_t)ctx->L.P * 4, hipMemcpyHostToDevice));
  if (which == ALS_VEC_WORKER_THETA && ctx->bf) {
    Worker& w = ctx->w[worker];
    RUN(cast_copy(w.theta, w.lp, ctx->L.P, 1, w.stream));
    ALS_HIP(hipStreamSynchronize(w.stream));
  }
  return ALS_OK;
}

extern "C" int als_get_losses(als_ctx* ctx, int worker, float* host_out, int n) {
  int rc = check_ctx_worker(ctx, worker);
  if (rc) return rc;
  Worker& w = ctx->w[worker];
  if (!host_out || n < 0 || n > w.last_n) return set_error(ALS_ERR_INVALID, "n outside 0..%d", w.last_n);
  ALS_HIP(hipStreamSynchronize(w.stream));
  memcpy(host_out, w.losses_host, (size_t)n * 4);
  return ALS_OK;
}

extern "C" int64_t als_server_t(als_ctx* ctx) { return ctx ? ctx->t : -1; }
extern "C" int64_t als_worker_adam_steps(als_ctx* ctx, int worker) {
  if (check_ctx_worker(ctx, worker)) return -1;
  return ctx->w[worker].adam_n;
}

// ---- stand-alone kernel entry points ---------------------------------------------------------
extern "C" int als_k_dn_group(float* theta, float* m, float* delta, float* const* theta_start,
                              float* const* theta_worker, void* const* bf16_worker, int G, int64_t P,
                              int N, int64_t t0, double outer_lr, double beta, double c, int restart,
                              void* stream) {
  if (G < 1 || G > ALS_DN_MAX_GROUP || P < 0 || N < 1 || t0 < 0) return set_error(ALS_ERR_INVALID, "G, P, N or t0 out of range");
  if (!(c >= 0 && c <= 1.0 / N + 1e-12)) return set_error(ALS_ERR_INVALID, "c must lie in [0, 1/N]");
  if (P == 0) return ALS_OK;
  if (!theta || !m || !delta || !theta_start || !theta_worker) return set_error(ALS_ERR_INVALID, "null argument");
  DnGroup dg;
  memset(&dg, 0, sizeof dg);
  dg.G = G; dg.restart = restart ? 1 : 0;
  for (int j = 0; j < ALS_DN_MAX_GROUP; j++) dg.weight[j] = 1.0f;
  for (int j = 0; j < G; j++) {
    if (!theta_start[j] || !theta_worker[j]) return set_error(ALS_ERR_INVALID, "null worker vector");
    dg.theta_start[j] = theta_start[j]; dg.theta_worker[j] = theta_worker[j];
    dg.start_out[j] = theta_start[j];
    dg.lp_out[j] = bf16_worker ? (bf16*)bf16_worker[j] : nullptr;
    if ((t0 + j + 1) % N == 0) dg.boundary_mask |= 1u << j;
  }
  dg.lr = (float)outer_lr; dg.beta = (float)beta; dg.c_beta = (float)(c * beta);
  dg.cb_boundary = (float)((1.0 - c * N + c) * beta); dg.Nf = (float)N;
  return dn_group(theta, m, delta, dg, P, (hipStream_t)stream);
}

extern "C" int als_k_adamw(float* theta, const float* grad, float* m, float* v, void* bf16_out, int64_t P,
                           int64_t P_decay, int64_t step, double lr, double beta1, double beta2,
                           double eps, double wd, void* stream) {
  if (P < 0 || P_decay < 0 || step < 1) return set_error(ALS_ERR_INVALID, "P, P_decay or step out of range");
  if (P == 0) return ALS_OK;
  if (!theta || !grad || !m || !v) return set_error(ALS_ERR_INVALID, "null argument");
  AdamArgs a;
  a.lr = (float)lr; a.beta1 = (float)beta1; a.beta2 = (float)beta2; a.eps = (float)eps; a.wd = (float)wd;
  a.bc1 = (float)(1.0 - pow(beta1, (double)step));
  a.bc2 = (float)(1.0 - pow(beta2, (double)step));
  return adamw(theta, grad, m, v, (bf16*)bf16_out, P, P_decay, a, (hipStream_t)stream);
}

namespace {
// the product of the als_k_gemm* entry points: operands without padding
GemmDesc plain_desc(const void* A, const void* B, void* C, int M, int N, int K, int a_layout, int b_layout, int in_dtype,
                    int out_dtype, int epi, void* ws_dev, size_t ws_bytes) {
  GemmDesc g;
  memset(&g, 0, sizeof g);
  g.A = A; g.B = B; g.C = C; g.M = M; g.N = N; g.K = K; g.a_layout = a_layout; g.b_layout = b_layout;
  g.lda = a_layout == 0 ? K : M; g.ldb = b_layout == 0 ? N : K; g.ldc = N;
  g.in_bf16 = in_dtype == ALS_DTYPE_BF16; g.c_bf16 = out_dtype == ALS_DTYPE_BF16; g.epi = epi;
  g.ws = (float*)ws_dev; g.ws_bytes = ws_dev ? ws_bytes : 0;
  return g;
}
}  // namespace

extern "C" int als_k_gemm(const void* A, const void* B, void* C, int M, int N, int K, int a_layout,
                          int b_layout, int in_dtype, int out_dtype, int use_mfma, void* ws_dev,
                          size_t ws_bytes, void* stream) {
  if (!A || !B || !C) return set_error(ALS_ERR_INVALID, "null argument");
  const GemmDesc g = plain_desc(A, B, C, M, N, K, a_layout, b_layout, in_dtype, out_dtype, EPI_STORE, ws_dev, ws_bytes);
  if (use_mfma) {
    if (!gemm_mfma_supported(g)) return set_error(ALS_ERR_INVALID, "shape/dtype not supported by the MFMA GEMM");
    return gemm_mfma(g, (hipStream_t)stream);
  }
  return gemm_generic(g, (hipStream_t)stream);
}

// ---- the entry point that allocates nothing ---------------------------------------------------
// Split-K partials of the stand-alone weight-gradient product live in this file-scope device
// array instead of a caller workspace.  Every GPU the library runs on holds its own copy of the
// array until the process ends; the host only ever uses the address hipGetSymbolAddress() returns
// for the current device (the array's name in host code is a stand-in, not a device address).
static __device__ __align__(256) unsigned char scratch[ALS_STATIC_WS_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];   // per device, filled at the first call on that device

int scratch_for_current_device(void** out) {
  int dev = -1;
  ALS_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return als::set_error(ALS_ERR_INVALID, "device index %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    ALS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return als::set_error(ALS_ERR_HIP, "hipGetSymbolAddress returned a null address");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return ALS_OK;
}
}  // namespace

extern "C" int als_k_gemm_static_ws(const void* A, const void* B, void* C, int M, int N, int K, int a_layout,
                                    int b_layout, int out_dtype, void* stream) {
  if (!A || !B || !C) return set_error(ALS_ERR_INVALID, "null argument");
  if (M <= 0 || N <= 0 || K <= 0) return set_error(ALS_ERR_INVALID, "M, N, K must be positive");
  // two fp32 partials of the product must fit, so that the split along K has room to happen
  if ((uint64_t)M * (uint64_t)N * sizeof(float) * 2 > (uint64_t)ALS_STATIC_WS_BYTES)
    return set_error(ALS_ERR_INVALID, "als_k_gemm_static_ws: M x N = %d x %d exceeds the static workspace "
                     "(2 fp32 partials must fit %zu bytes, i.e. M*N <= %zu)", M, N, (size_t)ALS_STATIC_WS_BYTES,
                     (size_t)ALS_STATIC_WS_BYTES / 8);
  GemmDesc g = plain_desc(A, B, C, M, N, K, a_layout, b_layout, ALS_DTYPE_BF16, out_dtype, EPI_STORE, nullptr, 0);
  if (!gemm_mfma_supported(g)) return set_error(ALS_ERR_INVALID, "shape/dtype not supported by the MFMA GEMM");
  void* ws = nullptr;
  int rc = scratch_for_current_device(&ws);
  if (rc) return rc;
  g.ws = (float*)ws; g.ws_bytes = ALS_STATIC_WS_BYTES;
  return gemm_mfma(g, (hipStream_t)stream);
}

namespace {
// workspace of the stand-alone grouped weight-gradient call: tables, then partial tiles
struct DwWsLayout { size_t probs, items, split, partial, total; };
DwWsLayout dw_ws_layout(int n, int n_tiles) {
  auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
  DwWsLayout l;
  l.probs = 0;
  l.items = up(l.probs + (size_t)n * sizeof(DwProblem));
  l.split = up(l.items + (size_t)dw_plan_max_items(n_tiles) * sizeof(DwItem));
  l.partial = up(l.split + (size_t)dw_plan_max_split(n_tiles) * sizeof(DwSplitTile));
  l.total = l.partial + (size_t)DW_PLAN_CUS * 65536 * sizeof(float);
  return l;
}
int dw_tiles(int n, const int* M, const int* N) {
  int t = 0;
  for (int i = 0; i < n; i++) t += ((M[i] + 255) / 256) * ((N[i] + 255) / 256);
  return t;
}
}  // namespace

extern "C" size_t als_k_gemm_dw_grouped_ws_bytes(int n, const int* M, const int* N) {
  if (n <= 0 || !M || !N) return 0;
  for (int i = 0; i < n; i++)
    if (M[i] <= 0 || N[i] <= 0) return 0;
  return dw_ws_layout(n, dw_tiles(n, M, N)).total;
}

extern "C" int als_k_gemm_dw_grouped(int n, const void* const* X, const void* const* dY, float* const* C,
                                     const int* M, const int* N, int K, void* ws_dev, size_t ws_bytes,
                                     void* stream) {
  if (n <= 0 || n > 4096 || !X || !dY || !C || !M || !N || !ws_dev) return set_error(ALS_ERR_INVALID, "null argument or bad count");
  std::vector<DwProblem> probs(n);
  for (int i = 0; i < n; i++) {
    if (!X[i] || !dY[i] || !C[i]) return set_error(ALS_ERR_INVALID, "product %d: null pointer", i);
    if (M[i] <= 0 || N[i] <= 0 || !dw_group_supported(M[i], N[i], K, M[i], N[i]))
      return set_error(ALS_ERR_INVALID, "product %d: %d x %d over %d not supported (M, N multiples of 128, K of 64)", i, M[i], N[i], K);
    if ((uintptr_t)X[i] % 16 || (uintptr_t)dY[i] % 16 || (uintptr_t)C[i] % 16)
      return set_error(ALS_ERR_INVALID, "product %d: pointers must be 16-byte aligned", i);
    probs[i] = DwProblem{(const bf16*)X[i], (const bf16*)dY[i], C[i], M[i], N[i], M[i], N[i], {0, 0}};
  }
  const int n_tiles = dw_tiles(n, M, N);
  const DwWsLayout l = dw_ws_layout(n, n_tiles);
  if ((uintptr_t)ws_dev % 256) return set_error(ALS_ERR_INVALID, "workspace must be 256-byte aligned");
  if (ws_bytes < l.total) return set_error(ALS_ERR_INVALID, "workspace too small: %zu bytes given, %zu needed", ws_bytes, l.total);
  std::vector<DwItem> items(dw_plan_max_items(n_tiles));
  std::vector<DwSplitTile> split(dw_plan_max_split(n_tiles) + 1);
  const DwPlan plan = dw_group_plan(probs.data(), n, K, items.data(), split.data());
  char* ws = (char*)ws_dev;
  hipStream_t st = (hipStream_t)stream;
  ALS_HIP(hipMemcpyAsync(ws + l.probs, probs.data(), (size_t)n * sizeof(DwProblem), hipMemcpyHostToDevice, st));
  ALS_HIP(hipMemcpyAsync(ws + l.items, items.data(), (size_t)plan.n_items * sizeof(DwItem), hipMemcpyHostToDevice, st));
  if (plan.n_split)
    ALS_HIP(hipMemcpyAsync(ws + l.split, split.data(), (size_t)plan.n_split * sizeof(DwSplitTile), hipMemcpyHostToDevice, st));
  ALS_HIP(hipStreamSynchronize(st));   // the tables above are host temporaries
  return dw_group_launch((const DwProblem*)(ws + l.probs), (const DwItem*)(ws + l.items),
                         (const DwSplitTile*)(ws + l.split), plan, (float*)(ws + l.partial), st);
}

// Host only: the work-item list als_k_gemm_dw_grouped would launch for these shapes, for checking
// on the CPU that it covers every tile and every K slice exactly once and stays inside its tables.
extern "C" int als_k_gemm_dw_grouped_plan(int n, const int* M, const int* N, int K, int max_items,
                                          int32_t* items_out, int max_split, int32_t* split_out,
                                          int32_t* counts_out) {
  if (n <= 0 || n > 4096 || !M || !N || !counts_out || (max_items > 0 && !items_out) || (max_split > 0 && !split_out))
    return set_error(ALS_ERR_INVALID, "null argument or bad count");
  std::vector<DwProblem> probs(n);
  for (int i = 0; i < n; i++) {
    if (M[i] <= 0 || N[i] <= 0 || !dw_group_supported(M[i], N[i], K, M[i], N[i]))
      return set_error(ALS_ERR_INVALID, "product %d: %d x %d over %d not supported (M, N multiples of 128, K of 64)", i, M[i], N[i], K);
    probs[i] = DwProblem{nullptr, nullptr, nullptr, M[i], N[i], M[i], N[i], {0, 0}};
  }
  const int n_tiles = dw_tiles(n, M, N);
  std::vector<DwItem> items(dw_plan_max_items(n_tiles));
  std::vector<DwSplitTile> split(dw_plan_max_split(n_tiles) + 1);
  const DwPlan plan = dw_group_plan(probs.data(), n, K, items.data(), split.data());
  counts_out[0] = plan.n_items; counts_out[1] = plan.n_split; counts_out[2] = plan.n_partial_tiles;
  counts_out[3] = dw_plan_max_items(n_tiles); counts_out[4] = dw_plan_max_split(n_tiles); counts_out[5] = DW_PLAN_CUS;
  for (int i = 0; i < plan.n_items && i < max_items; i++) {
    const DwItem& it = items[i];
    int32_t* o = items_out + 6 * (int64_t)i;
    o[0] = it.prob; o[1] = it.tm; o[2] = it.tn; o[3] = it.slot; o[4] = it.slice0; o[5] = it.nk;
  }
  for (int i = 0; i < plan.n_split && i < max_split; i++) {
    const DwSplitTile& t = split[i];
    int32_t* o = split_out + 5 * (int64_t)i;
    o[0] = t.prob; o[1] = t.tm; o[2] = t.tn; o[3] = t.slot0; o[4] = t.nslots;
  }
  return ALS_OK;
}

namespace {
int desc_ex(GemmDesc* g, const void* A, const void* B, void* C, int M, int N, int K, int a_layout, int b_layout, int in_dtype,
            int out_dtype, int epi, const float* R, void* C2, const void* U, void* ws_dev, size_t ws_bytes) {
  if (!A || !B || !C) return set_error(ALS_ERR_INVALID, "null argument");
  if (epi < 0 || epi > 3 || (epi == EPI_RESID && !R) || (epi == EPI_GELU && !C2) || (epi == EPI_DGELU && !U))
    return set_error(ALS_ERR_INVALID, "epilogue %d lacks its operand", epi);
  *g = plain_desc(A, B, C, M, N, K, a_layout, b_layout, in_dtype, out_dtype, epi, ws_dev, ws_bytes);
  g->R = R; g->ldr = N; g->C2 = C2; g->U = U;
  return ALS_OK;
}
}  // namespace

extern "C" int als_k_gemm_ex(const void* A, const void* B, void* C, int M, int N, int K, int a_layout,
                             int b_layout, int in_dtype, int out_dtype, int use_mfma, int epi, const float* R,
                             void* C2, const void* U, void* ws_dev, size_t ws_bytes, void* stream) {
  GemmDesc g;
  int rc = desc_ex(&g, A, B, C, M, N, K, a_layout, b_layout, in_dtype, out_dtype, epi, R, C2, U, ws_dev, ws_bytes);
  if (rc) return rc;
  if (use_mfma) {
    if (!gemm_mfma_supported(g)) return set_error(ALS_ERR_INVALID, "shape/dtype/epilogue not supported by the MFMA GEMM");
    return gemm_mfma(g, (hipStream_t)stream);
  }
  return gemm_generic(g, (hipStream_t)stream);
}

// Measurement and test hooks: a product and an attention as a worker step issues them.
extern "C" int als_k_step_gemm(const void* A, const void* B, void* C, int M, int N, int K, int a_layout, int b_layout,
                               int in_dtype, int out_dtype, int flags, int epi, const float* R, void* C2, const void* U,
                               void* ws_dev, size_t ws_bytes, void* stream) {
  GemmDesc g;
  int rc = desc_ex(&g, A, B, C, M, N, K, a_layout, b_layout, in_dtype, out_dtype, epi, R, C2, U, ws_dev, ws_bytes);
  if (rc) return rc;
  return gemm(g, !(flags & 1), (hipStream_t)stream);
}

extern "C" int als_k_step_attention_fwd(const void* qkv, void* o, float* lse, int B, int S, int h, int dh, int dtype, int flags,
                                        void* stream) {
  if (!qkv || !o || !lse) return set_error(ALS_ERR_INVALID, "null argument");
  return attention_fwd(qkv, o, lse, B, S, h, dh, dtype == ALS_DTYPE_BF16, !(flags & 1), (hipStream_t)stream);
}

extern "C" int als_k_step_attention_bwd(const void* qkv, const void* o, const void* d_o, const float* lse, float* dscratch,
                                        void* dqkv, int B, int S, int h, int dh, int dtype, int flags, void* stream) {
  if (!qkv || !o || !d_o || !lse || !dscratch || !dqkv) return set_error(ALS_ERR_INVALID, "null argument");
  return attention_bwd(qkv, o, d_o, lse, dscratch, dqkv, B, S, h, dh, dtype == ALS_DTYPE_BF16, !(flags & 1), (hipStream_t)stream);
}

extern "C" int als_replay_route(const als_config* cfg, int streams) {
  int rc = validate_config(cfg);
  if (rc) return rc;
  return replay_pays(*cfg, streams);
}

extern "C" int als_fail_capture(int on) {
  g_fail_capture = on != 0;
  return ALS_OK;
}

extern "C" int als_replay_info(als_ctx* ctx, int32_t* graphs_out, int64_t* steps_out, char* error_out, int error_len) {
  if (!ctx || !graphs_out || !steps_out || !error_out || error_len < 1) return set_error(ALS_ERR_INVALID, "null argument");
  snprintf(error_out, error_len, "%s", ctx->capture_error);
  *graphs_out = 0; *steps_out = 0;
  for (const Worker& w : ctx->w) { *graphs_out += w.step_graph != nullptr; *steps_out += w.replayed; }
  return ALS_OK;
}

extern "C" int als_k_gemm_route(int M, int N, int K, int a_layout, int b_layout, int in_dtype, int out_dtype, int epi, int flags,
                                size_t ws_bytes, char* out, int out_len) {
  if (!out || out_len < 1 || M <= 0 || N <= 0 || K <= 0) return set_error(ALS_ERR_INVALID, "null argument or empty shape");
  void* any = (void*)(uintptr_t)256;   // stands for aligned operands, never read
  GemmDesc g = plain_desc(any, any, any, M, N, K, a_layout, b_layout, in_dtype, out_dtype, epi, ws_bytes ? any : nullptr, ws_bytes);
  g.R = (const float*)any; g.ldr = N; g.C2 = any; g.U = any;
  gemm_route(g, !(flags & 1), out, out_len);
  return ALS_OK;
}

extern "C" int als_k_token_order_route(int T, int V, int n_steps, char* out, int out_len) {
  if (!out || out_len < 1 || T < 1 || V < 2 || n_steps < 1) return set_error(ALS_ERR_INVALID, "null argument or bad size");
  snprintf(out, out_len, "%s", token_order_route(T, V, n_steps));
  return ALS_OK;
}

extern "C" int als_k_embed_grad_route(int T, int V, int d, char* out, int out_len) {
  if (!out || out_len < 1 || T < 1 || V < 2 || d < 64 || d > 1024) return set_error(ALS_ERR_INVALID, "null argument or bad size");
  snprintf(out, out_len, "%s", embed_grad_route(T, V, d));
  return ALS_OK;
}

extern "C" int als_k_attention_fwd(const void* qkv, void* o, float* lse, int B, int S, int h, int dh,
                                   int dtype, int use_mfma, void* stream) {
  if (!qkv || !o || !lse) return set_error(ALS_ERR_INVALID, "null argument");
  int bf = dtype == ALS_DTYPE_BF16;
  if (use_mfma) {
    if (!attention_mfma_supported(S, dh, bf)) return set_error(ALS_ERR_INVALID, "shape/dtype not supported by the MFMA attention");
    // tensors at any other address are taken by the vector code
    if (attention_mfma_aligned(qkv, nullptr)) return attention_fwd_mfma(qkv, o, lse, B, S, h, dh, (hipStream_t)stream);
  }
  return attention_fwd_generic(qkv, o, lse, B, S, h, dh, bf, (hipStream_t)stream);
}

extern "C" int als_k_attention_bwd(const void* qkv, const void* o, const void* d_o, const float* lse,
                                   float* dscratch, void* dqkv, int B, int S, int h, int dh, int dtype,
                                   int use_mfma, void* stream) {
  if (!qkv || !o || !d_o || !lse || !dscratch || !dqkv) return set_error(ALS_ERR_INVALID, "null argument");
  int bf = dtype == ALS_DTYPE_BF16;
  if (use_mfma) {
    if (!attention_mfma_supported(S, dh, bf)) return set_error(ALS_ERR_INVALID, "shape/dtype not supported by the MFMA attention");
    if (attention_mfma_aligned(qkv, d_o)) return attention_bwd_mfma(qkv, o, d_o, lse, dscratch, dqkv, B, S, h, dh, (hipStream_t)stream);
  }
  return attention_bwd_generic(qkv, o, d_o, lse, dscratch, dqkv, B, S, h, dh, bf, (hipStream_t)stream);
}
