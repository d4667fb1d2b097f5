// Internal declarations shared by the library's translation units (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "../../include/als.h"

namespace als {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// 16 bytes per lane from base + voff straight into 1 KB of LDS at lds_addr, lane l to bytes 16 l .. 16 l + 15.  Outside the compiler's wait
// tracking: the wavefront waits for its own (vmcnt) before the barrier that precedes the first read.
__device__ __forceinline__ void global_to_lds_16(const void* base, unsigned voff, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(base) : "memory");
}

int set_error(int code, const char* fmt, ...);

#define ALS_HIP(expr)                                                                      \
  do {                                                                                     \
    hipError_t e_ = (expr);                                                                \
    if (e_ != hipSuccess)                                                                  \
      return als::set_error(ALS_ERR_HIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), \
                            __FILE__, __LINE__);                                           \
  } while (0)

#define ALS_CHECK_LAUNCH() ALS_HIP(hipGetLastError())

// ---- parameter layout -----------------------------------------------------------------
struct Layout {
  int64_t E, Ppos, Wout, gf;
  int64_t Wqkv[64], Wo[64], W1[64], W2[64], g1[64], g2[64];
  int64_t P, P_decay;
};
int validate_config(const als_config* c);
int head_width(const als_config& c);  // head_dim, or d/h when head_dim is 0
void make_layout(const als_config& c, Layout* L);

// ---- GEMM -------------------------------------------------------------------------------
enum Epilogue {
  EPI_STORE = 0,   // C = acc
  EPI_RESID = 1,   // C(fp32) = R(fp32) + acc
  EPI_GELU = 2,    // C = gelu_tanh'(acc) (kept for the backward pass), C2 = gelu_tanh(acc)
  EPI_DGELU = 3,   // C = acc * U, U = the saved gelu_tanh'(pre-activation)
};

struct GemmDesc {
  const void* A; const void* B;
  int M, N, K;
  int a_layout;  // 0: A[m*lda + k] ; 1: A[k*lda + m]
  int b_layout;  // 0: B[k*ldb + n] ; 1: B[n*ldb + k]
  int64_t lda, ldb;
  int in_bf16;   // operands bf16 (else fp32)
  void* C; int64_t ldc; int c_bf16;  // output type
  int epi;
  const float* R; int64_t ldr;       // EPI_RESID
  void* C2;                          // EPI_GELU second output (same type/ld as C)
  const void* U;                     // EPI_DGELU saved derivative (operand type, ld = ldc)
  float* ws; size_t ws_bytes;        // scratch for split-K partials (may be null)
};
inline int64_t gemm_tiles(int M, int N, int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn); }
int gemm_generic(const GemmDesc& g, hipStream_t st);
// fp32 operands and results on the fp32 matrix instruction (gemm_mfma_f32.hip): any shape, layout and epilogue
bool gemm_mfma_f32_supported(const GemmDesc& g);
int gemm_mfma_f32(const GemmDesc& g, hipStream_t st);
bool gemm_mfma_supported(const GemmDesc& g);
int gemm_mfma(const GemmDesc& g, hipStream_t st);
// bf16 operands, any shape and alignment (gemm_mfma_any.hip); X Y, X Y^T and X^T Y
bool gemm_mfma_any_supported(const GemmDesc& g);
int gemm_mfma_any(const GemmDesc& g, hipStream_t st);
double gemm_mfma_any_us(const GemmDesc& g);   // about what it takes, in microseconds
// what gemm_mfma_supported takes with a_layout 0, in tiles of 128 x 128 or 64 x 64 with deep prefetch (gemm_mfma_deep.hip)
int gemm_mfma_deep(const GemmDesc& g, int tile, hipStream_t st);
// als_prof_enable or als_k_set_gemm_tile is in force
bool gemm_hooks_active();
// picks a matrix-core kernel when allowed and supported
int gemm(const GemmDesc& g, bool allow_mfma, hipStream_t st);
// the name of the kernel and tile that each of these takes for a product (no GPU call)
const char* gemm_mfma_any_route(const GemmDesc& g);
const char* gemm_mfma_f32_route(const GemmDesc& g);
void gemm_mfma_route(const GemmDesc& g, char* out, int out_len);
void gemm_route(const GemmDesc& g, bool allow_mfma, char* out, int out_len);

// All weight gradients of a backward pass (X^T dY over the batch's tokens, bf16 operands, fp32
// results) as ONE launch of the 256 x 256 MFMA kernel.  The host turns the list of products into
// work items: whole rounds of tiles run unsplit over the full contraction and write C directly;
// the tiles of the last, partial round are split along K so that they fill the chip too, into
// 256 x 256 partial tiles that a second small kernel adds in slot order.  The records below are what
// the two kernels read from device memory.
struct DwProblem {
  const bf16* A; const bf16* B; float* C;   // A stored [K, M], B stored [K, N], C [M, N]; M, N multiples of 128
  int M, N, lda, ldb;
  int pad[2];
};
struct DwItem {
  int prob, tm, tn;
  int slot;         // -1: whole tile, result straight into C; else index of the partial tile in the workspace
  int slice0, nk;   // K slices of 64
  int pad[2];
};
struct DwSplitTile { int prob, tm, tn, slot0, nslots, pad[3]; };
static_assert(sizeof(DwProblem) == 48 && sizeof(DwItem) == 32 && sizeof(DwSplitTile) == 32, "table records");
struct DwPlan {
  int n_items, n_split, n_partial_tiles;   // partial tiles are 256 x 256 floats each
  double flops;
};
// Number of CUs the plan fills (MI355X).
constexpr int DW_PLAN_CUS = 256;
// Upper bounds of what dw_group_plan writes for n_tiles tiles in all.
inline int dw_plan_max_items(int n_tiles) { return n_tiles + DW_PLAN_CUS; }
inline int dw_plan_max_split(int n_tiles) { return n_tiles < DW_PLAN_CUS ? n_tiles : DW_PLAN_CUS; }
bool dw_group_supported(int M, int N, int K, int64_t lda, int64_t ldb);
// Shapes only are read from probs (pointers may still be null); items / split receive the tables
// in launch order (room for dw_plan_max_items / dw_plan_max_split records).
DwPlan dw_group_plan(const DwProblem* probs, int n_probs, int K, DwItem* items, DwSplitTile* split);
int dw_group_launch(const DwProblem* d_probs, const DwItem* d_items, const DwSplitTile* d_split, const DwPlan& plan,
                    float* partial_tiles, hipStream_t st);

// The same for products that have no aligned kernel (fp32, odd sizes): whole tiles of the kernels of gemm_mfma_any.hip and
// gemm_mfma_f32.hip, the list of products in the kernel's arguments.
constexpr int DW_LIST_MAX = 64;   // products of one launch (the arguments stay below 4 KB); longer lists take several
struct DwList {
  struct Product { const void* A; const void* B; float* C; int M, N, tiles_n, tile0; };
  int n, K;
  Product p[DW_LIST_MAX];
  // the product that tile id belongs to (tile0 ascends from 0)
  __device__ __forceinline__ int find(int tile) const {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
      const int mid = (lo + hi) / 2;
      if (p[mid].tile0 <= tile) lo = mid; else hi = mid;
    }
    return lo;
  }
  // the next products of a list, in tiles of bm x bn; returns how many
  int fill(const DwProblem* probs, int count, int K_, int bm, int bn, int* tiles) {
    n = count < DW_LIST_MAX ? count : DW_LIST_MAX;
    K = K_;
    *tiles = 0;
    for (int i = 0; i < n; i++) {
      const DwProblem& q = probs[i];
      p[i] = Product{q.A, q.B, q.C, q.M, q.N, (q.N + bn - 1) / bn, *tiles};
      *tiles += (q.M + bm - 1) / bm * p[i].tiles_n;
    }
    return n;
  }
};
inline int64_t dw_list_tiles(const DwProblem* probs, int n, int bm, int bn) {
  int64_t t = 0;
  for (int i = 0; i < n; i++) t += gemm_tiles(probs[i].M, probs[i].N, bm, bn);
  return t;
}
int gemm_mfma_any_dw_list(const DwProblem* probs, int n, int K, hipStream_t st);   // bf16 operands
int gemm_mfma_f32_dw_list(const DwProblem* probs, int n, int K, hipStream_t st);   // fp32 operands (A and B point to floats)

// ---- attention ----------------------------------------------------------------------------
int attention_fwd_generic(const void* qkv, void* o, float* lse, int B, int S, int h, int dh,
                          int bf, hipStream_t st);
int attention_bwd_generic(const void* qkv, const void* o, const void* d_o, const float* lse,
                          float* dscratch, void* dqkv, int B, int S, int h, int dh, int bf,
                          hipStream_t st);
// the same in fp32 arithmetic for heads of 32 and 64 and any length up to 1024: fp32 storage on the fp32 matrix instruction
// (attention_mfma_f32.hip), bf16 storage on the bf16 one (attention_mfma_any.hip)
bool attention_mfma_any_supported(const void* a, const void* b, const void* c, const void* e, int B, int S, int h, int dh);
int attention_fwd_mfma_f32(const void* qkv, void* o, float* lse, int B, int S, int h, int dh, hipStream_t st);
int attention_bwd_mfma_f32(const void* qkv, const void* o, const void* d_o, const float* lse, float* dscratch, void* dqkv, int B,
                           int S, int h, int dh, hipStream_t st);
int attention_fwd_mfma_any(const void* qkv, void* o, float* lse, int B, int S, int h, int dh, hipStream_t st);
int attention_bwd_mfma_any(const void* qkv, const void* o, const void* d_o, const float* lse, void* dqkv, int B, int S, int h, int dh,
                           hipStream_t st);
bool attention_mfma_supported(int S, int dh, int bf);
bool attention_mfma_aligned(const void* qkv, const void* d_o);   // d_o may be null
int attention_fwd_mfma(const void* qkv, void* o, float* lse, int B, int S, int h, int dh,
                       hipStream_t st);
int attention_bwd_mfma(const void* qkv, const void* o, const void* d_o, const float* lse,
                       float* dscratch, void* dqkv, int B, int S, int h, int dh, hipStream_t st);
// picks a matrix-core kernel when allowed and supported
int attention_fwd(const void* qkv, void* o, float* lse, int B, int S, int h, int dh, int bf, bool allow_mfma, hipStream_t st);
int attention_bwd(const void* qkv, const void* o, const void* d_o, const float* lse, float* dscratch, void* dqkv, int B, int S,
                  int h, int dh, int bf, bool allow_mfma, hipStream_t st);

// ---- elementwise / reductions ----------------------------------------------------------------
struct AdamArgs {
  float lr, beta1, beta2, eps, wd, bc1, bc2;
};
// What changes from one step of a worker to the next, in device memory: a step that is replayed as a graph has the same kernel
// arguments every time.  The kernels that need any of it take a pointer to it, and with a null pointer their own arguments.  It holds
// up to ALS_STATE_STEPS steps in a row; the first kernel of a step sets its AdamW scalars, the last one goes on to the next step.
#define ALS_STATE_STEPS 64
struct StepState {
  const int32_t* tok;      // [steps][B, S + 1]
  const int32_t* offset;   // what embed_sort made of them, [steps][V + 1] and [steps][B S]
  const int32_t* pos;
  float* loss_out;         // [steps]
  int64_t tok_step;        // elements of a step
  int offset_step, pos_step;
  int step;                // the one that runs
  AdamArgs adam;           // its own
  struct { float lr, bc1, bc2; } scalars[ALS_STATE_STEPS];
};
int set_step_state(StepState* ss, const StepState& v, hipStream_t st);
// center = 0: RMSNorm ; 1: LayerNorm with gain and no bias
int rmsnorm_fwd(const float* x, const float* g, void* y, float* rstd, int T, int d, float eps,
                int out_bf16, int center, hipStream_t st);
// the same for the rows E[tok] + Ppos, which are also written to x
int embed_rmsnorm_fwd(const int32_t* tok, const float* E, const float* Ppos, float* x, const float* g, void* y, float* rstd, int B,
                      int S, int d, int V, float eps, int out_bf16, int center, hipStream_t st, StepState* ss);
// dx_out = (dx_in ? dx_in : 0) + rmsnorm_backward(dy); optional low-precision copy of dx_out;
// the gain gradient, sum over rows of dy * xhat, is left in partial[nblk][d], nblk = rmsnorm_bwd_blocks(T), for embed_bwd to add.
int rmsnorm_bwd_blocks(int T);
int rmsnorm_bwd(const float* dy, const float* x, const float* rstd, const float* g,
                const float* dx_in, float* dx_out, void* dx_lp, int lp_bf16, float* partial, int T, int d, int center, hipStream_t st);
// logits and dlogits in bf16 or both in fp32; they may be the same buffer
int cross_entropy(const void* logits, const int32_t* tok, float* loss_row, void* dlogits, int bf, int B, int S, int V,
                  hipStream_t st, const StepState* ss);
// Orders each step's input positions by token id (see elementwise.hip; rank is scratch); offset is
// [n_steps][V+1], rank and pos are [n_steps][B*S].
// first (with its contents v): the state that the replayed steps begin with
int embed_sort(const int32_t* tok, int n_steps, int B, int S, int V, int32_t* offset, int32_t* rank,
               int32_t* pos, hipStream_t st, StepState* first = nullptr, const StepState* v = nullptr);
// which kernel that is (no GPU call)
const char* token_order_route(int64_t T, int V, int n_steps);
// nset consecutive sets of [nblk][d] partials and the gain gradients that they add up to, nset consecutive rows of d
struct NormPartials { const float* partial; float* dg; int nblk, nset; };
// dE, dPpos, the mean loss and the norms' gain gradients; scratch: 2 * ceil(B*S / 32) * d floats (partial rows of position lists that cross 32-position chunks)
int embed_bwd(const int32_t* tok, const int32_t* offset, const int32_t* pos, const float* dx, float* dE,
              float* dPpos, float* scratch, const float* loss_row, float* loss_out, int B, int S, int d, int V, const NormPartials& np,
              hipStream_t st, const StepState* ss);
// how many launches that takes (no GPU call)
const char* embed_grad_route(int T, int V, int d);
int cast_copy(const float* src, void* dst, int64_t n, int dst_bf16, hipStream_t st);

int adamw(float* theta, const float* grad, float* m, float* v, bf16* lp, int64_t P,
          int64_t P_decay, const AdamArgs& a, hipStream_t st, StepState* ss = nullptr);

#define ALS_DN_MAX_GROUP 16
struct DnGroup {
  const float* theta_start[ALS_DN_MAX_GROUP];
  float* theta_worker[ALS_DN_MAX_GROUP];
  float* start_out[ALS_DN_MAX_GROUP];
  bf16* lp_out[ALS_DN_MAX_GROUP];
  int G;
  int restart;
  unsigned boundary_mask;  // bit j set: event j is an N-th event
  float lr, beta, c_beta, cb_boundary, Nf;  // c*beta ; (1 - cN + c)*beta
  // comparison rules of the paper's "Existing Fixes": per-event weight on the pseudo-gradient
  // (polynomial staleness discount; 1 = none), delay-compensation strength lambda (0 = off),
  // buffered mode (no parameter change between N-th events, which apply Nesterov on Delta/N)
  float weight[ALS_DN_MAX_GROUP];
  float dc_lambda;
  int buffered;
};
int dn_group(float* theta, float* m, float* delta, const DnGroup& g, int64_t P, hipStream_t st);
int restart_copy(const float* theta, float* master, float* start, bf16* lp, int64_t P,
                 hipStream_t st);

}  // namespace als
