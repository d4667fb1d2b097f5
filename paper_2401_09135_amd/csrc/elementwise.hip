// HBM-bound kernels of the hot path: fused AdamW (inner optimiser), fused pseudo-gradient +
// Delayed Nesterov event(s) + worker restart (Alg. 3 and the restart of Alg. 2), embedding,
// RMSNorm, softmax cross-entropy and the small reductions around them.
#include "common.h"
#include <atomic>
#include <math.h>

namespace als {

static inline int blocks_for(int64_t n_items, int per_block, int cap) {
  int64_t b = (n_items + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

__device__ __forceinline__ void store_bf16x4(bf16* p, float4 v) {
  bf16x4 o;
  o[0] = (bf16)v.x; o[1] = (bf16)v.y; o[2] = (bf16)v.z; o[3] = (bf16)v.w;
  *reinterpret_cast<bf16x4*>(p) = o;
}

// ------------------------------------------------------------------------------------------
// AdamW, one pass over the flat vectors: reads grad, theta, m, v; writes theta, m, v and the
// bf16 working copy.  16 + 12 (+2) bytes per parameter.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float adam_one(float& th, float g, float& m, float& v, bool decay,
                                          const AdamArgs& a) {
  m = a.beta1 * m + (1.0f - a.beta1) * g;
  v = a.beta2 * v + (1.0f - a.beta2) * g * g;
  float mhat = m / a.bc1;
  float vhat = v / a.bc2;
  float upd = mhat / (sqrtf(vhat) + a.eps);
  if (decay) upd += a.wd * th;
  th -= a.lr * upd;
  return th;
}

// Streaming kernels below move 4 float4 per lane and iteration with non-temporal accesses
// (nothing they touch is reused before it leaves the caches): measured 6.0-6.1 TB/s on MI355X
// against 6.35 TB/s for a plain copy.
#define STREAM_U 4
__device__ __forceinline__ f32x4 ldnt(const float* p, int64_t i4) {
  return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p) + i4);
}
__device__ __forceinline__ void stnt(float* p, int64_t i4, f32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p) + i4);
}
__device__ __forceinline__ void stnt_bf16(bf16* p, int64_t i4, f32x4 v) {
  bf16x4 o;
  o[0] = (bf16)v[0]; o[1] = (bf16)v[1]; o[2] = (bf16)v[2]; o[3] = (bf16)v[3];
  __builtin_nontemporal_store(o, reinterpret_cast<bf16x4*>(p) + i4);
}
static inline int stream_blocks(int64_t n4, int u) {
  int64_t b = (n4 + 256 * u - 1) / (256 * u);
  return (int)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

// STATE: the scalars from the state of replayed steps (a template: a vector of 0.8 M took 0.1 us of 6 longer with the question in the kernel)
template <bool STATE>
__global__ __launch_bounds__(256) void adamw_kernel(float* __restrict__ theta,
                                                    const float* __restrict__ grad,
                                                    float* __restrict__ m, float* __restrict__ v,
                                                    bf16* __restrict__ lp, int64_t n4,
                                                    int64_t decay4, AdamArgs a, StepState* ss, bool last) {
  if (STATE) {
    a = ss->adam;
    if (last && blockIdx.x == 0 && threadIdx.x == 0) ss->step++;   // nothing in this kernel reads it
  }
  const int64_t stride = (int64_t)gridDim.x * 256 * STREAM_U;
  for (int64_t i0 = (int64_t)blockIdx.x * 256 * STREAM_U + threadIdx.x; i0 < n4; i0 += stride) {
    f32x4 th[STREAM_U], g[STREAM_U], mm[STREAM_U], vv[STREAM_U];
#pragma unroll
    for (int u = 0; u < STREAM_U; u++) {
      int64_t i = i0 + u * 256;
      if (i < n4) { th[u] = ldnt(theta, i); g[u] = ldnt(grad, i); mm[u] = ldnt(m, i); vv[u] = ldnt(v, i); }
    }
#pragma unroll
    for (int u = 0; u < STREAM_U; u++) {
      int64_t i = i0 + u * 256;
      if (i < n4) {
        bool dec = i < decay4;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          float t = th[u][e], mo = mm[u][e], ve = vv[u][e];
          adam_one(t, g[u][e], mo, ve, dec, a);
          th[u][e] = t; mm[u][e] = mo; vv[u][e] = ve;
        }
        stnt(theta, i, th[u]); stnt(m, i, mm[u]); stnt(v, i, vv[u]);
        if (lp) stnt_bf16(lp, i, th[u]);
      }
    }
  }
}

__global__ void adamw_tail_kernel(float* theta, const float* grad, float* m, float* v, bf16* lp,
                                  int64_t begin, int64_t P, int64_t P_decay, AdamArgs a, StepState* ss) {
  if (ss) a = ss->adam;
  if (ss && blockIdx.x == 0 && threadIdx.x == 0) ss->step++;
  int64_t i = begin + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  float th = theta[i], mm = m[i], vv = v[i];
  adam_one(th, grad[i], mm, vv, i < P_decay, a);
  theta[i] = th; m[i] = mm; v[i] = vv;
  if (lp) lp[i] = (bf16)th;
}

int adamw(float* theta, const float* grad, float* m, float* v, bf16* lp, int64_t P,
          int64_t P_decay, const AdamArgs& a, hipStream_t st, StepState* ss) {
  if (P <= 0) return ALS_OK;
  // the vector body covers whole float4 groups that do not straddle the decay boundary
  int64_t n4 = 0, decay4 = 0;
  if (P_decay % 4 == 0 || P_decay >= P) {
    n4 = P / 4;
    decay4 = P_decay >= P ? n4 : P_decay / 4;
  }
  if (n4 > 0) {
    const dim3 grid(stream_blocks(n4, STREAM_U));
    if (ss) hipLaunchKernelGGL(adamw_kernel<true>, grid, dim3(256), 0, st, theta, grad, m, v, lp, n4, decay4, a, ss, n4 * 4 == P);
    else hipLaunchKernelGGL(adamw_kernel<false>, grid, dim3(256), 0, st, theta, grad, m, v, lp, n4, decay4, a, ss, false);
    ALS_CHECK_LAUNCH();
  }
  int64_t begin = n4 * 4;
  if (begin < P) {
    int blocks = blocks_for(P - begin, 256, 1 << 30);
    hipLaunchKernelGGL(adamw_tail_kernel, dim3(blocks), dim3(256), 0, st, theta, grad, m, v, lp,
                       begin, P, P_decay, a, ss);
    ALS_CHECK_LAUNCH();
  }
  return ALS_OK;
}

__global__ void set_step_state_kernel(StepState* ss, StepState v) {
  if (threadIdx.x == 0) *ss = v;
}
int set_step_state(StepState* ss, const StepState& v, hipStream_t st) {
  hipLaunchKernelGGL(set_step_state_kernel, dim3(1), dim3(64), 0, st, ss, v);
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}

// ------------------------------------------------------------------------------------------
// Pseudo-gradient + Delayed Nesterov for a group of G workers in one pass, optionally fused
// with the restart copy.  Per element, in event order j = 0..G-1:
//   g = theta_start_j - theta_worker_j ; Delta += g
//   N-th event:  m = beta m + Delta/N ; theta -= eps ((1 - cN + c) beta m + g/N) ; Delta = 0
//   otherwise:   theta -= eps (c beta m + g/N)
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void dn_event_scalar(float& th, float& mm, float& de, float ts, float tw,
                                                bool boundary, bool use_m, float wj, const DnGroup& g) {
  float gj = ts - tw;
  // delay compensation: g + lambda g g (theta_now - theta_at_worker_start)
  if (g.dc_lambda != 0.0f) gj = gj + g.dc_lambda * gj * gj * (th - ts);
  if (wj != 1.0f) gj = wj * gj;  // staleness discount
  de += gj;
  if (g.buffered) {  // buffered averaging: Nesterov on Delta/N at every N-th event, nothing in between
    if (boundary) {
      float gbar = de / g.Nf;
      mm = g.beta * mm + gbar;
      th = th - g.lr * (g.beta * mm + gbar);
      de = 0.0f;
    }
    return;
  }
  if (boundary) {
    mm = g.beta * mm + de / g.Nf;
    th = th - g.lr * (g.cb_boundary * mm + gj / g.Nf);
    de = 0.0f;
  } else if (use_m) {
    th = th - g.lr * (g.c_beta * mm + gj / g.Nf);
  } else {
    th = th - g.lr * (gj / g.Nf);
  }
}

// U float4 per lane in flight (4 for one or two events, fewer for larger groups, whose 2 G
// worker vectors already keep many loads in flight).
template <int U>
__global__ __launch_bounds__(256) void dn_group_kernel(float* theta, float* m, float* delta, DnGroup g,
                                                       int64_t n4) {
  const bool use_m = g.c_beta != 0.0f;
  const bool touch_m = use_m || g.boundary_mask != 0u;
  const int64_t stride = (int64_t)gridDim.x * 256 * U;
  for (int64_t i0 = (int64_t)blockIdx.x * 256 * U + threadIdx.x; i0 < n4; i0 += stride) {
    f32x4 th[U], de[U], mm[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      int64_t i = i0 + u * 256;
      mm[u] = (f32x4){0.f, 0.f, 0.f, 0.f};
      if (i < n4) {
        th[u] = ldnt(theta, i); de[u] = ldnt(delta, i);
        if (touch_m) mm[u] = ldnt(m, i);
      }
    }
    if constexpr (U == 4) {   // one or two events: everything is requested at once
      for (int j = 0; j < g.G; j++) {
        f32x4 ts[U], tw[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
          int64_t i = i0 + u * 256;
          if (i < n4) { ts[u] = ldnt(g.theta_start[j], i); tw[u] = ldnt(g.theta_worker[j], i); }
        }
        const bool boundary = (g.boundary_mask >> j) & 1u;
        const float wj = g.weight[j];
#pragma unroll
        for (int u = 0; u < U; u++)
          if (i0 + u * 256 < n4) {
#pragma unroll
            for (int e = 0; e < 4; e++) {
              float t = th[u][e], mo = mm[u][e], d = de[u][e];
              dn_event_scalar(t, mo, d, ts[u][e], tw[u][e], boundary, use_m, wj, g);
              th[u][e] = t; mm[u][e] = mo; de[u][e] = d;
            }
          }
      }
    } else {
    // Events are taken four at a time, and the worker vectors of the NEXT four are requested
    // before the current four are applied: the loop over events has a run-time trip count, and
    // without this every event would wait for its own two loads with nothing else in flight.
    f32x4 tsA[4][U], twA[4][U], tsB[4][U], twB[4][U];
    auto load4 = [&](int j0, f32x4 (&ts)[4][U], f32x4 (&tw)[4][U]) {
#pragma unroll
      for (int jj = 0; jj < 4; jj++)
        if (j0 + jj < g.G) {
#pragma unroll
          for (int u = 0; u < U; u++) {
            int64_t i = i0 + u * 256;
            if (i < n4) { ts[jj][u] = ldnt(g.theta_start[j0 + jj], i); tw[jj][u] = ldnt(g.theta_worker[j0 + jj], i); }
          }
        }
    };
    auto apply4 = [&](int j0, const f32x4 (&ts)[4][U], const f32x4 (&tw)[4][U]) {
#pragma unroll
      for (int jj = 0; jj < 4; jj++)
        if (j0 + jj < g.G) {
          const bool boundary = (g.boundary_mask >> (j0 + jj)) & 1u;
          const float wj = g.weight[j0 + jj];
#pragma unroll
          for (int u = 0; u < U; u++)
            if (i0 + u * 256 < n4) {
#pragma unroll
              for (int e = 0; e < 4; e++) {
                float t = th[u][e], mo = mm[u][e], d = de[u][e];
                dn_event_scalar(t, mo, d, ts[jj][u][e], tw[jj][u][e], boundary, use_m, wj, g);
                th[u][e] = t; mm[u][e] = mo; de[u][e] = d;
              }
            }
        }
    };
    load4(0, tsA, twA);
    for (int j0 = 0; j0 < g.G; j0 += 8) {
      if (j0 + 4 < g.G) load4(j0 + 4, tsB, twB);
      apply4(j0, tsA, twA);
      if (j0 + 8 < g.G) load4(j0 + 8, tsA, twA);
      if (j0 + 4 < g.G) apply4(j0 + 4, tsB, twB);
    }
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      int64_t i = i0 + u * 256;
      if (i < n4) {
        stnt(theta, i, th[u]); stnt(delta, i, de[u]);
        if (g.boundary_mask != 0u) stnt(m, i, mm[u]);
        if (g.restart)
          for (int j = 0; j < g.G; j++) {
            stnt(g.theta_worker[j], i, th[u]); stnt(g.start_out[j], i, th[u]);
            if (g.lp_out[j]) stnt_bf16(g.lp_out[j], i, th[u]);
          }
      }
    }
  }
}

// scalar tail (P not a multiple of 4)
__global__ void dn_group_tail_kernel(float* theta, float* m, float* delta, DnGroup g, int64_t begin, int64_t P) {
  int64_t i = begin + threadIdx.x;
  if (i >= P) return;
  const bool use_m = g.c_beta != 0.0f;
  float th = theta[i], de = delta[i], mm = (use_m || g.boundary_mask) ? m[i] : 0.0f;
  for (int j = 0; j < g.G; j++)
    dn_event_scalar(th, mm, de, g.theta_start[j][i], g.theta_worker[j][i], (g.boundary_mask >> j) & 1u, use_m, g.weight[j], g);
  theta[i] = th; delta[i] = de;
  if (g.boundary_mask) m[i] = mm;
  if (g.restart)
    for (int j = 0; j < g.G; j++) {
      g.theta_worker[j][i] = th; g.start_out[j][i] = th;
      if (g.lp_out[j]) g.lp_out[j][i] = (bf16)th;
    }
}

// Restart of the G workers of a group from the new theta as a pass of its own: read 4, write 10 G
// bytes per parameter.  A write-dominated pass runs closer to the HBM peak than the same writes
// mixed into the event pass (whose 2 G + 3 read streams and 3 G + 3 write streams together reached
// 61-64 % of the peak; the event pass alone runs at the single-event rate, this one near the
// write-only rate), which more than pays for reading theta once more.
__global__ __launch_bounds__(256) void restart_group_kernel(const float* __restrict__ theta, DnGroup g, int64_t P) {
  const int64_t n4 = P / 4;
  const int64_t stride = (int64_t)gridDim.x * 256 * STREAM_U;
  for (int64_t i0 = (int64_t)blockIdx.x * 256 * STREAM_U + threadIdx.x; i0 < n4; i0 += stride) {
    f32x4 t[STREAM_U];
#pragma unroll
    for (int u = 0; u < STREAM_U; u++)
      if (i0 + u * 256 < n4) t[u] = ldnt(theta, i0 + u * 256);
    for (int j = 0; j < g.G; j++) {
#pragma unroll
      for (int u = 0; u < STREAM_U; u++)
        if (i0 + u * 256 < n4) reinterpret_cast<f32x4*>(g.theta_worker[j])[i0 + u * 256] = t[u];
#pragma unroll
      for (int u = 0; u < STREAM_U; u++)
        if (i0 + u * 256 < n4) reinterpret_cast<f32x4*>(g.start_out[j])[i0 + u * 256] = t[u];
      if (g.lp_out[j]) {
#pragma unroll
        for (int u = 0; u < STREAM_U; u++)
          if (i0 + u * 256 < n4) {
            bf16x4 o;
            o[0] = (bf16)t[u][0]; o[1] = (bf16)t[u][1]; o[2] = (bf16)t[u][2]; o[3] = (bf16)t[u][3];
            reinterpret_cast<bf16x4*>(g.lp_out[j])[i0 + u * 256] = o;
          }
      }
    }
  }
  if (blockIdx.x == 0) {
    for (int64_t i = n4 * 4 + threadIdx.x; i < P; i += blockDim.x) {
      float t = theta[i];
      for (int j = 0; j < g.G; j++) {
        g.theta_worker[j][i] = t; g.start_out[j][i] = t;
        if (g.lp_out[j]) g.lp_out[j][i] = (bf16)t;
      }
    }
  }
}

int dn_group(float* theta, float* m, float* delta, const DnGroup& g_in, int64_t P, hipStream_t st) {
  // groups of more than two workers: events first, then the restart as its own pass
  const bool split_restart = g_in.restart && g_in.G > 2;
  DnGroup g = g_in;
  if (split_restart) g.restart = 0;
  if (g.G < 1 || g.G > ALS_DN_MAX_GROUP) return set_error(ALS_ERR_INVALID, "dn_group: G out of range");
  if (P <= 0) return ALS_OK;
  int64_t n4 = P / 4;
  if (n4 > 0) {
    if (g.G <= 2)
      hipLaunchKernelGGL(dn_group_kernel<4>, dim3(stream_blocks(n4, 4)), dim3(256), 0, st, theta, m, delta, g, n4);
    else
      hipLaunchKernelGGL(dn_group_kernel<2>, dim3(stream_blocks(n4, 2)), dim3(256), 0, st, theta, m, delta, g, n4);
    ALS_CHECK_LAUNCH();
  }
  if (n4 * 4 < P) {
    hipLaunchKernelGGL(dn_group_tail_kernel, dim3(1), dim3(64), 0, st, theta, m, delta, g, n4 * 4, P);
    ALS_CHECK_LAUNCH();
  }
  if (split_restart) {
    hipLaunchKernelGGL(restart_group_kernel, dim3(stream_blocks(n4 > 0 ? n4 : 1, STREAM_U)), dim3(256), 0, st, theta, g, P);
    ALS_CHECK_LAUNCH();
  }
  return ALS_OK;
}

// theta -> worker master, round-start snapshot and bf16 working copy (read 4, write up to 10).
__global__ __launch_bounds__(256) void restart_kernel(const float* __restrict__ theta,
                                                      float* __restrict__ master,
                                                      float* __restrict__ start,
                                                      bf16* __restrict__ lp, int64_t P) {
  const int64_t n4 = P / 4;
  const int64_t stride = (int64_t)gridDim.x * 256 * STREAM_U;
  for (int64_t i0 = (int64_t)blockIdx.x * 256 * STREAM_U + threadIdx.x; i0 < n4; i0 += stride) {
    f32x4 t[STREAM_U];
#pragma unroll
    for (int u = 0; u < STREAM_U; u++)
      if (i0 + u * 256 < n4) t[u] = ldnt(theta, i0 + u * 256);
#pragma unroll
    for (int u = 0; u < STREAM_U; u++) {
      int64_t i = i0 + u * 256;
      if (i < n4) {
        if (master) stnt(master, i, t[u]);
        if (start) stnt(start, i, t[u]);
        if (lp) stnt_bf16(lp, i, t[u]);
      }
    }
  }
  if (blockIdx.x == 0) {
    for (int64_t i = n4 * 4 + threadIdx.x; i < P; i += blockDim.x) {
      float t = theta[i];
      if (master) master[i] = t;
      if (start) start[i] = t;
      if (lp) lp[i] = (bf16)t;
    }
  }
}

int restart_copy(const float* theta, float* master, float* start, bf16* lp, int64_t P,
                 hipStream_t st) {
  if (P <= 0) return ALS_OK;
  hipLaunchKernelGGL(restart_kernel, dim3(stream_blocks(P / 4, STREAM_U)), dim3(256), 0, st, theta, master,
                     start, lp, P);
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}

int cast_copy(const float* src, void* dst, int64_t n, int dst_bf16, hipStream_t st) {
  if (dst_bf16) return restart_copy(src, nullptr, nullptr, (bf16*)dst, n, st);
  return restart_copy(src, (float*)dst, nullptr, nullptr, n, st);
}

// Embedding gradient without float atomics, so that a step is bit-reproducible.
// (1) embed_sort: one workgroup per step orders the T input positions by token id, equal tokens in
//     position order: offset[v] .. offset[v+1] delimit the positions holding token v inside pos[].
//     It depends on the tokens only, so one launch prepares every step of a local round.
// (2) embed_bwd: a pass over 32-position chunks of that list and a pass over vocabulary rows
//     (described at the kernels below).
//
// The order is a least-significant-digit radix sort of the positions by token id (digits of at most
// 8 bits: one pass for V <= 256, two for V <= 65536).  A tile of at most 16384 positions is ranked at a time:
// wavefront w owns up to 1024 consecutive ones, 64 per iteration, and finds the lanes that hold the same
// digit with one ballot per digit bit, so a rank costs one counter access per 64 positions and no
// comparison of positions with each other.  What bounds it is that chain of 16 counter updates per
// pass and the gathers of ids through L2; a round has one workgroup per step.  One launch at a time, T = 16384, V = 8192: 761 us
// with every position compared against the 1024 of its chunk, 54 us so; V = 32000: 785 and 69; T = 512: 20 and 13.  This kernel
// is left for what the next one does not take: more than one tile, or V from 32768 on.
constexpr int SORT_ITEMS = 16, SORT_TILE = 1024 * SORT_ITEMS;

__global__ __launch_bounds__(1024) void embed_sort_kernel(const int32_t* __restrict__ tok, int B,
                                                          int S, int V, int npass, int digit_bits, int32_t* offset,
                                                          int32_t* rank, int32_t* pos) {
  __shared__ int cnt[16][256];   // per wavefront and digit: count, then next output index
  __shared__ int base[256];      // per digit: next output index of the tile to come
  __shared__ int wmin[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T = B * S, ndig = 1 << digit_bits;
  const int32_t* tk = tok + (int64_t)blockIdx.x * B * (S + 1);
  int32_t* off = offset + (int64_t)blockIdx.x * (V + 1);
  int32_t* buf[2] = {pos + (int64_t)blockIdx.x * T, rank + (int64_t)blockIdx.x * T};
  // t / S by multiplication: exact for t < 2^22 and 1 < S <= 1024 (t (M S - 2^32) < 2^32)
  const unsigned M = S > 1 ? 0xffffffffu / (unsigned)S + 1u : 0u;
  auto token_at = [&](int t) {
    const int row = S > 1 ? (int)__umulhi((unsigned)t, M) : t;
    int id = tk[t + row];   // tokens are [B, S + 1], positions [B, S]
    return id < 0 ? 0 : (id >= V ? V - 1 : id);
  };
  const uint64_t below = (1ull << lane) - 1;
  // positions per wavefront and tile: a short list is dealt to all 16 wavefronts, 64 at least to each
  const int per_wave = T >= SORT_TILE ? 64 * SORT_ITEMS : (T + 1023) / 1024 * 64;

  for (int p = 0; p < npass; p++) {
    const int32_t* src = p == 0 ? nullptr : buf[(npass - p) & 1];   // the first pass reads positions in order
    int32_t* dst = buf[(npass - 1 - p) & 1];                         // the last one writes pos
    const int shift = p * digit_bits;
    auto exclusive_base = [&]() {   // base[] from digit totals to exclusive sums, by one wavefront
      int carry = 0;
      for (int d0 = 0; d0 < ndig; d0 += 64) {
        const int x = d0 + lane < ndig ? base[d0 + lane] : 0;
        int incl = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int n = __shfl_up(incl, o, 64);
          if (lane >= o) incl += n;
        }
        if (d0 + lane < ndig) base[d0 + lane] = carry + incl - x;
        carry += __shfl(incl, 63, 64);
      }
    };
    int item[SORT_ITEMS], dig[SORT_ITEMS], rk[SORT_ITEMS];
    auto load_tile = [&](int t0) {   // all loads of a tile in flight together
#pragma unroll
      for (int it = 0; it < SORT_ITEMS; it++) {
        const int i = t0 + wv * per_wave + it * 64 + lane;
        item[it] = it * 64 < per_wave && i < T ? (src ? src[i] : i) : -1;
      }
#pragma unroll
      for (int it = 0; it < SORT_ITEMS; it++)
        dig[it] = item[it] >= 0 ? (token_at(item[it]) >> shift) & (ndig - 1) : -1;
    };
    if (T > SORT_TILE) {   // several tiles: the digit totals of the whole list first
      if (tid < 256) base[tid] = 0;
      __syncthreads();
      for (int t0 = 0; t0 < T; t0 += SORT_TILE) {
        load_tile(t0);
#pragma unroll
        for (int it = 0; it < SORT_ITEMS; it++)
          if (dig[it] >= 0) atomicAdd(&base[dig[it]], 1);
      }
      __syncthreads();
      if (wv == 0) exclusive_base();
    }
    for (int t0 = 0; t0 < T; t0 += SORT_TILE) {
      for (int i = tid; i < 16 * 256; i += 1024) (&cnt[0][0])[i] = 0;
      __syncthreads();
      load_tile(t0);
#pragma unroll
      for (int it = 0; it < SORT_ITEMS; it++) {
        if (it * 64 < per_wave) {
          const bool active = dig[it] >= 0;
          uint64_t same = __ballot(active);
          for (int b = 0; b < digit_bits; b++) {
            const bool bit = (dig[it] >> b) & 1;
            const uint64_t set = __ballot(bit);
            same &= bit ? set : ~set;
          }
          // wavefront-private counters: its LDS operations complete in order
          volatile int* c = &cnt[wv][active ? dig[it] : 0];
          const int before = *c;
          rk[it] = before + __popcll(same & below);
          if (active && (same & below) == 0) *c = before + __popcll(same);
        }
      }
      __syncthreads();
      if (T <= SORT_TILE) {   // one tile: its counts are the totals
        if (tid < ndig) {
          int n = 0;
#pragma unroll
          for (int w = 0; w < 16; w++) n += cnt[w][tid];
          base[tid] = n;
        }
        __syncthreads();
        if (wv == 0) exclusive_base();
        __syncthreads();
      }
      if (tid < ndig) {
        int next = base[tid];
#pragma unroll
        for (int w = 0; w < 16; w++) {
          const int c = cnt[w][tid];
          cnt[w][tid] = next;
          next += c;
        }
        base[tid] = next;
      }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < SORT_ITEMS; it++)
        if (dig[it] >= 0) dst[cnt[wv][dig[it]] + rk[it]] = item[it];
      __syncthreads();
    }
  }

  // offset[v] = first index whose token is >= v: T everywhere, the index where a token's run starts,
  // then the minimum over all larger tokens (from the end of the vocabulary, 4096 entries at a time)
  const int32_t* sorted = buf[0];
  for (int v = tid; v <= V; v += 1024) off[v] = T;
  __syncthreads();
  for (int i0 = 0; i0 < T; i0 += 8 * 1024) {   // 8 positions per thread in flight
    int id[8], prev[8];
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const int i = i0 + u * 1024 + tid;
      id[u] = i < T ? sorted[i] : 0;
      prev[u] = lane == 0 && i > 0 && i < T ? sorted[i - 1] : 0;
    }
#pragma unroll
    for (int u = 0; u < 8; u++) {
      id[u] = token_at(id[u]);
      if (lane == 0) prev[u] = token_at(prev[u]);
    }
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const int i = i0 + u * 1024 + tid;
      const int left = __shfl_up(id[u], 1, 64);
      if (i < T && (i == 0 || (lane ? left : prev[u]) != id[u])) off[id[u]] = i;
    }
  }
  __syncthreads();
  int carry = T;   // minimum over everything behind the current 4096 entries
  for (int v0 = V / 4096 * 4096; v0 >= 0; v0 -= 4096) {
    const int v = v0 + 4 * tid;
    int x[4];
#pragma unroll
    for (int e = 3; e >= 0; e--) {
      x[e] = v + e <= V ? off[v + e] : T;
      if (e < 3 && x[e + 1] < x[e]) x[e] = x[e + 1];
    }
    int m = x[0];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int n = __shfl_down(m, o, 64);
      if (lane + o < 64 && n < m) m = n;
    }
    const int behind_lane = __shfl_down(m, 1, 64);
    if (lane == 0) wmin[wv] = m;
    __syncthreads();
    int behind = carry, all = carry;
    for (int w = 0; w < 16; w++) {
      const int n = wmin[w];
      if (w > wv && n < behind) behind = n;
      if (n < all) all = n;
    }
    if (lane < 63 && behind_lane < behind) behind = behind_lane;
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (v + e <= V) off[v + e] = x[e] < behind ? x[e] : behind;
    carry = all;
    __syncthreads();
  }
}

// The same for one tile and a vocabulary whose offsets fit LDS (V < 32768), all of it there: tokens are read once, with
// their position in the low 14 bits, every pass permutes them through LDS, and the offsets are formed there, each wavefront a
// run of the vocabulary.  Above, every pass gathers the tokens again and the offsets make the round through L2 once per 4096
// entries.  Inside rounds of several workers (slower than alone), the kernel above and this one, T = 16384, V = 8192: 68 us and 45; T = 8192, V = 32000: 69 and 38; T = 512, V = 1024: 14.5 and 11.5.
constexpr int SORT_LDS_V = 32768, SORT_POS_BITS = 14;
static_assert(SORT_TILE <= 1 << SORT_POS_BITS, "positions of a tile");
inline __host__ __device__ int sort_run(int V) { return (V + 1 + 4095) / 4096 * 256; }   // offsets of one wavefront

__global__ __launch_bounds__(1024) void embed_sort_lds_kernel(const int32_t* __restrict__ tok, int B, int S, int V, int npass,
                                                              int digit_bits, int32_t* __restrict__ offset, int32_t* __restrict__ pos) {
  extern __shared__ __attribute__((aligned(16))) int sbuf[];   // T keys, then 16 sort_run(V) offsets
  __shared__ int cnt[16][256];   // per wavefront and digit: count, then next output index
  __shared__ int base[256];
  __shared__ int wmin[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T = B * S, ndig = 1 << digit_bits;
  const int32_t* tk = tok + (int64_t)blockIdx.x * B * (S + 1);
  int32_t* off = offset + (int64_t)blockIdx.x * (V + 1);
  const uint64_t below = (1ull << lane) - 1;
  const int per_wave = (T + 1023) / 1024 * 64;   // consecutive positions of a wavefront
  unsigned key[SORT_ITEMS];
  int dig[SORT_ITEMS], rk[SORT_ITEMS];
#pragma unroll
  for (int it = 0; it < SORT_ITEMS; it++) {
    const int i = wv * per_wave + it * 64 + lane;
    key[it] = 0;
    if (it * 64 < per_wave && i < T) {
      const int id = tk[i + i / S];   // tokens are [B, S + 1], positions [B, S]
      key[it] = (unsigned)(id < 0 ? 0 : (id >= V ? V - 1 : id)) << SORT_POS_BITS | (unsigned)i;
    }
  }
  for (int p = 0; p < npass; p++) {
    const int shift = SORT_POS_BITS + p * digit_bits;
    for (int i = tid; i < 16 * 256; i += 1024) (&cnt[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; it++) {
      if (it * 64 < per_wave) {
        const bool active = wv * per_wave + it * 64 + lane < T;
        dig[it] = (key[it] >> shift) & (ndig - 1);
        uint64_t same = __ballot(active);
        for (int b = 0; b < digit_bits; b++) {
          const bool bit = (dig[it] >> b) & 1;
          const uint64_t set = __ballot(bit);
          same &= bit ? set : ~set;
        }
        // wavefront-private counters: its LDS operations complete in order
        volatile int* c = &cnt[wv][active ? dig[it] : 0];
        const int before = *c;
        rk[it] = before + __popcll(same & below);
        if (active && (same & below) == 0) *c = before + __popcll(same);
      }
    }
    __syncthreads();
    if (tid < ndig) {
      int n = 0;
#pragma unroll
      for (int w = 0; w < 16; w++) n += cnt[w][tid];
      base[tid] = n;
    }
    __syncthreads();
    if (wv == 0) {   // totals to exclusive sums
      int carry = 0;
      for (int d0 = 0; d0 < ndig; d0 += 64) {
        const int x = d0 + lane < ndig ? base[d0 + lane] : 0;
        int incl = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int n = __shfl_up(incl, o, 64);
          if (lane >= o) incl += n;
        }
        if (d0 + lane < ndig) base[d0 + lane] = carry + incl - x;
        carry += __shfl(incl, 63, 64);
      }
    }
    __syncthreads();
    if (tid < ndig) {
      int next = base[tid];
#pragma unroll
      for (int w = 0; w < 16; w++) {
        const int c = cnt[w][tid];
        cnt[w][tid] = next;
        next += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; it++)
      if (wv * per_wave + it * 64 + lane < T && it * 64 < per_wave) sbuf[cnt[wv][dig[it]] + rk[it]] = (int)key[it];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; it++) {
      const int i = wv * per_wave + it * 64 + lane;
      if (it * 64 < per_wave && i < T) key[it] = (unsigned)sbuf[i];
    }
  }
#pragma unroll
  for (int it = 0; it < SORT_ITEMS; it++) {   // dig: the token before this one
    const int i = wv * per_wave + it * 64 + lane;
    if (it * 64 < per_wave && i < T) {
      pos[(int64_t)blockIdx.x * T + i] = key[it] & ((1u << SORT_POS_BITS) - 1);
      dig[it] = i > 0 ? (int)((unsigned)sbuf[i - 1] >> SORT_POS_BITS) : -1;
    }
  }
  __syncthreads();

  // offset[v] = first index whose token is >= v: T everywhere, the index where a token's run starts, then the minimum over
  // all larger tokens
  const int run = sort_run(V), v_end = (wv + 1) * run;
  for (int v = tid; v < 16 * run; v += 1024) sbuf[v] = T;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < SORT_ITEMS; it++) {
    const int i = wv * per_wave + it * 64 + lane, id = (int)(key[it] >> SORT_POS_BITS);
    if (it * 64 < per_wave && i < T && dig[it] != id) sbuf[id] = i;
  }
  __syncthreads();
  int m = T;
  for (int v = wv * run + lane; v < v_end; v += 64) m = sbuf[v] < m ? sbuf[v] : m;
#pragma unroll
  for (int o = 32; o; o >>= 1) {
    const int n = __shfl_xor(m, o, 64);
    m = n < m ? n : m;
  }
  if (lane == 0) wmin[wv] = m;
  __syncthreads();
  int carry = T;   // minimum over everything behind the current 256 entries
  for (int w = wv + 1; w < 16; w++) carry = wmin[w] < carry ? wmin[w] : carry;
  for (int v0 = v_end - 256; v0 >= wv * run; v0 -= 256) {
    const int v = v0 + 4 * lane;
    int x[4];
#pragma unroll
    for (int e = 3; e >= 0; e--) {
      x[e] = sbuf[v + e];
      if (e < 3 && x[e + 1] < x[e]) x[e] = x[e + 1];
    }
    int all = x[0];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int n = __shfl_down(all, o, 64);
      if (lane + o < 64 && n < all) all = n;
    }
    int behind = __shfl_down(all, 1, 64);
    if (lane == 63 || carry < behind) behind = carry;
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (v + e <= V) off[v + e] = x[e] < behind ? x[e] : behind;
    const int first = __shfl(all, 0, 64);
    carry = first < carry ? first : carry;
  }
}

// The same by counting, for small steps: a position's place in the order is the number of (token, position) pairs before its own, and
// offset[v] the number of tokens below v.  A lane has one of the T + V + 1 questions and the 16 wavefronts of a workgroup share the pairs,
// read from LDS by all lanes at once; the questions of a step are dealt to as many workgroups as they need, where the sort above is
// a chain of passes in one.  It grows with the steps of a call, which the sort takes side by side.
__global__ __launch_bounds__(1024) void embed_rank_kernel(const int32_t* __restrict__ tok, int B, int S, int V,
                                                          int32_t* __restrict__ offset, int32_t* __restrict__ pos, StepState* first,
                                                          StepState state) {
  if (first && blockIdx.x == 0 && blockIdx.y == 0) {   // word by word: a copy by one thread is a chain of 110 stores
    const unsigned* src = reinterpret_cast<const unsigned*>(&state);
    for (unsigned i = threadIdx.x; i < sizeof(StepState) / 4; i += 1024) reinterpret_cast<unsigned*>(first)[i] = src[i];
  }
  extern __shared__ __attribute__((aligned(16))) unsigned pair[];   // token and position, padded to 64 with the largest value
  __shared__ int part[16][64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T = B * S, Tp = (T + 63) & ~63;
  const int32_t* tk = tok + (int64_t)blockIdx.y * B * (S + 1);
  for (int i = tid; i < Tp; i += 1024) {
    unsigned k = 0xffffffffu;
    if (i < T) {
      const int id = tk[i + i / S];   // tokens are [B, S + 1], positions [B, S]
      k = (unsigned)(id < 0 ? 0 : (id >= V ? V - 1 : id)) << SORT_POS_BITS | (unsigned)i;
    }
    pair[i] = k;
  }
  __syncthreads();
  const int question = blockIdx.x * 64 + lane, t = question - (V + 1);   // first the V + 1 offsets, then the T positions
  const unsigned q = t < 0 ? (unsigned)question << SORT_POS_BITS : t < T ? pair[t] : 0u;
  int n = 0;
#pragma unroll 4
  for (int i = wv * (Tp / 16); i < (wv + 1) * (Tp / 16); i += 4) {
    const u32x4 k = *reinterpret_cast<const u32x4*>(pair + i);
    n += (k[0] < q) + (k[1] < q) + (k[2] < q) + (k[3] < q);
  }
  part[wv][lane] = n;
  __syncthreads();
  if (wv == 0 && t < T) {
#pragma unroll
    for (int w = 1; w < 16; w++) n += part[w][lane];
    if (t < 0) offset[(int64_t)blockIdx.y * (V + 1) + question] = n;
    else pos[(int64_t)blockIdx.y * T + n] = t;
  }
}

// About what each of them takes, in us, from T = 64..12000, V = 64..131072, 1 to 200 steps in a call.  Counting: the comparisons and a
// part per workgroup; the sort, one workgroup a step: T, and V for the offsets, in LDS below SORT_LDS_V.  Counting / sort measured:
//   T 256, V 256: 3.2 / 8.1, 200 steps 7.2 / 8.6        T 512, V 1024: 3.2 / 9.2, 50 steps 6.7 / 9.7, 200 steps 21 / 10
//   T 512, V 8192, 16 steps: 10.4 / 12.3, 50: 28 / 13   T 1024, V 32000: 6.1 / 20.5, 4 steps 15 / 21, 8 steps 27 / 21
//   T 2048, V 4096: 5.0 / 12.0, 16 steps 20.5 / 12.4    T 4096, V 32000: 16.6 / 24.9, 2 steps 26 / 25
//   T 8192, V 1024: 13 / 18, 2 steps 21 / 19            T 512, V 131072: 9.9 / 92
// The list of positions in LDS ends the range at T = 12247.
constexpr double RANK_MAX = 150e6;   // comparisons of all steps of a call
static bool counting_pays(int64_t T, int V, int n_steps) {
  const double questions = (double)T + V + 1, comparisons = T * questions * n_steps, blocks = ceil(questions / 64) * n_steps;
  const double counting = 3.0 + 1e-3 * blocks + 1.05e-7 * comparisons, sort = 7.5 + 1.3e-3 * T + (V < SORT_LDS_V ? 3.7e-4 : 7e-4) * V;
  return T <= SORT_TILE && V <= 1 << 17 && n_steps <= 4096 && comparisons <= RANK_MAX && counting <= sort;
}
const char* token_order_route(int64_t T, int V, int n_steps) {
  return counting_pays(T, V, n_steps) ? "counting" : T <= SORT_TILE && V < SORT_LDS_V ? "sort in LDS" : "sort";
}

int embed_sort(const int32_t* tok, int n_steps, int B, int S, int V, int32_t* offset, int32_t* rank,
               int32_t* pos, hipStream_t st, StepState* first, const StepState* v) {
  if (n_steps <= 0) return ALS_OK;
  if (counting_pays((int64_t)B * S, V, n_steps)) {
    const int64_t T = (int64_t)B * S, questions = T + V + 1;
    hipLaunchKernelGGL(embed_rank_kernel, dim3((unsigned)((questions + 63) / 64), n_steps), dim3(1024), (size_t)((T + 63) & ~63) * 4, st, tok,
                       B, S, V, offset, pos, first, first ? *v : StepState{});
    ALS_CHECK_LAUNCH();
    return ALS_OK;
  }
  if (first) {
    const int rc = set_step_state(first, *v, st);
    if (rc) return rc;
  }
  int bits = 1;
  while (bits < 31 && (1 << bits) < V) bits++;
  const int npass = (bits + 7) / 8, digit_bits = (bits + npass - 1) / npass;
  const int T = B * S;
  if (T <= SORT_TILE && V < SORT_LDS_V) {
    const int offs = 16 * sort_run(V);
    static std::atomic<bool> attr_set{false};  // the call is idempotent: a race only repeats it
    if (!attr_set.load(std::memory_order_acquire)) {
      ALS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(embed_sort_lds_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  SORT_LDS_V * 4));
      attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(embed_sort_lds_kernel, dim3(n_steps), dim3(1024), (size_t)(T > offs ? T : offs) * 4, st, tok, B, S, V, npass,
                       digit_bits, offset, pos);
    ALS_CHECK_LAUNCH();
    return ALS_OK;
  }
  hipLaunchKernelGGL(embed_sort_kernel, dim3(n_steps), dim3(1024), 0, st, tok, B, S, V, npass, digit_bits, offset, rank, pos);
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}

// dE from the sorted position list, in two passes that never leave a long list to one block:
//   chunks: block c walks sorted positions [32 c, 32 c + 32), 8 row loads in flight, adding the
//     rows of equal tokens in list order.  A token whose whole list lies in this chunk is written
//     to dE at once; a list that continues into the next chunk leaves its part in scratch slot
//     (c, 1); one that began in an earlier chunk leaves its part in slot (c, 0).
//   rows: one wavefront per vocabulary row: zeros for a token that does not occur, nothing for a
//     list inside one chunk, else slot (first, 1) + slots (first+1 .. last, 0) in chunk order.
// Every sum has a fixed order, so the result does not depend on scheduling.
//
// The first pass is bound by latency where the batch is small, so where each token's part goes is read for all 32 positions at
// once, ahead of the walk (at every change of token it cost up to 32 dependent reads), and the sums over batches and the
// mean loss, which read the same step's results, are further blocks of the launch instead of launches.
// T = 512, d = 256: 15.3 + 2.6 + 2.3 us before, 11 now; T = 1024, d = 896: 42 + 5.6 + 4.6, 15 now.  So are the sums of the norms' partials,
// a launch of 3 to 5 us (13 for 25 norms of d = 896) until then.
constexpr int EMB_CH = 32;
#define EMB_MAXD4 4  // float4 slots per lane in the row pass: d <= 1024

// dPpos[s,:] = sum_b dx[b,s,:] in batch order
__device__ __forceinline__ void embed_bwd_pos(const float* __restrict__ dx, float* __restrict__ dPpos, int s, int B, int S, int d4) {
  const float4* dx4 = reinterpret_cast<const float4*>(dx);
  for (int c = threadIdx.x; c < d4; c += 256) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int b0 = 0; b0 < B; b0 += 8) {  // 8 loads in flight, added in batch order
      float4 x[8];
#pragma unroll
      for (int u = 0; u < 8; u++)
        x[u] = b0 + u < B ? dx4[((int64_t)(b0 + u) * S + s) * d4 + c] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 8; u++)
        if (b0 + u < B) { acc.x += x[u].x; acc.y += x[u].y; acc.z += x[u].z; acc.w += x[u].w; }
    }
    reinterpret_cast<float4*>(dPpos)[(int64_t)s * d4 + c] = acc;
  }
}

// out[0] = mean of v[0..T): 1024 strided sums, added per 64 and then in order
__device__ __forceinline__ void mean_rows(const float* __restrict__ v, float* __restrict__ out, int T) {
  __shared__ float sh[16];
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
  for (int i0 = 0; i0 < T; i0 += 1024)
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int i = i0 + u * 256 + threadIdx.x;
      acc[u] += i < T ? v[i] : 0.0f;
    }
#pragma unroll
  for (int u = 0; u < 4; u++) {
    acc[u] = wave_sum(acc[u]);
    if ((threadIdx.x & 63) == 0) sh[u * 4 + (threadIdx.x >> 6)] = acc[u];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float r = sh[0];
    for (int i = 1; i < 16; i++) r += sh[i];
    out[0] = r / (float)T;
  }
}

// out[j][c] = sum_b partial[j][b][c] for consecutive sets of partials: 32 columns of one set per block, 32 row groups of 32 threads' columns
// each adding every 32nd partial (8 independent loads in flight: it is pure load latency), combined in a fixed order.
__device__ __forceinline__ void sum_partials(const float* __restrict__ partial, float* __restrict__ out, int j, int c0, int nblk, int d) {
  __shared__ float sh[32][33];
  partial += (int64_t)j * nblk * d;
  const int cl = threadIdx.x & 31, c = c0 + cl;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int rg = (threadIdx.x >> 5) + 8 * q;
    float acc = 0.0f;
    if (c < d)
      for (int b0 = rg; b0 < nblk; b0 += 32 * 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {
          const int b = b0 + 32 * u;
          v[u] = b < nblk ? partial[(int64_t)b * d + c] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 8; u++) acc += v[u];
      }
    sh[rg][cl] = acc;
  }
  __syncthreads();
  if (threadIdx.x < 32 && c < d) {
    float t = sh[0][cl];
#pragma unroll
    for (int r = 1; r < 32; r++) t += sh[r][cl];
    out[(int64_t)j * d + c] = t;
  }
}

// What else reads the same step's results, one block each: S positions, the mean loss, the sums of the gain-gradient partials.
__device__ __forceinline__ void embed_bwd_rest(int e, const float* dx, float* dPpos, const float* loss_row, float* loss_out, int B, int S, int d,
                                               const NormPartials& np) {
  const int cols = (d + 31) / 32;
  if (e < S) embed_bwd_pos(dx, dPpos, e, B, S, d / 4);
  else if (e == S) mean_rows(loss_row, loss_out, B * S);
  else sum_partials(np.partial, np.dg, (e - S - 1) / cols, (e - S - 1) % cols * 32, np.nblk, d);
}

// blocks: the chunks, then the rest
__global__ __launch_bounds__(256) void embed_bwd_chunks_kernel(
    const int32_t* __restrict__ tok, const int32_t* __restrict__ offset, const int32_t* __restrict__ pos,
    const float* __restrict__ dx, float* __restrict__ dE, float* __restrict__ scratch, float* __restrict__ dPpos,
    const float* __restrict__ loss_row, float* __restrict__ loss_out, int B, int S, int V, int d, int nchunk, NormPartials np,
    const StepState* ss) {
  if (ss) {
    const int step = ss->step;
    tok = ss->tok + step * ss->tok_step; offset = ss->offset + (int64_t)step * ss->offset_step;
    pos = ss->pos + (int64_t)step * ss->pos_step; loss_out = ss->loss_out + step;
  }
  __shared__ int s_pos[EMB_CH], s_tok[EMB_CH], s_dst[EMB_CH];   // s_dst: -1 = dE, else the scratch slot
  const int T = B * S, c = blockIdx.x, i0 = c * EMB_CH, tid = threadIdx.x;
  const int d4 = d / 4;
  if (c >= nchunk) {
    embed_bwd_rest(c - nchunk, dx, dPpos, loss_row, loss_out, B, S, d, np);
    return;
  }
  const int n = T - i0 < EMB_CH ? T - i0 : EMB_CH;
  if (tid < n) {
    int t = pos[i0 + tid];
    int id = tok[(int64_t)(t / S) * (S + 1) + (t % S)];
    id = id < 0 ? 0 : (id >= V ? V - 1 : id);
    const int cf = offset[id] / EMB_CH, cl = (offset[id + 1] - 1) / EMB_CH;
    s_pos[tid] = t;
    s_tok[tid] = id;
    s_dst[tid] = cf == cl ? -1 : 2 * c + (c == cf ? 1 : 0);
  }
  __syncthreads();
  const float4* dx4 = reinterpret_cast<const float4*>(dx);
  for (int col = tid; col < d4; col += 256) {   // one pass for d <= 1024
    auto flush = [&](int j, float4 acc) {   // the list that position j ends
      const int slot = s_dst[j];
      float4* dst = slot < 0 ? reinterpret_cast<float4*>(dE) + (int64_t)s_tok[j] * d4 : reinterpret_cast<float4*>(scratch) + (int64_t)slot * d4;
      dst[col] = acc;
    };
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int cur = s_tok[0];
    for (int j0 = 0; j0 < n; j0 += 8) {
      float4 x[8];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        int j = j0 + u;
        x[u] = j < n ? dx4[(int64_t)s_pos[j] * d4 + col] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < 8; u++) {
        int j = j0 + u;
        if (j < n) {
          int tk = s_tok[j];
          if (tk != cur) {  // block-uniform
            flush(j - 1, acc);
            acc = make_float4(0.f, 0.f, 0.f, 0.f);
            cur = tk;
          }
          acc.x += x[u].x; acc.y += x[u].y; acc.z += x[u].z; acc.w += x[u].w;
        }
      }
    }
    flush(n - 1, acc);
  }
}

__global__ __launch_bounds__(256) void embed_bwd_rows_kernel(const int32_t* __restrict__ offset,
                                                             const float* __restrict__ scratch,
                                                             float* __restrict__ dE, int V, int d, const StepState* ss) {
  if (ss) offset = ss->offset + (int64_t)ss->step * ss->offset_step;
  const int lane = threadIdx.x & 63;
  const int v = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (v >= V) return;
  const int beg = offset[v], end = offset[v + 1];
  const int d4 = d / 4;
  float4* out = reinterpret_cast<float4*>(dE) + (int64_t)v * d4;
  if (beg == end) {
    for (int col = lane; col < d4; col += 64) out[col] = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  const int cf = beg / EMB_CH, cl = (end - 1) / EMB_CH;
  if (cf == cl) return;  // written by the chunk pass
  const float4* sc = reinterpret_cast<const float4*>(scratch);
#pragma unroll
  for (int s = 0; s < EMB_MAXD4; s++) {
    int col = lane + 64 * s;
    if (col >= d4) break;
    float4 acc = sc[(int64_t)(2 * cf + 1) * d4 + col];
#pragma unroll 8
    for (int c = cf + 1; c <= cl; c++) {
      float4 x = sc[(int64_t)(2 * c) * d4 + col];
      acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
    }
    out[col] = acc;
  }
}

// Small steps in one launch: a workgroup per vocabulary row, whose four wavefronts share its list, every fourth position each, and add
// their sums in order, 256 columns at a time.
__global__ __launch_bounds__(256) void embed_bwd_lists_kernel(const int32_t* __restrict__ offset, const int32_t* __restrict__ pos,
                                                              const float* __restrict__ dx, float* __restrict__ dE, float* __restrict__ dPpos,
                                                              const float* __restrict__ loss_row, float* __restrict__ loss_out, int B, int S, int V,
                                                              int d, NormPartials np, const StepState* ss) {
  if (ss) {
    const int step = ss->step;
    offset = ss->offset + (int64_t)step * ss->offset_step; pos = ss->pos + (int64_t)step * ss->pos_step; loss_out = ss->loss_out + step;
  }
  __shared__ f32x4 sums[3][64];
  const int v = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6, d4 = d / 4;
  if (v >= V) {
    embed_bwd_rest(v - V, dx, dPpos, loss_row, loss_out, B, S, d, np);
    return;
  }
  const int beg = offset[v], end = offset[v + 1];
  const f32x4* dx4 = reinterpret_cast<const f32x4*>(dx);
  for (int c0 = 0; c0 < d4; c0 += 64) {
    const int col = c0 + lane;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int j0 = beg + w; j0 < end; j0 += 32) {   // 8 rows in flight
      f32x4 x[8];
#pragma unroll
      for (int u = 0; u < 8; u++) x[u] = j0 + 4 * u < end && col < d4 ? dx4[(int64_t)pos[j0 + 4 * u] * d4 + col] : (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < 8; u++) acc += x[u];
    }
    if (end - beg > 1) {   // workgroup-uniform
      if (c0) __syncthreads();
      if (w) sums[w - 1][lane] = acc;
      __syncthreads();
      if (w == 0) acc = acc + sums[0][lane] + sums[1][lane] + sums[2][lane];
    }
    if (w == 0 && col < d4) reinterpret_cast<f32x4*>(dE)[(int64_t)v * d4 + col] = acc;
  }
}

// The most frequent token's list, a sixth of the positions of a Zipf(1.1) text, is one workgroup's in the one launch, once for every 256
// columns: that product bounds it, and the fewer rows there are the longer their lists.  Above 8192 rows most workgroups find an empty list.  One launch / two, in us (V = 64 / 1024 / 8192):
//   T 256, d 256: 4.6 / 4.1 / 6.7 and 9.7 / 11 / 12       T 256, d 512: 6.4 / 5.9 / 8.2 and 10 / 12 / 14     T 128, d 1024: 6.7 / 7.2 / 11 and 11 / 12 / 17
//   T 512, d 256: 7.3 / 6.0 / 6.8 and 10 / 11 / 12        T 512, d 512: 12 / 9.4 / 11 and 11 / 12 / 14       T 256, d 1024: 11 / 12 / 16 and 12 / 13 / 17
//   T 512, d 1024: 21 / 19 / 32 and 13 / 15 / 18          T 1024, d 256: 11 / 8.4 / 8.4 and 10 / 12 / 13
//   T 256, V 32000, d 256: 15.2 and 16.4
static bool one_launch_pays(int T, int V, int d) { return T <= 512 && V <= 8192 && T * ((d + 255) / 256) <= (V < 256 ? 768 : 1024); }
const char* embed_grad_route(int T, int V, int d) { return one_launch_pays(T, V, d) ? "one launch" : "two launches"; }

int embed_bwd(const int32_t* tok, const int32_t* offset, const int32_t* pos, const float* dx, float* dE,
              float* dPpos, float* scratch, const float* loss_row, float* loss_out, int B, int S, int d, int V, const NormPartials& np,
              hipStream_t st, const StepState* ss) {
  if (d > 256 * EMB_MAXD4 || d % 4) return set_error(ALS_ERR_INVALID, "embed_bwd: d unsupported");
  const int rest = S + 1 + np.nset * ((d + 31) / 32);
  if (one_launch_pays(B * S, V, d)) {
    hipLaunchKernelGGL(embed_bwd_lists_kernel, dim3(V + rest), dim3(256), 0, st, offset, pos, dx, dE, dPpos, loss_row, loss_out, B, S, V, d, np,
                       ss);
    ALS_CHECK_LAUNCH();
    return ALS_OK;
  }
  const int nchunk = (B * S + EMB_CH - 1) / EMB_CH;
  hipLaunchKernelGGL(embed_bwd_chunks_kernel, dim3(nchunk + rest), dim3(256), 0, st, tok, offset, pos, dx, dE, scratch, dPpos,
                     loss_row, loss_out, B, S, V, d, nchunk, np, ss);
  ALS_CHECK_LAUNCH();
  hipLaunchKernelGGL(embed_bwd_rows_kernel, dim3((V + 3) / 4), dim3(256), 0, st, offset, scratch, dE, V, d, ss);
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}

// ------------------------------------------------------------------------------------------
// Normalisation over the feature dimension, one 64-lane wavefront per row:
//   RMSNorm   (CENTER = false): y = x * rsqrt(mean(x^2) + eps) * g
//   LayerNorm (CENTER = true):  y = (x - mean(x)) * rsqrt(mean((x - mean(x))^2) + eps) * g   (no bias)
// rstd[row] is saved for the backward pass (which recomputes the mean from the row it reads).
// ------------------------------------------------------------------------------------------
// EMBED: the rows are the embeddings, x[b*S+s,:] = E[tok[b,s],:] + Ppos[s,:] (tokens are [B,S+1]; inputs are s < S), formed and
// written here on the way into the first norm: one launch and one pass over x less than on their own.
struct EmbedArgs { const int32_t* tok; const float* E; const float* Ppos; float* x; int S, V; StepState* ss; };
#define RMS_MAXD4 4  // float4 slots per lane: d <= 1024
template <typename OT, bool CENTER, bool EMBED>
__global__ __launch_bounds__(256) void rmsnorm_fwd_kernel(const float* __restrict__ x, EmbedArgs em,
                                                          const float* __restrict__ g,
                                                          OT* __restrict__ y,
                                                          float* __restrict__ rstd, int T, int d,
                                                          float eps) {
  int lane = threadIdx.x & 63;
  int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= T) return;
  const int d4 = d / 4;
  const float4* xr = reinterpret_cast<const float4*>(x + (int64_t)row * d);
  const float4* pr = nullptr;
  if (EMBED) {
    const int b = row / em.S, s = row % em.S;
    const int32_t* tok = em.tok;
    if (em.ss) {
      const int step = em.ss->step;
      tok = em.ss->tok + step * em.ss->tok_step;
      if (blockIdx.x == 0 && threadIdx.x == 0) {
        em.ss->adam.lr = em.ss->scalars[step].lr;
        em.ss->adam.bc1 = em.ss->scalars[step].bc1;
        em.ss->adam.bc2 = em.ss->scalars[step].bc2;
      }
    }
    int id = tok[(int64_t)b * (em.S + 1) + s];
    id = id < 0 ? 0 : (id >= em.V ? em.V - 1 : id);  // out-of-range ids are clamped, never dereferenced
    xr = reinterpret_cast<const float4*>(em.E + (int64_t)id * d);
    pr = reinterpret_cast<const float4*>(em.Ppos + (int64_t)s * d);
  }
  const float4* g4 = reinterpret_cast<const float4*>(g);
  float4 v[RMS_MAXD4];  // the row is read once and stays in registers (d <= 1024)
  float sum = 0.0f;
#pragma unroll
  for (int s = 0; s < RMS_MAXD4; s++) {
    int c = lane + 64 * s;
    v[s] = c < d4 ? xr[c] : make_float4(0.f, 0.f, 0.f, 0.f);
    if (EMBED && c < d4) {
      const float4 q = pr[c];
      v[s] = make_float4(v[s].x + q.x, v[s].y + q.y, v[s].z + q.z, v[s].w + q.w);
      reinterpret_cast<float4*>(em.x + (int64_t)row * d)[c] = v[s];
    }
    sum += (v[s].x + v[s].y) + (v[s].z + v[s].w);
  }
  const float mean = CENTER ? wave_sum(sum) / (float)d : 0.0f;
  float ss = 0.0f;
#pragma unroll
  for (int s = 0; s < RMS_MAXD4; s++) {
    int c = lane + 64 * s;
    if (CENTER && c < d4) { v[s].x -= mean; v[s].y -= mean; v[s].z -= mean; v[s].w -= mean; }
    ss += v[s].x * v[s].x + v[s].y * v[s].y + v[s].z * v[s].z + v[s].w * v[s].w;
  }
  ss = wave_sum(ss);
  float r = 1.0f / sqrtf(ss / (float)d + eps);
  if (lane == 0) rstd[row] = r;
  OT* yr = y + (int64_t)row * d;
#pragma unroll
  for (int s = 0; s < RMS_MAXD4; s++) {
    int c = lane + 64 * s;
    if (c < d4) {
      float4 gg = g4[c];
      float4 o = make_float4(v[s].x * r * gg.x, v[s].y * r * gg.y, v[s].z * r * gg.z, v[s].w * r * gg.w);
      if (sizeof(OT) == 2) store_bf16x4(reinterpret_cast<bf16*>(yr) + 4 * c, o);
      else reinterpret_cast<float4*>(yr)[c] = o;
    }
  }
}

template <bool EMBED>
static int norm_fwd(const float* x, const EmbedArgs& em, const float* g, void* y, float* rstd, int T, int d, float eps,
                    int out_bf16, int center, hipStream_t st) {
  if (d > 256 * RMS_MAXD4 || d % 4) return set_error(ALS_ERR_INVALID, "rmsnorm_fwd: d unsupported");
  dim3 grid((T + 3) / 4), block(256);
  if (out_bf16) {
    if (center) hipLaunchKernelGGL((rmsnorm_fwd_kernel<bf16, true, EMBED>), grid, block, 0, st, x, em, g, (bf16*)y, rstd, T, d, eps);
    else hipLaunchKernelGGL((rmsnorm_fwd_kernel<bf16, false, EMBED>), grid, block, 0, st, x, em, g, (bf16*)y, rstd, T, d, eps);
  } else {
    if (center) hipLaunchKernelGGL((rmsnorm_fwd_kernel<float, true, EMBED>), grid, block, 0, st, x, em, g, (float*)y, rstd, T, d, eps);
    else hipLaunchKernelGGL((rmsnorm_fwd_kernel<float, false, EMBED>), grid, block, 0, st, x, em, g, (float*)y, rstd, T, d, eps);
  }
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}

int rmsnorm_fwd(const float* x, const float* g, void* y, float* rstd, int T, int d, float eps,
                int out_bf16, int center, hipStream_t st) {
  return norm_fwd<false>(x, EmbedArgs{}, g, y, rstd, T, d, eps, out_bf16, center, st);
}

int embed_rmsnorm_fwd(const int32_t* tok, const float* E, const float* Ppos, float* x, const float* g, void* y, float* rstd, int B,
                      int S, int d, int V, float eps, int out_bf16, int center, hipStream_t st, StepState* ss) {
  return norm_fwd<true>(nullptr, EmbedArgs{tok, E, Ppos, x, S, V, ss}, g, y, rstd, B * S, d, eps, out_bf16, center, st);
}

// Backward: xhat = x rstd (RMSNorm) or (x - mean x) rstd (LayerNorm) ; dxhat = dy g ;
// dx = rstd (dxhat - xhat mean(dxhat xhat))  [LayerNorm: also - mean(dxhat)] ;
// dg = sum_rows dy xhat.  Each block walks rows with a fixed stride and leaves one partial dg
// row; embed_bwd adds the partials in a fixed order.
#define RMS_BWD_MAXD4 4  // per-lane float4 slots: supports d <= 1024
// One wavefront per row, each row read once into registers; a wave keeps two rows in flight.
template <typename LT, bool CENTER>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(
    const float* __restrict__ dy, const float* __restrict__ x, const float* __restrict__ rstd,
    const float* __restrict__ g, const float* dx_in, float* dx_out, LT* __restrict__ dx_lp,
    float* __restrict__ partial, int T, int d) {
  extern __shared__ float smem[];  // [4][d]
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int d4 = d / 4;
  const float inv_d = 1.0f / (float)d;
  f32x4 dg[RMS_BWD_MAXD4], gg[RMS_BWD_MAXD4];
#pragma unroll
  for (int s = 0; s < RMS_BWD_MAXD4; s++) {
    dg[s] = (f32x4){0.f, 0.f, 0.f, 0.f};
    int c = lane + 64 * s;
    gg[s] = c < d4 ? reinterpret_cast<const f32x4*>(g)[c] : (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  const int stride = gridDim.x * 4;
  for (int row0 = blockIdx.x * 4 + w; row0 < T; row0 += 2 * stride) {
    f32x4 xv[2][RMS_BWD_MAXD4], dv[2][RMS_BWD_MAXD4], av[2][RMS_BWD_MAXD4];
    float r[2], dot[2], m1[2];
    bool ok[2];
#pragma unroll
    for (int u = 0; u < 2; u++) {
      int row = row0 + u * stride;
      ok[u] = row < T;
      r[u] = ok[u] ? rstd[row] : 0.0f;
#pragma unroll
      for (int s = 0; s < RMS_BWD_MAXD4; s++) {
        int c = lane + 64 * s;
        bool in = ok[u] && c < d4;
        int64_t o = (int64_t)row * d4 + c;
        xv[u][s] = in ? reinterpret_cast<const f32x4*>(x)[o] : (f32x4){0.f, 0.f, 0.f, 0.f};
        dv[u][s] = in ? reinterpret_cast<const f32x4*>(dy)[o] : (f32x4){0.f, 0.f, 0.f, 0.f};
        av[u][s] = (in && dx_in) ? reinterpret_cast<const f32x4*>(dx_in)[o] : (f32x4){0.f, 0.f, 0.f, 0.f};
      }
    }
#pragma unroll
    for (int u = 0; u < 2; u++) {
      if (CENTER) {  // the row's mean, recomputed from the row in registers
        float sx = 0.0f;
#pragma unroll
        for (int s = 0; s < RMS_BWD_MAXD4; s++) sx += (xv[u][s][0] + xv[u][s][1]) + (xv[u][s][2] + xv[u][s][3]);
        const float mean = wave_sum(sx) * inv_d;
#pragma unroll
        for (int s = 0; s < RMS_BWD_MAXD4; s++)
          if (lane + 64 * s < d4) xv[u][s] -= mean;
      }
      float acc = 0.0f, acc1 = 0.0f;
#pragma unroll
      for (int s = 0; s < RMS_BWD_MAXD4; s++) {
        xv[u][s] *= r[u];  // xhat
        f32x4 dh = dv[u][s] * gg[s];
        f32x4 t = dh * xv[u][s];
        acc += (t[0] + t[1]) + (t[2] + t[3]);
        if (CENTER) acc1 += (dh[0] + dh[1]) + (dh[2] + dh[3]);
      }
      dot[u] = wave_sum(acc) * inv_d;
      m1[u] = CENTER ? wave_sum(acc1) * inv_d : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < 2; u++) {
      int row = row0 + u * stride;
      if (!ok[u]) continue;
#pragma unroll
      for (int s = 0; s < RMS_BWD_MAXD4; s++) {
        int c = lane + 64 * s;
        if (c < d4) {
          dg[s] += dv[u][s] * xv[u][s];
          f32x4 o = r[u] * (dv[u][s] * gg[s] - m1[u] - xv[u][s] * dot[u]) + av[u][s];
          int64_t oi = (int64_t)row * d4 + c;
          reinterpret_cast<f32x4*>(dx_out)[oi] = o;
          if (dx_lp) {
            if (sizeof(LT) == 2) store_bf16x4(reinterpret_cast<bf16*>(dx_lp) + 4 * oi, make_float4(o[0], o[1], o[2], o[3]));
            else reinterpret_cast<f32x4*>(dx_lp)[oi] = o;
          }
        }
      }
    }
  }
#pragma unroll
  for (int s = 0; s < RMS_BWD_MAXD4; s++) {
    int c = lane + 64 * s;
    if (c < d4) reinterpret_cast<f32x4*>(smem + w * d)[c] = dg[s];
  }
  __syncthreads();
  for (int c = threadIdx.x; c < d; c += 256)
    partial[(int64_t)blockIdx.x * d + c] = smem[c] + smem[d + c] + smem[2 * d + c] + smem[3 * d + c];
}

int rmsnorm_bwd_blocks(int T) {
  int b = (T + 3) / 4;
  return b > 256 ? 256 : b;
}

int rmsnorm_bwd(const float* dy, const float* x, const float* rstd, const float* g,
                const float* dx_in, float* dx_out, void* dx_lp, int lp_bf16, float* partial, int T, int d, int center, hipStream_t st) {
  if (d > 256 * RMS_BWD_MAXD4 || d % 4) return set_error(ALS_ERR_INVALID, "rmsnorm_bwd: d unsupported");
  int nblk = rmsnorm_bwd_blocks(T);
  size_t sm = (size_t)4 * d * sizeof(float);
#define ALS_NORM_BWD(LT, CEN)                                                                                   \
  hipLaunchKernelGGL((rmsnorm_bwd_kernel<LT, CEN>), dim3(nblk), dim3(256), sm, st, dy, x, rstd, g, dx_in, dx_out, \
                     (LT*)dx_lp, partial, T, d)
  if (lp_bf16) {
    if (center) ALS_NORM_BWD(bf16, true); else ALS_NORM_BWD(bf16, false);
  } else {
    if (center) ALS_NORM_BWD(float, true); else ALS_NORM_BWD(float, false);
  }
#undef ALS_NORM_BWD
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}

// ------------------------------------------------------------------------------------------
// Softmax cross-entropy, one block per row: loss_row = logsumexp - logit[target];
// dlogits = (softmax - onehot) / T.  Logits and dlogits are both fp32, or both bf16 (the output GEMM
// rounds them like every other activation); dlogits may overwrite the logits: every element is read before it is written, by the thread that writes it.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float block_reduce(float v, bool is_max, float* sh) {
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  v = is_max ? wave_max(v) : wave_sum(v);
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  int nw = blockDim.x >> 6;
  float r = sh[0];
  for (int i = 1; i < nw; i++) r = is_max ? fmaxf(r, sh[i]) : r + sh[i];
  return r;
}

template <typename T>
__global__ __launch_bounds__(256) void cross_entropy_kernel(const T* logits, const int32_t* __restrict__ tok,
                                                            float* __restrict__ loss_row, T* dl, int S, int V,
                                                            float invT, const StepState* ss) {
  if (ss) tok = ss->tok + ss->step * ss->tok_step;
  __shared__ float sh[8];
  int t = blockIdx.x;
  int b = t / S, s = t % S;
  int tgt = tok[(int64_t)b * (S + 1) + s + 1];
  tgt = tgt < 0 ? 0 : (tgt >= V ? V - 1 : tgt);
  const T* lr = logits + (int64_t)t * V;
  const float ltgt = (float)lr[tgt];
  float mx = -INFINITY;
  for (int c = threadIdx.x; c < V; c += blockDim.x) mx = fmaxf(mx, (float)lr[c]);
  mx = block_reduce(mx, true, sh);
  float sum = 0.0f;
  for (int c = threadIdx.x; c < V; c += blockDim.x) sum += expf((float)lr[c] - mx);
  sum = block_reduce(sum, false, sh);   // its barriers also order the read of lr[tgt] before the writes below
  float lse = mx + logf(sum);
  if (threadIdx.x == 0) loss_row[t] = lse - ltgt;
  T* dr = dl + (int64_t)t * V;
  for (int c = threadIdx.x; c < V; c += blockDim.x) {
    float p = expf((float)lr[c] - lse);
    if (c == tgt) p -= 1.0f;
    dr[c] = (T)(p * invT);
  }
}

// Same in bf16, reading the row once: each thread keeps up to 32 logits in registers, so a block of BS
// threads covers V <= 32 BS.  Rows of an odd V start at any element: 16-byte accesses at element alignment, and the
// last, partial group of 8 one by one (EDGE).  600 rows of 5003 in bf16: 19 us with three scalar passes, 8.6
// now.  fp32 mode keeps the three passes (1024 rows of 2000: 10.4 us, 6.6 this way) and their order of sums.
struct __attribute__((packed, aligned(2))) ce_b8 { bf16x8 v; };
template <int BS, bool EDGE>
__global__ __launch_bounds__(BS) void cross_entropy_reg_kernel(const bf16* logits, const int32_t* __restrict__ tok,
                                                               float* __restrict__ loss_row, bf16* dl, int S, int V,
                                                               float invT, const StepState* ss) {
  if (ss) tok = ss->tok + ss->step * ss->tok_step;
  __shared__ float sh[16];
  int t = blockIdx.x;
  int b = t / S, s = t % S;
  int tgt = tok[(int64_t)b * (S + 1) + s + 1];
  tgt = tgt < 0 ? 0 : (tgt >= V ? V - 1 : tgt);
  // a lane owns 8 consecutive columns per slot (16-byte loads, one 16-byte bf16 store)
  const bf16* row = logits + (int64_t)t * V;
  const float ltgt = (float)row[tgt];
  const int v8 = EDGE ? (V + 7) / 8 : V / 8;
  f32x4 x[4][2];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    int c = threadIdx.x + i * BS;
    if (c < v8) {
      if (EDGE && 8 * c + 8 > V) {
#pragma unroll
        for (int e = 0; e < 8; e++) x[i][e >> 2][e & 3] = 8 * c + e < V ? (float)row[8 * c + e] : -INFINITY;
      } else {
        bf16x8 r = EDGE ? reinterpret_cast<const ce_b8*>(row + 8 * c)->v : reinterpret_cast<const bf16x8*>(row)[c];
#pragma unroll
        for (int e = 0; e < 8; e++) x[i][e >> 2][e & 3] = (float)r[e];
      }
#pragma unroll
      for (int q = 0; q < 2; q++)
        mx = fmaxf(fmaxf(mx, fmaxf(x[i][q][0], x[i][q][1])), fmaxf(x[i][q][2], x[i][q][3]));
    }
  }
  mx = block_reduce(mx, true, sh);
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    int c = threadIdx.x + i * BS;
    if (c < v8) {
#pragma unroll
      for (int q = 0; q < 2; q++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
          x[i][q][e] = EDGE && 8 * c + 4 * q + e >= V ? 0.0f : expf(x[i][q][e] - mx);
          sum += x[i][q][e];
        }
    }
  }
  sum = block_reduce(sum, false, sh);
  float inv = 1.0f / sum;
  if (threadIdx.x == 0) loss_row[t] = mx + logf(sum) - ltgt;
  bf16* dr = dl + (int64_t)t * V;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    int c = threadIdx.x + i * BS;
    if (c < v8) {
      float p[8];
#pragma unroll
      for (int e = 0; e < 8; e++) {
        p[e] = x[i][e >> 2][e & 3] * inv;
        if (8 * c + e == tgt) p[e] -= 1.0f;
        p[e] *= invT;
      }
      if (EDGE && 8 * c + 8 > V) {
#pragma unroll
        for (int e = 0; e < 7; e++)
          if (8 * c + e < V) dr[8 * c + e] = (bf16)p[e];
      } else {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] = (bf16)p[e];
        if (EDGE) reinterpret_cast<ce_b8*>(dr + 8 * c)->v = o;
        else *reinterpret_cast<bf16x8*>(dr + 8 * c) = o;
      }
    }
  }
}

int cross_entropy(const void* logits, const int32_t* tok, float* loss_row, void* dlogits, int bf, int B, int S, int V,
                  hipStream_t st, const StepState* ss) {
  const int T = B * S;
  const float invT = 1.0f / (float)T;
  const bf16* lb = (const bf16*)logits;
  bf16* db = (bf16*)dlogits;
  if (bf && V <= 32 * 1024) {   // longer rows do not fit the registers of a block
    const bool big = V > 32 * 256, edge = V % 8 != 0;
#define ALS_CE_LAUNCH(BS, EDGE) \
  hipLaunchKernelGGL((cross_entropy_reg_kernel<BS, EDGE>), dim3(T), dim3(BS), 0, st, lb, tok, loss_row, db, S, V, invT, ss)
    if (big) { if (edge) ALS_CE_LAUNCH(1024, true); else ALS_CE_LAUNCH(1024, false); }
    else { if (edge) ALS_CE_LAUNCH(256, true); else ALS_CE_LAUNCH(256, false); }
#undef ALS_CE_LAUNCH
  } else if (bf) {
    hipLaunchKernelGGL(cross_entropy_kernel<bf16>, dim3(T), dim3(256), 0, st, lb, tok, loss_row, db, S, V, invT, ss);
  } else {
    hipLaunchKernelGGL(cross_entropy_kernel<float>, dim3(T), dim3(256), 0, st, (const float*)logits, tok, loss_row,
                       (float*)dlogits, S, V, invT, ss);
  }
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}

}  // namespace als
