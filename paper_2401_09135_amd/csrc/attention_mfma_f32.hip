// Causal attention on fp32 storage, heads of 32 or 64 and any sequence length up to 1024: fp32 arithmetic, the products on
// the fp32 matrix instruction v_mfma_f32_16x16x4_f32 (whole fp32 products and sums, no operand is rounded).  qkv is [B*S, 3d]: q at column hd*dh,
// k at d + hd*dh, v at 2d + hd*dh.
//
// One wavefront owns 16 NT queries (forward, dQ) or 16 NT keys (dK and dV) of one head and walks 16-row tiles of the other
// side; the four wavefronts of a workgroup take neighbouring blocks of one head, so that they find each other's tiles in
// the CU's L1, and share nothing else: no LDS, no barrier.  Where that gives the chip few wavefronts, the four of a workgroup
// share one block of 16 rows instead (SPLIT): each walks every fourth tile of the other side, and their results are put
// together through LDS in order at the end.  Every operand is loaded straight into MFMA fragments, 8 or
// 16 bytes per lane:
//   MFMA lane layout (lane l, group g = l / 16): A row l%16, contraction g; B column l%16, contraction g; accumulator
//   element v: row 4 g + v, column l%16.
// The order of the contraction and of the output rows is free as long as both operands agree, and is chosen so that no value
// ever moves between lanes: in the score products step (i, e) takes head dimension CH (4 i + g) + e, CH consecutive ones per
// lane; the probabilities (accumulator rows = keys 4 g + v) are step v's operand of the next product as they lie; and that
// product's output row m of block t is head dimension DT m + t, so that a lane loads DT consecutive elements of V (K, Q, dO) and
// ends with DH/4 consecutive elements of the result.
//
// What bounds it: the fp32 matrix rate (64 flops per clock and SIMD, a 16th of bf16's) for long sequences, the chain of
// tile loads and dependent MFMAs of a single wavefront for short ones.  Against one wavefront per query with scalar products
// in vector code (attention_generic.hip), forward / backward in us, same distance from a float64 reference:
//   B 8, S 1000, 16 heads of 64: 2250 / 9484 -> 379 / 1218
//   B 8, S 32, 2 heads of 32: 5.3 / 9.9 -> 7.2 / 9.6, which is why small calls stay with the other kernels.
#include "common.h"
#include <math.h>

namespace als {

namespace {

// 16-byte (or smaller) groups of storage elements widened to fp32
template <int N> struct Vec { float v[N]; };
template <int N>
__device__ __forceinline__ Vec<N> ldv(const float* p) {
  Vec<N> r;
#pragma unroll
  for (int i = 0; i < N; i++) r.v[i] = 0.0f;
  if constexpr (N == 2) {
    const float2 x = *reinterpret_cast<const float2*>(p);
    r.v[0] = x.x; r.v[1] = x.y;
  } else {
#pragma unroll
    for (int q = 0; q < N / 4; q++) {
      const f32x4 x = reinterpret_cast<const f32x4*>(p)[q];
#pragma unroll
      for (int e = 0; e < 4; e++) r.v[4 * q + e] = x[e];
    }
  }
  return r;
}
template <int N>
__device__ __forceinline__ void stv(float* p, const float* v) {
#pragma unroll
  for (int q = 0; q < N / 4; q++) reinterpret_cast<f32x4*>(p)[q] = (f32x4){v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
}
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ float quad_sum(float v) {   // over the four lane groups
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
__device__ __forceinline__ float quad_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}

// The head dimensions of one row that a lane feeds to the score products: DH/4 values in contraction-step order.
template <int DH>
struct RowFrag {
  static constexpr int CH = 4, NL = DH / 4 / CH;
  Vec<CH> c[NL];
  __device__ __forceinline__ void load(const float* row, int g) {
#pragma unroll
    for (int i = 0; i < NL; i++) c[i] = ldv<CH>(row + CH * (4 * i + g));
  }
};
// acc[row of a][row of b] += a . b over the head width
template <int DH>
__device__ __forceinline__ f32x4 row_product(const RowFrag<DH>& a, const RowFrag<DH>& b) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < RowFrag<DH>::NL; i++)
#pragma unroll
    for (int e = 0; e < RowFrag<DH>::CH; e++) acc = mfma4(a.c[i].v[e], b.c[i].v[e], acc);
  return acc;
}

// A 16-row tile as the first operand of the second products: rows 4 g + v (v = step), DT consecutive dimensions per lane.
template <int DH>
struct ColFrag {
  static constexpr int DT = DH / 16;
  Vec<DT> r[4];
  // rows beyond `last` are read from row `last`: their weight is zero
  __device__ __forceinline__ void load(const float* base, int64_t ld, int row0, int last, int lane) {
    const int g = lane >> 4;
#pragma unroll
    for (int v = 0; v < 4; v++) {
      const int row = row0 + 4 * g + v;
      r[v] = ldv<DT>(base + (int64_t)(row < last ? row : last) * ld + DT * (lane & 15));
    }
  }
  // out[t][dims][columns] += tile^T p ; p: accumulator layout (row 4 g + v, column l%16)
  __device__ __forceinline__ void product(const f32x4& p, f32x4 (&out)[DT]) const {
#pragma unroll
    for (int v = 0; v < 4; v++)
#pragma unroll
      for (int t = 0; t < DT; t++) out[t] = mfma4(r[v].v[t], p[v], out[t]);
  }
  // The same for a tile in which some (row, column) pairs are masked (p = 0 there): a value that is not finite would
  // turn 0 * inf into a NaN in columns that do not see its row.  Such values are left out of the products and added
  // where they are seen, which a tile without them (every tile, in practice) pays one test for.
  template <typename Seen>
  __device__ __forceinline__ void product_masked(const f32x4& p, f32x4 (&out)[DT], int lane, Seen seen) const {
    bool odd = false;
    ColFrag f = *this;
#pragma unroll
    for (int v = 0; v < 4; v++)
#pragma unroll
      for (int t = 0; t < DT; t++)
        if (!(fabsf(r[v].v[t]) < INFINITY)) { odd = true; f.r[v].v[t] = 0.0f; }
    f.product(p, out);
    if (__any(odd)) {
      const int g = lane >> 4, c = lane & 15;
#pragma unroll
      for (int v = 0; v < 4; v++)
#pragma unroll 1
        for (int rg = 0; rg < 4; rg++) {   // row 4 rg + v of the tile
          const float pr = __shfl(p[v], 16 * rg + c, 64);
#pragma unroll
          for (int t = 0; t < DT; t++)
#pragma unroll
            for (int q = 0; q < 4; q++) {  // this lane's output row 4 g + q of block t
              const float x = __shfl(r[v].v[t], 16 * rg + 4 * g + q, 64);
              if (!(fabsf(x) < INFINITY) && seen(4 * rg + v, c)) out[t][q] += pr * x;
            }
        }
    }
  }
  // a lane's DH/4 consecutive output dimensions of its column
  static __device__ __forceinline__ void store(float* row, const f32x4 (&out)[DT], float mul, float div, int lane) {
    float o[4 * DT];
#pragma unroll
    for (int q = 0; q < 4; q++)
#pragma unroll
      for (int t = 0; t < DT; t++) o[q * DT + t] = out[t][q] * mul / div;
    stv<4 * DT>(row + 4 * DT * (lane >> 4), o);
  }
};

// Wavefront -> (block of 16 NT rows, head, sample).  Consecutive workgroups go to different XCDs: each XCD is given a
// contiguous run of them, so that the blocks of one head share an L2.
struct Block { int row0, hd, b; };
template <bool SPLIT>
__device__ __forceinline__ bool block_of(int S, int h, int rows, bool last_first, Block& out) {
  const int nblk = (S + rows - 1) / rows, per_pair = SPLIT ? nblk : (nblk + 3) / 4;
  const int n = gridDim.x, per = n / 8, i = blockIdx.x;
  const int id = i < per * 8 ? (i % 8) * per + i / 8 : i;
  const int pair = id / per_pair;
  int blk = SPLIT ? id % per_pair : (id % per_pair) * 4 + (threadIdx.x >> 6);
  if (blk >= nblk) return false;
  if (last_first) blk = nblk - 1 - blk;   // the longest rows of keys first
  out = Block{blk * rows, pair % h, pair / h};
  return true;
}

// The accumulators that the wavefronts of a SPLIT workgroup leave for the one that adds them.
template <int N>
struct Parts { f32x4 v[4][N][64]; };

template <int DH, int NT, bool SPLIT>
__global__ __launch_bounds__(256, 2) void attn_fwd_f32_kernel(const float* __restrict__ qkv, float* __restrict__ o,
                                                                  float* __restrict__ lse, int S, int h, float scale) {
  typedef ColFrag<DH> CF;
  Block bk;
  if (!block_of<SPLIT>(S, h, 16 * NT, true, bk)) return;   // never in a SPLIT workgroup
  const int wv = SPLIT ? threadIdx.x >> 6 : 0;
  constexpr int STEP = SPLIT ? 64 : 16;   // from one tile of this wavefront to its next
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15, last = S - 1, q0 = bk.row0;
  const int d = h * DH;
  const int64_t ld = 3 * (int64_t)d;
  const float* base = qkv + (int64_t)bk.b * S * ld + bk.hd * DH;
  RowFrag<DH> qf[NT], kf, kn;
  f32x4 acc[NT][CF::DT];
  float m[NT], l[NT];
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int q = q0 + 16 * n + c;
    qf[n].load(base + (int64_t)(q < last ? q : last) * ld, g);
    m[n] = -INFINITY; l[n] = 0.0f;
#pragma unroll
    for (int t = 0; t < CF::DT; t++) acc[n][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  const int q_last = q0 + 16 * NT - 1 < last ? q0 + 16 * NT - 1 : last;
  const int kr0 = 16 * wv + c;
  kf.load(base + d + (int64_t)(kr0 < last ? kr0 : last) * ld, g);
  for (int k0 = 16 * wv; k0 <= q_last; k0 += STEP) {
    CF vf;
    vf.load(base + 2 * d, ld, k0, last, lane);
    const int kr = k0 + STEP + c;
    kn.load(base + d + (int64_t)(kr < last ? kr : last) * ld, g);
#pragma unroll
    for (int n = 0; n < NT; n++) {
      if (k0 > q0 + 16 * n + 15) continue;   // wave-uniform: no key of the tile is seen
      const int q = q0 + 16 * n + c;
      const bool masked = k0 + 15 > q0 + 16 * n;
      f32x4 s = row_product<DH>(kf, qf[n]);
#pragma unroll
      for (int v = 0; v < 4; v++) s[v] = masked && k0 + 4 * g + v > q ? -INFINITY : s[v] * scale;
      const float mx = fmaxf(m[n], quad_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
      if (__any(mx != m[n])) {
        const float alpha = mx == m[n] ? 1.0f : expf(m[n] - mx);
        l[n] *= alpha;
#pragma unroll
        for (int t = 0; t < CF::DT; t++) acc[n][t] *= alpha;
        m[n] = mx;
      }
      const float ref = mx == -INFINITY ? 0.0f : mx;
#pragma unroll
      for (int v = 0; v < 4; v++) { s[v] = expf(s[v] - ref); l[n] += s[v]; }
      if (masked) vf.product_masked(s, acc[n], lane, [&](int r, int col) { return k0 + r <= q0 + 16 * n + col; });
      else vf.product(s, acc[n]);
    }
    kf = kn;
  }
  if constexpr (SPLIT) {   // rescale to the largest maximum of a query and add
    static_assert(NT == 1, "one block of rows");
    __shared__ Parts<CF::DT> parts;
    __shared__ float pm[4][64], pl[4][64];
#pragma unroll
    for (int t = 0; t < CF::DT; t++) parts.v[wv][t][lane] = acc[0][t];
    pm[wv][lane] = m[0];
    pl[wv][lane] = l[0];
    __syncthreads();
    if (wv) return;
    const float mx = fmaxf(fmaxf(pm[0][lane], pm[1][lane]), fmaxf(pm[2][lane], pm[3][lane]));
    m[0] = mx; l[0] = 0.0f;
#pragma unroll
    for (int t = 0; t < CF::DT; t++) acc[0][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; w++) {
      const float f = pm[w][lane] == mx ? 1.0f : expf(pm[w][lane] - mx);
      l[0] += f * pl[w][lane];
#pragma unroll
      for (int t = 0; t < CF::DT; t++) acc[0][t] += f * parts.v[w][t][lane];
    }
  }
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int q = q0 + 16 * n + c;
    const float sum = quad_sum(l[n]);
    if (q > last) continue;
    CF::store(o + ((int64_t)bk.b * S + q) * d + bk.hd * DH, acc[n], 1.0f, sum, lane);
    if (g == 0) lse[((int64_t)bk.b * h + bk.hd) * S + q] = m[n] + logf(sum);
  }
}

// dq_i = sum_{j<=i} ds_ij k_j,  ds_ij = p_ij (do_i.v_j - D_i) scale,  D_i = do_i.o_i (left for the other pass)
template <int DH, int NT, bool SPLIT>
__global__ __launch_bounds__(256, 2) void attn_dq_f32_kernel(const float* __restrict__ qkv, const float* __restrict__ o,
                                                                     const float* __restrict__ d_o, const float* __restrict__ lse,
                                                                     float* __restrict__ Dbuf, float* __restrict__ dqkv, int S,
                                                                     int h, float scale) {
  typedef ColFrag<DH> CF;
  typedef RowFrag<DH> RF;
  Block bk;
  if (!block_of<SPLIT>(S, h, 16 * NT, true, bk)) return;   // never in a SPLIT workgroup
  const int wv = SPLIT ? threadIdx.x >> 6 : 0;
  constexpr int STEP = SPLIT ? 64 : 16;   // from one tile of this wavefront to its next
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15, last = S - 1, q0 = bk.row0;
  const int d = h * DH;
  const int64_t ld = 3 * (int64_t)d;
  const float* base = qkv + (int64_t)bk.b * S * ld + bk.hd * DH;
  const int64_t stat = ((int64_t)bk.b * h + bk.hd) * S;
  RF qf[NT], gf[NT], kf, vf, kn, vn;
  f32x4 acc[NT][CF::DT];
  float Dq[NT], lq[NT];
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int q = q0 + 16 * n + c, qc = q < last ? q : last;
    const int64_t orow = ((int64_t)bk.b * S + qc) * d + bk.hd * DH;
    qf[n].load(base + (int64_t)qc * ld, g);
    gf[n].load(d_o + orow, g);
    RF of;
    of.load(o + orow, g);
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < RF::NL; i++)
#pragma unroll
      for (int e = 0; e < RF::CH; e++) s += gf[n].c[i].v[e] * of.c[i].v[e];
    Dq[n] = quad_sum(s);
    lq[n] = lse[stat + qc];
    if (wv == 0 && g == 0 && q <= last) Dbuf[stat + q] = Dq[n];
#pragma unroll
    for (int t = 0; t < CF::DT; t++) acc[n][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  const int q_last = q0 + 16 * NT - 1 < last ? q0 + 16 * NT - 1 : last;
  {
    const int kr0 = 16 * wv + c;
    const int64_t kr = (int64_t)(kr0 < last ? kr0 : last) * ld;
    kf.load(base + d + kr, g);
    vf.load(base + 2 * d + kr, g);
  }
  for (int k0 = 16 * wv; k0 <= q_last; k0 += STEP) {
    CF kt;
    kt.load(base + d, ld, k0, last, lane);
    const int kr = k0 + STEP + c;
    const int64_t ko = (int64_t)(kr < last ? kr : last) * ld;
    kn.load(base + d + ko, g);
    vn.load(base + 2 * d + ko, g);
#pragma unroll
    for (int n = 0; n < NT; n++) {
      if (k0 > q0 + 16 * n + 15) continue;
      const int q = q0 + 16 * n + c;
      const bool masked = k0 + 15 > q0 + 16 * n;
      const f32x4 s = row_product<DH>(kf, qf[n]), dp = row_product<DH>(vf, gf[n]);
      f32x4 ds;
#pragma unroll
      for (int v = 0; v < 4; v++)
        ds[v] = masked && k0 + 4 * g + v > q ? 0.0f : expf(s[v] * scale - lq[n]) * (dp[v] - Dq[n]) * scale;
      if (masked) kt.product_masked(ds, acc[n], lane, [&](int r, int col) { return k0 + r <= q0 + 16 * n + col; });
      else kt.product(ds, acc[n]);
    }
    kf = kn;
    vf = vn;
  }
  if constexpr (SPLIT) {
    __shared__ Parts<CF::DT> parts;
#pragma unroll
    for (int t = 0; t < CF::DT; t++) parts.v[wv][t][lane] = acc[0][t];
    __syncthreads();
    if (wv) return;
#pragma unroll
    for (int w = 1; w < 4; w++)
#pragma unroll
      for (int t = 0; t < CF::DT; t++) acc[0][t] += parts.v[w][t][lane];
  }
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int q = q0 + 16 * n + c;
    if (q <= last) CF::store(dqkv + ((int64_t)bk.b * S + q) * ld + bk.hd * DH, acc[n], 1.0f, 1.0f, lane);
  }
}

// dk_j = sum_{i>=j} ds_ij q_i ; dv_j = sum_{i>=j} p_ij do_i
template <int DH, int NT, bool SPLIT>
__global__ __launch_bounds__(256, NT == 1 ? 2 : 1) void attn_dkv_f32_kernel(
    const float* __restrict__ qkv, const float* __restrict__ d_o, const float* __restrict__ lse, const float* __restrict__ Dbuf,
    float* __restrict__ dqkv, int S, int h, float scale) {
  typedef ColFrag<DH> CF;
  typedef RowFrag<DH> RF;
  Block bk;
  if (!block_of<SPLIT>(S, h, 16 * NT, false, bk)) return;   // never in a SPLIT workgroup
  const int wv = SPLIT ? threadIdx.x >> 6 : 0;
  constexpr int STEP = SPLIT ? 64 : 16;   // from one tile of this wavefront to its next
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15, last = S - 1, j0 = bk.row0;
  const int d = h * DH;
  const int64_t ld = 3 * (int64_t)d;
  const float* base = qkv + (int64_t)bk.b * S * ld + bk.hd * DH;
  const float* gbase = d_o + (int64_t)bk.b * S * d + bk.hd * DH;
  const int64_t stat = ((int64_t)bk.b * h + bk.hd) * S;
  RF kf[NT], vf[NT], qf, gf, qn, gn;
  f32x4 dk[NT][CF::DT], dv[NT][CF::DT];
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int j = j0 + 16 * n + c;
    const float* row = base + (int64_t)(j < last ? j : last) * ld;
    kf[n].load(row + d, g);
    vf[n].load(row + 2 * d, g);
#pragma unroll
    for (int t = 0; t < CF::DT; t++) { dk[n][t] = (f32x4){0.f, 0.f, 0.f, 0.f}; dv[n][t] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
  }
  auto load_rows = [&](int i0, RF& q, RF& go) {
    const int i = i0 + c < last ? i0 + c : last;
    q.load(base + (int64_t)i * ld, g);
    go.load(gbase + (int64_t)i * d, g);
  };
  load_rows(j0 + 16 * wv, qf, gf);
  for (int i0 = j0 + 16 * wv; i0 <= last; i0 += STEP) {
    CF qt, gt;
    float ls[4], Ds[4];
#pragma unroll
    for (int v = 0; v < 4; v++) {
      const int i = i0 + 4 * g + v < last ? i0 + 4 * g + v : last;
      ls[v] = lse[stat + i];
      Ds[v] = Dbuf[stat + i];
    }
    gt.load(gbase, d, i0, last, lane);
    qt.load(base, ld, i0, last, lane);
    load_rows(i0 + STEP, qn, gn);
#pragma unroll
    for (int n = 0; n < NT; n++) {
      const int j = j0 + 16 * n + c;
      if (i0 + 15 < j0 + 16 * n) continue;   // wave-uniform: every query of the tile precedes every key
      const bool masked = i0 < j0 + 16 * n + 15 || i0 + 15 > last;
      f32x4 p = row_product<DH>(qf, kf[n]);
      const f32x4 dp = row_product<DH>(gf, vf[n]);
      f32x4 ds;
#pragma unroll
      for (int v = 0; v < 4; v++) {
        const int i = i0 + 4 * g + v;
        const bool out = masked && (j > i || i > last);
        p[v] = out ? 0.0f : expf(p[v] * scale - ls[v]);
        ds[v] = out ? 0.0f : p[v] * (dp[v] - Ds[v]) * scale;
      }
      if (masked) {
        auto seen = [&](int r, int col) { return j0 + 16 * n + col <= i0 + r && i0 + r <= last; };
        gt.product_masked(p, dv[n], lane, seen);
        qt.product_masked(ds, dk[n], lane, seen);
      } else {
        gt.product(p, dv[n]);
        qt.product(ds, dk[n]);
      }
    }
    qf = qn;
    gf = gn;
  }
  if constexpr (SPLIT) {   // wavefront 0 adds and stores dk, wavefront 1 dv
    __shared__ Parts<2 * CF::DT> parts;
#pragma unroll
    for (int t = 0; t < CF::DT; t++) {
      parts.v[wv][t][lane] = dk[0][t];
      parts.v[wv][CF::DT + t][lane] = dv[0][t];
    }
    __syncthreads();
    const int j = j0 + c;
    if (wv > 1 || j > last) return;
    f32x4 sum[CF::DT];
#pragma unroll
    for (int t = 0; t < CF::DT; t++) {
      sum[t] = parts.v[0][wv * CF::DT + t][lane];
#pragma unroll
      for (int w = 1; w < 4; w++) sum[t] += parts.v[w][wv * CF::DT + t][lane];
    }
    CF::store(dqkv + ((int64_t)bk.b * S + j) * ld + bk.hd * DH + (1 + wv) * d, sum, 1.0f, 1.0f, lane);
    return;
  }
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int j = j0 + 16 * n + c;
    if (j > last) continue;
    float* row = dqkv + ((int64_t)bk.b * S + j) * ld + bk.hd * DH;
    CF::store(row + d, dk[n], 1.0f, 1.0f, lane);
    CF::store(row + 2 * d, dv[n], 1.0f, 1.0f, lane);
  }
}

// Two row blocks per wavefront halve the tile traffic of the other side but also the number of wavefronts: taken once
// one block each would give every SIMD (1024 on the chip) more than four.  Up to there, four wavefronts per row block (returned as
// 0) where there is more than a tile for each second one: the chain of tiles is a quarter as long (figures above), and at 4096 blocks,
// where the chip is full either way, still shorter (16 heads of 32, B 16, S 256, fp32: forward, dQ, dK and dV 35 + 43 + 63 us to 31 + 46 + 54).
inline int row_blocks(int B, int S, int h) { return (int64_t)B * h * ((S + 15) / 16) > 4096 ? 2 : S > 32 ? 0 : 1; }
inline dim3 grid_of(int B, int S, int h, int nt, bool split) {
  const int nblk = (S + 16 * nt - 1) / (16 * nt);
  return dim3((unsigned)(split ? nblk : (nblk + 3) / 4) * h * B);
}

template <int DH, int NT, bool SPLIT>
int fwd_t(const void* qkv, void* o, float* lse, int B, int S, int h, hipStream_t st) {
  hipLaunchKernelGGL((attn_fwd_f32_kernel<DH, NT, SPLIT>), grid_of(B, S, h, NT, SPLIT), dim3(256), 0, st, (const float*)qkv, (float*)o, lse, S, h,
                     1.0f / sqrtf((float)DH));
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}
template <int DH, int NT, bool SPLIT>
int bwd_t(const void* qkv, const void* o, const void* d_o, const float* lse, float* dscratch, void* dqkv, int B, int S, int h,
          hipStream_t st) {
  const float scale = 1.0f / sqrtf((float)DH);
  const dim3 grid = grid_of(B, S, h, NT, SPLIT);
  hipLaunchKernelGGL((attn_dq_f32_kernel<DH, NT, SPLIT>), grid, dim3(256), 0, st, (const float*)qkv, (const float*)o,
                     (const float*)d_o, lse, dscratch, (float*)dqkv, S, h, scale);
  ALS_CHECK_LAUNCH();
  hipLaunchKernelGGL((attn_dkv_f32_kernel<DH, NT, SPLIT>), grid, dim3(256), 0, st, (const float*)qkv, (const float*)d_o,
                     lse, dscratch, (float*)dqkv, S, h, scale);
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}

}  // namespace

#define ALS_ATTN_ROWS(DH, CALL) (rows == 2 ? CALL(DH, 2, false) : rows == 1 ? CALL(DH, 1, false) : CALL(DH, 1, true))

// Head widths of 32 and 64, 16-byte aligned tensors (rows are then aligned too); the grid is one-dimensional.  Up to 32
// positions of up to 64 heads the kernels with one wavefront per row are as fast or faster: a row there is one load and one
// exponential per lane, while here two tiles of dependent MFMAs follow each other in a single wavefront (figures above).
bool attention_mfma_any_supported(const void* a, const void* b, const void* c, const void* e, int B, int S, int h, int dh) {
  if (dh != 32 && dh != 64) return false;
  if (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c | (uintptr_t)e) % 16) return false;
  if (S <= 32 && (int64_t)B * h <= 64) return false;
  return B > 0 && S > 0 && h > 0 && S <= 1024 && (int64_t)((S + 63) / 64) * h * B < (1 << 23);
}

int attention_fwd_mfma_f32(const void* qkv, void* o, float* lse, int B, int S, int h, int dh, hipStream_t st) {
#define ALS_CALL(DH, NT, SPLIT) (fwd_t<DH, NT, SPLIT>(qkv, o, lse, B, S, h, st))
  const int rows = row_blocks(B, S, h);
  return dh == 64 ? ALS_ATTN_ROWS(64, ALS_CALL) : ALS_ATTN_ROWS(32, ALS_CALL);
#undef ALS_CALL
}

int attention_bwd_mfma_f32(const void* qkv, const void* o, const void* d_o, const float* lse, float* dscratch, void* dqkv, int B,
                           int S, int h, int dh, hipStream_t st) {
#define ALS_CALL(DH, NT, SPLIT) (bwd_t<DH, NT, SPLIT>(qkv, o, d_o, lse, dscratch, dqkv, B, S, h, st))
  const int rows = row_blocks(B, S, h);
  return dh == 64 ? ALS_ATTN_ROWS(64, ALS_CALL) : ALS_ATTN_ROWS(32, ALS_CALL);
#undef ALS_CALL
}

}  // namespace als
