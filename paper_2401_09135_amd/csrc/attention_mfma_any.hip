// Causal attention on bf16 storage for what the kernels of attention_mfma.hip do not take (heads of 32, any sequence length
// up to 1024), in fp32 arithmetic on the bf16 matrix instruction v_mfma_f32_16x16x32_bf16.  qkv is [B*S, 3d]: q at column
// hd*dh, k at d + hd*dh, v at 2d + hd*dh.
//
// The operands of the score products are bf16 as they lie in memory: their products are exact and the sums fp32.  The
// operands that are computed (probabilities and score gradients) stay whole fp32 values: each is cut into three bf16 parts of 8
// bits of its significand, high, middle and low, which give it back exactly from 2^-110 on and to 2^-133 (the smallest bf16) below, and the
// second products take one matrix instruction per part.  Against the fp32 instruction (v_mfma_f32_16x16x4_f32: a 16th of the rate; what attention_mfma_f32.hip does for fp32
// storage) that is 16 times fewer cycles for the scores and 5 times fewer for the rest.
//
// One wavefront owns 16 NT queries (forward, dQ) or 16 NT keys (dK and dV) of one head and walks the other side in steps of 32
// rows.  Where that gives the chip few wavefronts, the four of a workgroup share one block of 16 rows instead (SPLIT): each takes
// every fourth step, and their results are put together through LDS in order at the end.  Operands are loaded straight into
// MFMA fragments: no LDS and no barrier in the loop.
//   MFMA lane layout (lane l, group g = l / 16): A row l%16, contraction 8 g .. 8 g + 7; B column l%16, the same; accumulator
//   element v: row 4 g + v, column l%16.
// The order of a contraction is free as long as both operands agree.  Score products: chunk i of 32 head dimensions, 8
// consecutive ones per lane.  Second products: contraction 8 g + e is row 4 g + e of the step's first 16 rows (e < 4) or
// 4 g + e - 4 of its second, which is how the two accumulators of the scores lie; output row m of block t is head dimension
// DT m + t, so that a lane loads DT consecutive elements of V (K, Q, dO), packs its 8 rows pairwise with byte permutations and ends
// with DH/4 consecutive elements of the result.
//
// What bounds it: the exponentials and the cutting in vector code at long sequences, the chain of loads of a wavefront for small
// calls.  dQ and dK/dV are one launch: the row dots D_i = dO_i . O_i, which would tie the second to the first, are the
// diagonal of one more score product in both.  Forward / backward in us, on the fp32 instruction and here, at the same distance
// from a float64 reference:
//   B 3, S 200, 5 heads of 64: 7.4 / 19.9 -> 5.8 / 9.9;     B 8, S 256, 8 heads of 32: 12.2 / 33.3 -> 8.6 / 15.6
//   B 8, S 1000, 4 heads of 64: 66 / 202 -> 36 / 102;       B 8, S 1000, 16 heads of 64: 395 / 1260 -> 122 / 335
//   B 64, S 600, 8 heads of 32: 228 / 694 -> 125 / 303;     B 64, S 20, 4 heads of 64: 5.7 / 12.5 -> 4.5 / 5.2
#include "common.h"
#include <math.h>

namespace als {

namespace {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x4 mfma32(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ float quad_sum(float v) {   // over the four lane groups
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
__device__ __forceinline__ float quad_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ unsigned bits(float x) { return __builtin_bit_cast(unsigned, x); }
__device__ __forceinline__ float real(unsigned x) { return __builtin_bit_cast(float, x); }
__device__ __forceinline__ unsigned low_halves(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ unsigned high_halves(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// One row of 16 as a score operand: lane (g, c) holds dimensions 32 i + 8 g .. + 7 of row c.
template <int DH>
struct RowFrag {
  u32x4 c[DH / 32];
  __device__ __forceinline__ void load(const bf16* row, int g) {
#pragma unroll
    for (int i = 0; i < DH / 32; i++) c[i] = *reinterpret_cast<const u32x4*>(row + 32 * i + 8 * g);
  }
};
// [row of a][row of b] = a . b over the head width
template <int DH>
__device__ __forceinline__ f32x4 row_product(const RowFrag<DH>& a, const RowFrag<DH>& b) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < DH / 32; i++) acc = mfma32(a.c[i], b.c[i], acc);
  return acc;
}

// 8 fp32 values of a lane as three bf16 parts: the upper 8 bits of the significand, the next 8, the last 8.  Their sum is the value for
// |x| >= 2^-110; below that the last bits lie under 2^-133, the smallest bf16, and are left out.  An infinity has a high part only.
struct Parts3 {
  u32x4 hi, mid, lo;
  __device__ __forceinline__ Parts3(const float (&x)[8]) {
#pragma unroll
    for (int w = 0; w < 4; w++) {
      float r[2];
      hi[w] = high_halves(bits(x[2 * w]), bits(x[2 * w + 1]));
#pragma unroll
      for (int e = 0; e < 2; e++) {
        const float h = real(bits(x[2 * w + e]) & 0xffff0000u);
        r[e] = h == x[2 * w + e] ? 0.0f : x[2 * w + e] - h;
      }
      mid[w] = high_halves(bits(r[0]), bits(r[1]));
#pragma unroll
      for (int e = 0; e < 2; e++) r[e] -= real(bits(r[e]) & 0xffff0000u);
      lo[w] = high_halves(bits(r[0]), bits(r[1]));
    }
  }
};

// 32 rows as the first operand of the second products: lane (g, c) holds dimensions DT c .. + DT - 1 of rows 4 g + e and 16 + 4 g + e.
template <int DH>
struct ColFrag {
  static constexpr int DT = DH / 16, NW = DT / 2;
  unsigned w[8][NW];
  static __device__ __forceinline__ int row_of(int e, int g) { return (e & 4) * 4 + 4 * g + (e & 3); }
  // rows beyond `last` are read from row `last`: their weight is zero
  __device__ __forceinline__ void load(const bf16* base, int64_t ld, int row0, int last, int lane) {
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const int row = row0 + row_of(e, lane >> 4);
      const unsigned* p = reinterpret_cast<const unsigned*>(base + (int64_t)(row < last ? row : last) * ld + DT * (lane & 15));
      if constexpr (NW == 2) {
        const uint2 x = *reinterpret_cast<const uint2*>(p);
        w[e][0] = x.x; w[e][1] = x.y;
      } else w[e][0] = *p;
    }
  }
  // Values that are not finite: times a masked weight of 0, or a part of a weight that is 0, they would give NaN where the whole
  // product gives none.  They are taken out of the tile (true: there were some) and added where they are seen.
  __device__ __forceinline__ bool drop_non_finite() {
    u16x2 m = {0, 0};
#pragma unroll
    for (int e = 0; e < 8; e++)
#pragma unroll
      for (int q = 0; q < NW; q++) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w[e][q] & 0x7fff7fffu));
    if (__all(m[0] < 0x7f80 && m[1] < 0x7f80)) return false;
#pragma unroll
    for (int e = 0; e < 8; e++)
#pragma unroll
      for (int q = 0; q < NW; q++) {
        if ((w[e][q] & 0x7f80u) == 0x7f80u) w[e][q] &= 0xffff0000u;
        if ((w[e][q] & 0x7f800000u) == 0x7f800000u) w[e][q] &= 0xffffu;
      }
    return true;
  }
  // base, ld, row0, last: as for load()
  template <typename Seen>
  static __device__ __forceinline__ void add_non_finite(const bf16* base, int64_t ld, int row0, int last, const float (&p)[8], f32x4 (&out)[DT], int lane,
                                                        Seen seen) {
    const int g = lane >> 4, c = lane & 15;
#pragma unroll
    for (int e = 0; e < 8; e++)
#pragma unroll 1
      for (int rg = 0; rg < 4; rg++) {
        const float pr = __shfl(p[e], 16 * rg + c, 64);
        const int r = row_of(e, rg);
        const bf16* row = base + (int64_t)(row0 + r < last ? row0 + r : last) * ld;
#pragma unroll
        for (int t = 0; t < DT; t++)
#pragma unroll
          for (int q = 0; q < 4; q++) {   // this lane's output row 4 g + q of block t
            const float x = (float)row[DT * (4 * g + q) + t];
            if (!(fabsf(x) < INFINITY) && seen(r, c)) out[t][q] += pr * x;
          }
      }
  }
  // out[t][dims][columns] += tile^T p; p: 8 rows of a column per lane, as row_of numbers them
  __device__ __forceinline__ void product(const Parts3& p, f32x4 (&out)[DT]) const {
#pragma unroll
    for (int t = 0; t < DT; t++) {
      u32x4 a;
#pragma unroll
      for (int q = 0; q < 4; q++)
        a[q] = t & 1 ? high_halves(w[2 * q][t / 2], w[2 * q + 1][t / 2]) : low_halves(w[2 * q][t / 2], w[2 * q + 1][t / 2]);
      out[t] = mfma32(a, p.lo, out[t]);
      out[t] = mfma32(a, p.mid, out[t]);
      out[t] = mfma32(a, p.hi, out[t]);
    }
  }
  // a lane's DH/4 consecutive output dimensions of its column
  static __device__ __forceinline__ void store(bf16* row, const f32x4 (&out)[DT], float div, int lane) {
#pragma unroll
    for (int u = 0; u < DT / 2; u++) {
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; e++) o[e] = (bf16)(out[(8 * u + e) % DT][(8 * u + e) / DT] / div);
      *reinterpret_cast<bf16x8*>(row + 4 * DT * (lane >> 4) + 8 * u) = o;
    }
  }
};

// Workgroup id of n and wavefront -> (block of 16 NT rows, head, sample).  Consecutive workgroups go to different XCDs: each XCD
// is given a contiguous run of them, so that the blocks of one head share an L2.
struct Block { int row0, hd, b; };
template <bool SPLIT>
__device__ __forceinline__ bool block_of(int i, int n, int S, int h, int rows, bool last_first, Block& out) {
  const int nblk = (S + rows - 1) / rows, per_pair = SPLIT ? nblk : (nblk + 3) / 4;
  const int per = n / 8;
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
struct Shares { f32x4 v[4][N][64]; };

template <int DH, int NT, bool SPLIT>
__global__ __launch_bounds__(256, 2) void attn_any_fwd_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ o, float* __restrict__ lse, int S,
                                                              int h, float scale) {
  typedef ColFrag<DH> CF;
  typedef RowFrag<DH> RF;
  Block bk;
  if (!block_of<SPLIT>(blockIdx.x, gridDim.x, S, h, 16 * NT, true, bk)) return;   // never in a SPLIT workgroup
  const int wv = SPLIT ? threadIdx.x >> 6 : 0;
  constexpr int STEP = SPLIT ? 128 : 32;   // from one step of this wavefront to its next
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15, last = S - 1, q0 = bk.row0;
  const int d = h * DH;
  const int64_t ld = 3 * (int64_t)d;
  const bf16* base = qkv + (int64_t)bk.b * S * ld + bk.hd * DH;
  RF qf[NT], kf[2], kn[2];
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
  auto load_keys = [&](int k0, RF (&k)[2]) {
#pragma unroll
    for (int u = 0; u < 2; u++) {
      const int kr = k0 + 16 * u + c;
      k[u].load(base + d + (int64_t)(kr < last ? kr : last) * ld, g);
    }
  };
  load_keys(32 * wv, kf);
  for (int k0 = 32 * wv; k0 <= q_last; k0 += STEP) {
    CF vf;
    vf.load(base + 2 * d, ld, k0, last, lane);
    load_keys(k0 + STEP, kn);
    const bool odd = vf.drop_non_finite();
#pragma unroll
    for (int n = 0; n < NT; n++) {
      if (k0 > q0 + 16 * n + 15) continue;   // wave-uniform: no key of the step is seen
      const int q = q0 + 16 * n + c;
      const bool masked = k0 + 31 > q0 + 16 * n;
      float s[8];
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const f32x4 x = row_product<DH>(kf[u], qf[n]);
#pragma unroll
        for (int v = 0; v < 4; v++) s[4 * u + v] = masked && k0 + 16 * u + 4 * g + v > q ? -INFINITY : x[v] * scale;
      }
      float mx = s[0];
#pragma unroll
      for (int e = 1; e < 8; e++) mx = fmaxf(mx, s[e]);
      mx = fmaxf(m[n], quad_max(mx));
      if (__any(mx != m[n])) {
        const float alpha = mx == m[n] ? 1.0f : expf(m[n] - mx);
        l[n] *= alpha;
#pragma unroll
        for (int t = 0; t < CF::DT; t++) acc[n][t] *= alpha;
        m[n] = mx;
      }
      const float ref = mx == -INFINITY ? 0.0f : mx;
#pragma unroll
      for (int e = 0; e < 8; e++) { s[e] = expf(s[e] - ref); l[n] += s[e]; }
      vf.product(Parts3(s), acc[n]);
      if (odd) CF::add_non_finite(base + 2 * d, ld, k0, last, s, acc[n], lane, [&](int r, int col) { return k0 + r <= q0 + 16 * n + col; });
    }
    kf[0] = kn[0];
    kf[1] = kn[1];
  }
  if constexpr (SPLIT) {   // rescale to the largest maximum of a query and add
    static_assert(NT == 1, "one block of rows");
    __shared__ Shares<CF::DT> shares;
    __shared__ float pm[4][64], pl[4][64];
#pragma unroll
    for (int t = 0; t < CF::DT; t++) shares.v[wv][t][lane] = acc[0][t];
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
      for (int t = 0; t < CF::DT; t++) acc[0][t] += f * shares.v[w][t][lane];
    }
  }
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int q = q0 + 16 * n + c;
    const float sum = quad_sum(l[n]);
    if (q > last) continue;
    CF::store(o + ((int64_t)bk.b * S + q) * d + bk.hd * DH, acc[n], sum, lane);
    if (g == 0) lse[((int64_t)bk.b * h + bk.hd) * S + q] = m[n] + logf(sum);
  }
}

struct BwdArgs {
  const bf16* qkv; const bf16* o; const bf16* d_o; const float* lse; bf16* dqkv;
  int S, h;
  float scale;
};

// dq_i = sum_{j<=i} ds_ij k_j,  ds_ij = p_ij (do_i.v_j - D_i) scale,  D_i = do_i.o_i
template <int DH, int NT, bool SPLIT>
__device__ __forceinline__ void dq_block(const BwdArgs& a, const Block& bk, Shares<2 * (DH / 16)>* shares) {
  typedef ColFrag<DH> CF;
  typedef RowFrag<DH> RF;
  const int S = a.S, h = a.h;
  const int wv = SPLIT ? threadIdx.x >> 6 : 0;
  constexpr int STEP = SPLIT ? 128 : 32;
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15, last = S - 1, q0 = bk.row0;
  const int d = h * DH;
  const int64_t ld = 3 * (int64_t)d;
  const bf16* base = a.qkv + (int64_t)bk.b * S * ld + bk.hd * DH;
  const int64_t stat = ((int64_t)bk.b * h + bk.hd) * S;
  RF qf[NT], gf[NT], kf[2], vf[2], kn[2], vn[2];
  f32x4 acc[NT][CF::DT];
  float Dq[NT], lq[NT];
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int q = q0 + 16 * n + c, qc = q < last ? q : last;
    const int64_t orow = ((int64_t)bk.b * S + qc) * d + bk.hd * DH;
    qf[n].load(base + (int64_t)qc * ld, g);
    gf[n].load(a.d_o + orow, g);
    RF of;
    of.load(a.o + orow, g);
    const f32x4 dots = row_product<DH>(gf[n], of);   // the diagonal: element c % 4 of lane (c / 4, c)
    const float own = c & 2 ? (c & 1 ? dots[3] : dots[2]) : (c & 1 ? dots[1] : dots[0]);
    Dq[n] = __shfl(own, 16 * (c >> 2) + c, 64);
    lq[n] = a.lse[stat + qc];
#pragma unroll
    for (int t = 0; t < CF::DT; t++) acc[n][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  const int q_last = q0 + 16 * NT - 1 < last ? q0 + 16 * NT - 1 : last;
  auto load_rows = [&](int k0, RF (&k)[2], RF (&v)[2]) {
#pragma unroll
    for (int u = 0; u < 2; u++) {
      const int kr = k0 + 16 * u + c;
      const int64_t ko = (int64_t)(kr < last ? kr : last) * ld;
      k[u].load(base + d + ko, g);
      v[u].load(base + 2 * d + ko, g);
    }
  };
  load_rows(32 * wv, kf, vf);
  for (int k0 = 32 * wv; k0 <= q_last; k0 += STEP) {
    CF kt;
    kt.load(base + d, ld, k0, last, lane);
    load_rows(k0 + STEP, kn, vn);
    const bool odd = kt.drop_non_finite();
#pragma unroll
    for (int n = 0; n < NT; n++) {
      if (k0 > q0 + 16 * n + 15) continue;
      const int q = q0 + 16 * n + c;
      const bool masked = k0 + 31 > q0 + 16 * n;
      float ds[8];
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const f32x4 s = row_product<DH>(kf[u], qf[n]), dp = row_product<DH>(vf[u], gf[n]);
#pragma unroll
        for (int v = 0; v < 4; v++)
          ds[4 * u + v] = masked && k0 + 16 * u + 4 * g + v > q ? 0.0f : expf(s[v] * a.scale - lq[n]) * (dp[v] - Dq[n]) * a.scale;
      }
      kt.product(Parts3(ds), acc[n]);
      if (odd) CF::add_non_finite(base + d, ld, k0, last, ds, acc[n], lane, [&](int r, int col) { return k0 + r <= q0 + 16 * n + col; });
    }
#pragma unroll
    for (int u = 0; u < 2; u++) { kf[u] = kn[u]; vf[u] = vn[u]; }
  }
  if constexpr (SPLIT) {
#pragma unroll
    for (int t = 0; t < CF::DT; t++) shares->v[wv][t][lane] = acc[0][t];
    __syncthreads();
    if (wv) return;
#pragma unroll
    for (int w = 1; w < 4; w++)
#pragma unroll
      for (int t = 0; t < CF::DT; t++) acc[0][t] += shares->v[w][t][lane];
  }
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int q = q0 + 16 * n + c;
    if (q <= last) CF::store(a.dqkv + ((int64_t)bk.b * S + q) * ld + bk.hd * DH, acc[n], 1.0f, lane);
  }
}

// dk_j = sum_{i>=j} ds_ij q_i ; dv_j = sum_{i>=j} p_ij do_i
template <int DH, int NT, bool SPLIT>
__device__ __forceinline__ void dkv_block(const BwdArgs& a, const Block& bk, Shares<2 * (DH / 16)>* shares) {
  typedef ColFrag<DH> CF;
  typedef RowFrag<DH> RF;
  const int S = a.S, h = a.h;
  const int wv = SPLIT ? threadIdx.x >> 6 : 0;
  constexpr int STEP = SPLIT ? 128 : 32;
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15, last = S - 1, j0 = bk.row0;
  const int d = h * DH;
  const int64_t ld = 3 * (int64_t)d;
  const bf16* base = a.qkv + (int64_t)bk.b * S * ld + bk.hd * DH;
  const bf16* gbase = a.d_o + (int64_t)bk.b * S * d + bk.hd * DH;
  const bf16* obase = a.o + (int64_t)bk.b * S * d + bk.hd * DH;
  const int64_t stat = ((int64_t)bk.b * h + bk.hd) * S;
  RF kf[NT], vf[NT], qf[2], gf[2];
  f32x4 dk[NT][CF::DT], dv[NT][CF::DT];
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int j = j0 + 16 * n + c;
    const bf16* row = base + (int64_t)(j < last ? j : last) * ld;
    kf[n].load(row + d, g);
    vf[n].load(row + 2 * d, g);
#pragma unroll
    for (int t = 0; t < CF::DT; t++) { dk[n][t] = (f32x4){0.f, 0.f, 0.f, 0.f}; dv[n][t] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
  }
  auto load_rows = [&](int i0, RF (&q)[2], RF (&go)[2]) {
#pragma unroll
    for (int u = 0; u < 2; u++) {
      const int i = i0 + 16 * u + c < last ? i0 + 16 * u + c : last;
      q[u].load(base + (int64_t)i * ld, g);
      go[u].load(gbase + (int64_t)i * d, g);
    }
  };
  for (int i0 = j0 + 32 * wv; i0 <= last; i0 += STEP) {
    CF qt, gt;
    RF of[2];
    float ls[8], Ds[8];
    load_rows(i0, qf, gf);
#pragma unroll
    for (int u = 0; u < 2; u++) {
      const int i = i0 + 16 * u + c < last ? i0 + 16 * u + c : last;
      of[u].load(obase + (int64_t)i * d, g);
    }
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const int i = i0 + CF::row_of(e, g);
      ls[e] = a.lse[stat + (i < last ? i : last)];
    }
    gt.load(gbase, d, i0, last, lane);
    qt.load(base, ld, i0, last, lane);
    const bool odd_g = gt.drop_non_finite(), odd_q = qt.drop_non_finite();
#pragma unroll
    for (int u = 0; u < 2; u++) {
      const f32x4 dots = row_product<DH>(gf[u], of[u]);
#pragma unroll
      for (int v = 0; v < 4; v++) Ds[4 * u + v] = __shfl(dots[v], 20 * g + v, 64);   // row 4 g + v: its diagonal lies in lane (g, 4 g + v)
    }
#pragma unroll
    for (int n = 0; n < NT; n++) {
      const int j = j0 + 16 * n + c;
      if (i0 + 31 < j0 + 16 * n) continue;   // wave-uniform: every query of the step precedes every key
      const bool masked = i0 < j0 + 16 * n + 15 || i0 + 31 > last;
      float p[8], ds[8];
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const f32x4 s = row_product<DH>(qf[u], kf[n]), dp = row_product<DH>(gf[u], vf[n]);
#pragma unroll
        for (int v = 0; v < 4; v++) {
          const int e = 4 * u + v, i = i0 + 16 * u + 4 * g + v;
          const bool out = masked && (j > i || i > last);
          p[e] = out ? 0.0f : expf(s[v] * a.scale - ls[e]);
          ds[e] = out ? 0.0f : p[e] * (dp[v] - Ds[e]) * a.scale;
        }
      }
      auto seen = [&](int r, int col) { return j0 + 16 * n + col <= i0 + r && i0 + r <= last; };
      gt.product(Parts3(p), dv[n]);
      qt.product(Parts3(ds), dk[n]);
      if (odd_g) CF::add_non_finite(gbase, d, i0, last, p, dv[n], lane, seen);
      if (odd_q) CF::add_non_finite(base, ld, i0, last, ds, dk[n], lane, seen);
    }
  }
  if constexpr (SPLIT) {   // wavefront 0 adds and stores dk, wavefront 1 dv
#pragma unroll
    for (int t = 0; t < CF::DT; t++) {
      shares->v[wv][t][lane] = dk[0][t];
      shares->v[wv][CF::DT + t][lane] = dv[0][t];
    }
    __syncthreads();
    const int j = j0 + c;
    if (wv > 1 || j > last) return;
    f32x4 sum[CF::DT];
#pragma unroll
    for (int t = 0; t < CF::DT; t++) {
      sum[t] = shares->v[0][wv * CF::DT + t][lane];
#pragma unroll
      for (int w = 1; w < 4; w++) sum[t] += shares->v[w][wv * CF::DT + t][lane];
    }
    CF::store(a.dqkv + ((int64_t)bk.b * S + j) * ld + bk.hd * DH + (1 + wv) * d, sum, 1.0f, lane);
    return;
  }
#pragma unroll
  for (int n = 0; n < NT; n++) {
    const int j = j0 + 16 * n + c;
    if (j > last) continue;
    bf16* row = a.dqkv + ((int64_t)bk.b * S + j) * ld + bk.hd * DH;
    CF::store(row + d, dk[n], 1.0f, lane);
    CF::store(row + 2 * d, dv[n], 1.0f, lane);
  }
}

// The first half of the workgroups form dK and dV, which take longer, the second half dQ.
template <int DH, int NT, bool SPLIT>
__global__ __launch_bounds__(256, 2) void attn_any_bwd_kernel(BwdArgs a) {
  __shared__ Shares<SPLIT ? 2 * (DH / 16) : 1> shares;
  auto* sh = reinterpret_cast<Shares<2 * (DH / 16)>*>(&shares);
  const int n = gridDim.x / 2, i = blockIdx.x;
  Block bk;
  if (i < n) {
    if (block_of<SPLIT>(i, n, a.S, a.h, 16 * NT, false, bk)) dkv_block<DH, NT, SPLIT>(a, bk, sh);
  } else {
    if (block_of<SPLIT>(i - n, n, a.S, a.h, 16 * NT, true, bk)) dq_block<DH, NT, SPLIT>(a, bk, sh);
  }
}

// Two row blocks per wavefront halve the tile traffic of the other side and the number of wavefronts; below `limit` blocks four
// wavefronts share one (returned as 0) where a row is longer than a step, above it they would only add to the traffic.  In us, a
// block per workgroup / two per wavefront (blocks):
//   forward: B 8, S 1000, 16 heads of 64 (8064): 121 / 134;  B 64, S 600, 8 heads of 64 (19456): 188 / 153, of 32: 126 / 125
//   backward, width 64: B 4, S 500, 6 heads (768): 34 / 57;  B 32, S 100, 8 heads (1792): 28 / 18;  B 8, S 1000, 4 heads (2016): 120 / 102
//   backward, width 32: B 16, S 256, 16 heads (4096): 46 / 45;  B 32, S 500, 4 heads (4096): 71 / 87;  B 64, S 600, 8 heads (19456): 343 / 303
inline int row_blocks(int B, int S, int h, int limit) { return (int64_t)B * h * ((S + 15) / 16) > limit ? 2 : S > 32 ? 0 : 1; }
inline int grid_of(int B, int S, int h, int nt, bool split) {
  const int nblk = (S + 16 * nt - 1) / (16 * nt);
  return (split ? nblk : (nblk + 3) / 4) * h * B;
}

template <int DH, int NT, bool SPLIT>
int fwd_t(const void* qkv, void* o, float* lse, int B, int S, int h, hipStream_t st) {
  hipLaunchKernelGGL((attn_any_fwd_kernel<DH, NT, SPLIT>), dim3(grid_of(B, S, h, NT, SPLIT)), dim3(256), 0, st, (const bf16*)qkv, (bf16*)o, lse, S, h,
                     1.0f / sqrtf((float)DH));
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}
template <int DH, int NT, bool SPLIT>
int bwd_t(const BwdArgs& a, int B, hipStream_t st) {
  hipLaunchKernelGGL((attn_any_bwd_kernel<DH, NT, SPLIT>), dim3(2 * grid_of(B, a.S, a.h, NT, SPLIT)), dim3(256), 0, st, a);
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}

}  // namespace

#define ALS_ATTN_ROWS(DH, CALL) (rows == 2 ? CALL(DH, 2, false) : rows == 1 ? CALL(DH, 1, false) : CALL(DH, 1, true))

int attention_fwd_mfma_any(const void* qkv, void* o, float* lse, int B, int S, int h, int dh, hipStream_t st) {
#define ALS_CALL(DH, NT, SPLIT) (fwd_t<DH, NT, SPLIT>(qkv, o, lse, B, S, h, st))
  const int rows = row_blocks(B, S, h, 8192);
  return dh == 64 ? ALS_ATTN_ROWS(64, ALS_CALL) : ALS_ATTN_ROWS(32, ALS_CALL);
#undef ALS_CALL
}

int attention_bwd_mfma_any(const void* qkv, const void* o, const void* d_o, const float* lse, void* dqkv, int B, int S, int h, int dh,
                           hipStream_t st) {
  const BwdArgs a{(const bf16*)qkv, (const bf16*)o, (const bf16*)d_o, lse, (bf16*)dqkv, S, h, 1.0f / sqrtf((float)dh)};
#define ALS_CALL(DH, NT, SPLIT) (bwd_t<DH, NT, SPLIT>(a, B, st))
  const int rows = row_blocks(B, S, h, dh == 64 ? 1536 : 4096);
  return dh == 64 ? ALS_ATTN_ROWS(64, ALS_CALL) : ALS_ATTN_ROWS(32, ALS_CALL);
#undef ALS_CALL
}

}  // namespace als
