// Causal multi-head attention on the gfx950 matrix cores, head width 64, bf16 operands with
// fp32 accumulation and fp32 online softmax: forward, and backward as two passes (dQ per
// query block; dK and dV per key block) that recompute the probabilities from the saved
// log-sum-exp, so no S x S matrix ever reaches HBM and no atomics are used.
//
// All score products are formed transposed where that helps the softmax: with
// S^T[key, q] = K Q^T the MFMA accumulator gives every lane ONE query column and 16 keys in
// registers, so row maxima and sums are in-register reductions plus a single cross-half
// shuffle, and the probabilities are already in the register layout the next product wants as
// its B operand (contraction index = key, permuted identically on the A side).
//
// MFMA lane layouts (lane l, half hf = l/32):  A fragment: row l%32, contraction 8 hf + e;
// B fragment: column l%32, contraction 8 hf + e;  accumulator element v: row
// 8 (v/4) + 4 hf + v%4, column l%32.  Using accumulator elements v = 8 kk + e of a 32-row
// block as contraction slots (hf, e) of the kk-th following product maps slot (hf, e) to row
// 16 kk + 8 (e/4) + 4 hf + e%4; the transposed A fragments are gathered with that same map by
// two LDS transpose loads (rows +0..3 and +8..11).
//
// A wavefront owns 64 queries in the forward and dQ kernels (two column blocks: each K and V fragment read from LDS serves both, and
// the products of one run while the exponentials of the other do), 32 keys in the dK/dV kernel; tiles of 64 rows go straight to LDS, one
// barrier a tile.  Against 32 queries, register-staged tiles and blocks in the order of the pairs, forward / backward in us:
//   B 16, S 1024, 14 heads: 66 / 196 -> 46 / 139     B 32, S 512, 8 heads: 27 / 82 -> 21 / 63     B 64, S 1024, 16 heads: 264 / 808 -> 220 / 701
//   B 1, S 1024, 14 heads: 18 / 51 -> 13 / 31        B 32, S 256, 4 heads: 8.0 / 21.4 -> 8.2 / 20.8
// What is left above the memory floor (B 16, S 1024: 117 MB forward, 18.6 us, which a forward without its tiles' work takes) is K and V
// from beyond the L2 (28 us with loads alone) and each block's own start; neither exponentials (7 %), products (8 %) nor LDS reads (7 %), and
// the order of a wavefront's instructions changes nothing (a software pipeline over halves of tiles: 46 us).
#include "common.h"
#include <atomic>
#include <math.h>
#include <type_traits>

namespace als {

namespace {

constexpr int DH = 64;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x8 lds_direct(const char* p) { return *reinterpret_cast<const bf16x8*>(p); }
__device__ __forceinline__ bf16x8 lds_tr2(const char* lo, const char* hi) {
  s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)lo);
  s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)hi);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int v = 0; v < 16; v++) z[v] = 0.0f;
  return z;
}
__device__ __forceinline__ bf16x8 pack8(const f32x16& x, int kk) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; e++) r[e] = (bf16)x[8 * kk + e];
  return r;
}
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0)
// A use of fragments that were loaded from global memory before a loop: the compiler then waits
// for those loads HERE.  Without it, it re-checks them inside the loop with a count that also
// covers the loop's own freshly issued tile loads, i.e. every iteration waits for its prefetch.
__device__ __forceinline__ void settle(const bf16x8 (&f)[4]) {
  asm volatile("" ::"v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]));
}

// Workgroup -> (block along the sequence, head, sample): the longest blocks of all (head, sample) pairs first, then the next
// shorter ones.  A block of the causal triangle is up to S / 64 tiles long and there are few rounds of them, so what starts last has
// to be short, and the blocks that one CU holds at a time should differ in length; pair by pair (B 16, S 1024, 14 heads: 1792 blocks of 2
// to 16 tiles; B 32, S 512, 8 heads) the three kernels took 62 + 174 and 24 + 74 us, this way 46 + 139 and 21 + 63.  Ids go round-robin to
// the 8 XCDs, so the blocks of a pair share an L2 wherever the number of pairs is a multiple of 8.  Many pairs are taken in groups of
// at least 256, whose K and V (256 KB a pair at S 1024) the last-level cache holds.
struct BlockId { int blk, hd, b; };
__device__ __forceinline__ BlockId block_id(int nblk, int h, int B) {
  const int pairs = h * B, groups = pairs < 512 ? 1 : pairs / 256, size = ((pairs + groups - 1) / groups + 7) & ~7;
  const int i = blockIdx.x, g = i / (size * nblk), j = i - g * size * nblk;
  const int n = pairs - g * size < size ? pairs - g * size : size;
  const int blk = j / n, pair = g * size + (j - blk * n);
  return {blk, pair % h, pair / h};
}

// write a transposed accumulator pair (rows = head dim, column = this lane's token) as bf16
__device__ __forceinline__ void store_rows(bf16* dst, const f32x16 (&acc)[2], float mul, int hf) {
#pragma unroll
  for (int dt = 0; dt < 2; dt++)
#pragma unroll
    for (int g = 0; g < 4; g++) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; e++) o[e] = (bf16)(acc[dt][4 * g + e] * mul);
      *reinterpret_cast<bf16x4*>(dst + dt * 32 + 8 * g + 4 * hf) = o;
    }
}

// ---- operand tiles loaded straight into LDS ----------------------------------------------------
// A tile is 64 rows of 128 bytes without padding; wavefront instruction i (global_load_lds_dwordx4) fills rows 8 i .. 8 i + 7.  Row R
// keeps its 16-byte chunk c at position c ^ perm(R), perm(R) = the bits of (R >> 1) & 7 in reverse: the 16 rows that a pass of a
// direct fragment read touches lie in 16 different 16-byte columns of the 64 banks, and so do the 4 rows x 64 bytes of
// a transpose read (rows R and R + 2 differ in bit 2 of the position).
constexpr int T64 = 64 * 128;
__device__ __forceinline__ int row_perm(int R) { return ((R >> 1) & 1) << 2 | ((R >> 2) & 1) << 1 | ((R >> 3) & 1); }
// byte offset, from the tile's first row, that this lane fetches for instruction i
__device__ __forceinline__ unsigned tile_voff(int lane, int i, int64_t ld) {
  const int R = 8 * i + (lane >> 3);
  return (unsigned)(R * (int)ld * 2 + (((lane & 7) ^ row_perm(R)) << 4));
}
// LDS offsets of this lane's fragments.  Direct: rows base + lane % 32, chunk 2 kk + lane / 32; base a multiple of 32.
__device__ __forceinline__ int frag_off(int lane, int kk) {
  const int R = lane & 31;
  return R * 128 + (((2 * kk + (lane >> 5)) ^ row_perm(R)) << 4);
}
// Transposed: rows base + 4 (lane / 32) + 0..3 (half 0) or + 8..11 (half 1), columns 32 cb ..; base a multiple of 16.
__device__ __forceinline__ int tr_frag_off(int lane, int cb, int half) {
  const int R = 8 * half + 4 * (lane >> 5) + ((lane & 15) >> 2);
  const int chunk = 4 * cb + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  return R * 128 + ((chunk ^ row_perm(R)) << 4) + 8 * (lane & 1);
}
// the value of the lane 32 away that has the same column, without a trip through the LDS pipe
__device__ __forceinline__ float other_half(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
  return __builtin_bit_cast(float, (threadIdx.x & 32) ? r[0] : r[1]);
}

// The W wavefronts that share a pair of tiles (K and V, or Q and dO) move 8 / W KB of each: one scalar address per two instructions,
// the permutation repeats every 16 rows.
template <int W>
struct TileFeed {
  static constexpr int LI = 8 / W;   // an even number: every wavefront starts a period
  static_assert(LI % 2 == 0, "");
  const bf16 *p0, *p1;
  int64_t ld0, ld1;
  unsigned v0[2], v1[2], dst;
  __device__ __forceinline__ TileFeed(const bf16* first, const bf16* second, int64_t ld0_, int64_t ld1_, int lane, int w, const char* lds)
      : p0(first + w * LI * 8 * ld0_), p1(second + w * LI * 8 * ld1_), ld0(ld0_), ld1(ld1_),
        dst((unsigned)(uintptr_t)(__attribute__((address_space(3))) const char*)(lds) + w * LI * 1024) {
#pragma unroll
    for (int i = 0; i < 2; i++) { v0[i] = tile_voff(lane, i, ld0); v1[i] = tile_voff(lane, i, ld1); }
  }
  __device__ __forceinline__ void issue(int tile, int stage) const {   // stage counts pairs of tiles
    const bf16 *a = p0 + (int64_t)tile * 64 * ld0, *c = p1 + (int64_t)tile * 64 * ld1;
    const unsigned to = dst + stage * (2 * T64);
#pragma unroll
    for (int i = 0; i < LI; i++) global_to_lds_16(a + (i >> 1) * 16 * ld0, v0[i & 1], to + i * 1024);
#pragma unroll
    for (int i = 0; i < LI; i++) global_to_lds_16(c + (i >> 1) * 16 * ld1, v1[i & 1], to + T64 + i * 1024);
  }
};

// 4 x 4 rows of a transposed accumulator (32 head dimensions) as bf16
__device__ __forceinline__ void store_quads(bf16* dst, const f32x4 (&acc)[4], float mul, int hf) {
#pragma unroll
  for (int g = 0; g < 4; g++) {
    bf16x4 r;
#pragma unroll
    for (int e = 0; e < 4; e++) r[e] = (bf16)(acc[g][e] * mul);
    *reinterpret_cast<bf16x4*>(dst + 8 * g + 4 * hf) = r;
  }
}
constexpr int SHARE = 4 * 16 * 256;   // bytes of one wavefront's four accumulators in LDS
__device__ __forceinline__ void leave_share(float* to, int lane, const f32x16* acc) {
#pragma unroll
  for (int p = 0; p < 4; p++)
#pragma unroll
    for (int g = 0; g < 4; g++)
      *reinterpret_cast<f32x4*>(to + p * 1024 + g * 256 + lane * 4) = (f32x4){acc[p][4 * g], acc[p][4 * g + 1], acc[p][4 * g + 2], acc[p][4 * g + 3]};
}
// Adds the accumulators of the KS wavefronts that share an output, in their order: every one leaves its four in LDS and hands 4 / KS of
// the sums to put(part, rows).
template <int W, int KS, typename Put>
__device__ __forceinline__ void add_shares(char* smem, int wave, int lane, const f32x16* acc, Put put) {
  static_assert(W * SHARE <= 4 * T64, "the shares must fit the operand stages");
  __syncthreads();
  leave_share(reinterpret_cast<float*>(smem + wave * SHARE), lane, acc);
  __syncthreads();
  const float* first = reinterpret_cast<const float*>(smem + (wave % W) * SHARE);
#pragma unroll
  for (int p = 0; p < 4 / KS; p++) {
    const int part = wave / W * (4 / KS) + p;
    f32x4 sum[4];
#pragma unroll
    for (int j = 0; j < KS; j++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(first + j * (W * SHARE / 4) + part * 1024 + g * 256 + lane * 4);
        sum[g] = j ? sum[g] + v : v;
      }
    put(part, sum);
  }
}

// ------------------------------------------------------------------------------------------
// forward: QW KS wavefronts; wavefront (qg, ks) owns 64 queries, two column blocks A and B of 32, and every KS-th tile of 64 keys
// ------------------------------------------------------------------------------------------
template <int QW, int KS>
__global__ __launch_bounds__(64 * QW * KS, 2) void attn_fwd_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ o,
                                                                   float* __restrict__ lse, int S, int h, int B, float scale_log2) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];   // 2 stages x KS x (K, V)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), hf = lane >> 5;
  const int qg = wave % QW, ks = wave / QW;
  const int nblk = S / (64 * QW);
  const BlockId id = block_id(nblk, h, B);
  const int q0 = (nblk - 1 - id.blk) * (64 * QW), hd = id.hd, b = id.b;
  const int d = h * DH;
  const int64_t ld = 3 * (int64_t)d;
  const bf16* base = qkv + (int64_t)b * S * ld + hd * DH;
  const int qw = q0 + qg * 64;

  bf16x8 qf[2][4];
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int kk = 0; kk < 4; kk++)
      qf[x][kk] = *reinterpret_cast<const bf16x8*>(base + (int64_t)(qw + 32 * x + (lane & 31)) * ld + kk * 16 + hf * 8);

  const int n_tiles = (q0 + 64 * QW) / 64, n_iter = (n_tiles + KS - 1) / KS;
  TileFeed<QW> feed(base + d, base + 2 * d, ld, ld, lane, qg, smem + ks * (2 * T64));
  auto issue = [&](int it) {
    const int t = it * KS + ks;   // the tail of the last iteration is a tile that was loaded before, not used
    feed.issue(t < n_tiles ? t : n_tiles - 1, (it & 1) * KS);
  };
  int k_off[4], v_off[2][2];
#pragma unroll
  for (int kk = 0; kk < 4; kk++) k_off[kk] = frag_off(lane, kk);
#pragma unroll
  for (int dt = 0; dt < 2; dt++)
#pragma unroll
    for (int s = 0; s < 2; s++) v_off[dt][s] = tr_frag_off(lane, dt, s);

  f32x16 oacc[2][2] = {{zero16(), zero16()}, {zero16(), zero16()}};
  float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.0f, 0.0f};
  float neg[2] = {0.0f, 0.0f};   // -m_run in log2 units, 0 while every score seen is -inf (their probabilities are then 0, not NaN)

  // One tile of 64 keys.  DIAG: the tile that starts at this wavefront's first query: block A sees its first half up to the
  // diagonal, block B all of the first half and the second up to the diagonal.
  auto tile = [&](const char* Ks, auto diag) {
    constexpr bool DIAG = decltype(diag)::value;
    const char* Vs = Ks + T64;
    bf16x8 kfr[2][4];
#pragma unroll
    for (int kt = 0; kt < 2; kt++)
#pragma unroll
      for (int kk = 0; kk < 4; kk++) kfr[kt][kk] = lds_direct(Ks + kt * 4096 + k_off[kk]);
    f32x16 s[2][2];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int x = 0; x < 2; x++) {
#pragma unroll
      for (int kt = 0; kt < 2; kt++) s[x][kt] = zero16();
#pragma unroll
      for (int kk = 0; kk < 4; kk++)
#pragma unroll
        for (int kt = 0; kt < 2; kt++)
          if (!DIAG || kt <= x) s[x][kt] = MFMA(kfr[kt][kk], qf[x][kk], s[x][kt]);
    }
    bf16x8 vfr[2][2][2];
    auto load_v = [&](int kt) {
#pragma unroll
      for (int kk = 0; kk < 2; kk++)
#pragma unroll
        for (int dt = 0; dt < 2; dt++) {
          const char* p = Vs + (kt * 32 + kk * 16) * 128;
          vfr[kt][kk][dt] = lds_tr2(p + v_off[dt][0], p + v_off[dt][1]);
        }
    };
    __builtin_amdgcn_sched_barrier(0);
    load_v(0);
    // running maximum in raw score units; probabilities are exp2((s - m) * scale_log2) with the scale folded into one fma per
    // element
    float mx[2];
#pragma unroll
    for (int x = 0; x < 2; x++) {
      float m = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 2; kt++) {
        if (DIAG && kt > x) continue;
#pragma unroll
        for (int v = 0; v < 16; v++) {
          if (DIAG && kt == x && 8 * (v >> 2) + 4 * hf + (v & 3) > (lane & 31)) s[x][kt][v] = -INFINITY;
          m = fmaxf(m, s[x][kt][v]);
        }
      }
      mx[x] = fmaxf(m, other_half(m));
    }
    // The reference point m_run only has to keep the exponentials in range, it need not be the
    // exact running maximum: it moves (and the accumulators are rescaled) only when some row's
    // maximum has grown by more than 2^8 in probability units since it was last set.  The first
    // tile with a score above -inf always sets it (m_run = -inf).
    if (__any((mx[0] - m_run[0]) * scale_log2 > 8.0f || (mx[1] - m_run[1]) * scale_log2 > 8.0f)) {  // wave-uniform
#pragma unroll
      for (int x = 0; x < 2; x++) {
        const float m_new = fmaxf(m_run[x], mx[x]), ref = m_new == -INFINITY ? 0.0f : m_new;
        const float alpha = fast_exp2((m_run[x] - ref) * scale_log2);
        l_run[x] *= alpha;
#pragma unroll
        for (int dt = 0; dt < 2; dt++)
#pragma unroll
          for (int v = 0; v < 16; v++) oacc[x][dt][v] *= alpha;
        m_run[x] = m_new;
        neg[x] = -ref * scale_log2;
      }
    }
    // the products of one 32 x 32 block run while the probabilities of the next are formed
    auto probs = [&](int x, int kt) {
      float lsum = 0.0f;
#pragma unroll
      for (int v = 0; v < 16; v++) {
        const float p = fast_exp2(fmaf(s[x][kt][v], scale_log2, neg[x]));
        s[x][kt][v] = p;
        lsum += p;
      }
      l_run[x] += lsum;
    };
    auto values = [&](int x, int kt) {
#pragma unroll
      for (int kk = 0; kk < 2; kk++) {
        const bf16x8 pf = pack8(s[x][kt], kk);
#pragma unroll
        for (int dt = 0; dt < 2; dt++) oacc[x][dt] = MFMA(vfr[kt][kk][dt], pf, oacc[x][dt]);
      }
    };
    probs(0, 0);
    __builtin_amdgcn_sched_barrier(0);
    values(0, 0);
    probs(1, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_v(1);
    values(1, 0);
    if (!DIAG) {
      probs(0, 1);
      __builtin_amdgcn_sched_barrier(0);
      values(0, 1);
    }
    probs(1, 1);
    __builtin_amdgcn_sched_barrier(0);
    values(1, 1);
  };

  issue(0);
#pragma unroll
  for (int x = 0; x < 2; x++) settle(qf[x]);
  const int jd = qw / 64;   // the tile with this wavefront's diagonal
  auto next = [&](int it) {
    // This wavefront's loads of the iteration have landed, and after the barrier everybody's have, and nobody reads the other
    // stage any more.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (it + 1 < n_iter) issue(it + 1);
    return smem + ((it & 1) * KS + ks) * (2 * T64);
  };
  int it = 0;
  for (; it * KS + ks < jd; it++) tile(next(it), std::false_type{});
  for (; it < n_iter; it++) {
    const char* Ks = next(it);
    if (it * KS + ks == jd) tile(Ks, std::true_type{});
  }
#pragma unroll
  for (int x = 0; x < 2; x++) l_run[x] += other_half(l_run[x]);

  if constexpr (KS == 1) {
#pragma unroll
    for (int x = 0; x < 2; x++) {
      const int q = qw + 32 * x + (lane & 31);
      store_rows(o + ((int64_t)b * S + q) * d + hd * DH, oacc[x], 1.0f / l_run[x], hf);
      if (hf == 0) lse[((int64_t)b * h + hd) * S + q] = (m_run[x] * scale_log2 + log2f(l_run[x])) * LN2;
    }
  } else {
    // Results of the wavefronts that share 64 queries: every one leaves its accumulators and statistics in LDS, wavefront ks adds
    // 4 / KS of the four (query block, 32 head dimensions) parts, in order of the wavefronts.
    constexpr int PART = SHARE + 4 * 256;
    static_assert(QW * PART <= 4 * T64, "the shares must fit the operand stages");
    __syncthreads();
    float* mine = reinterpret_cast<float*>(smem + wave * PART);
    leave_share(mine, lane, &oacc[0][0]);
#pragma unroll
    for (int x = 0; x < 2; x++) {
      mine[4096 + x * 64 + lane] = m_run[x];
      mine[4096 + 128 + x * 64 + lane] = l_run[x];
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 4 / KS; p++) {
      const int part = ks * (4 / KS) + p, x = part >> 1, dt = part & 1;
      const int q = qw + 32 * x + (lane & 31);
      const float* first = reinterpret_cast<const float*>(smem + qg * PART);
      constexpr int STEP = QW * PART / 4;   // from one sharing wavefront's floats to the next one's
      float M = first[4096 + x * 64 + lane];
#pragma unroll
      for (int j = 1; j < KS; j++) M = fmaxf(M, first[j * STEP + 4096 + x * 64 + lane]);
      float l = 0.0f;
      f32x4 acc[4];
#pragma unroll
      for (int j = 0; j < KS; j++) {
        const float* src = first + j * STEP;
        const float f = fast_exp2((src[4096 + x * 64 + lane] - M) * scale_log2);   // 0 for a wavefront without a tile
        l += f * src[4096 + 128 + x * 64 + lane];
#pragma unroll
        for (int g = 0; g < 4; g++) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(src + part * 1024 + g * 256 + lane * 4) * f;
          acc[g] = j ? acc[g] + v : v;
        }
      }
      store_quads(o + ((int64_t)b * S + q) * d + hd * DH + dt * 32, acc, 1.0f / l, hf);
      if (hf == 0 && dt == 0) lse[((int64_t)b * h + hd) * S + q] = (M * scale_log2 + log2f(l)) * LN2;
    }
  }
}

// ------------------------------------------------------------------------------------------
// backward, dQ (and the row dots D = rowsum(dO * O), which it leaves for the dK/dV pass): wavefronts as in the forward kernel.
// Per 64-key tile:
//   S^T = K Q^T ; dP^T = V dO^T ; dS^T = P^T (dP^T - D) ; dQ^T += K^T dS^T
// ------------------------------------------------------------------------------------------
template <int QW, int KS>
__global__ __launch_bounds__(64 * QW * KS, 2) void attn_bwd_dq_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ o,
                                                                      const bf16* __restrict__ d_o, const float* __restrict__ lse,
                                                                      float* __restrict__ D, bf16* __restrict__ dqkv, int S, int h, int B,
                                                                      float scale) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];   // 2 stages x KS x (K, V)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), hf = lane >> 5;
  const int qg = wave % QW, ks = wave / QW;
  const int nblk = S / (64 * QW);
  const BlockId id = block_id(nblk, h, B);
  const int q0 = (nblk - 1 - id.blk) * (64 * QW), hd = id.hd, b = id.b;
  const int d = h * DH;
  const int64_t ld = 3 * (int64_t)d;
  const bf16* base = qkv + (int64_t)b * S * ld + hd * DH;
  const float scale_log2 = scale * LOG2E;

  const int qw = q0 + qg * 64;
  const int n_tiles = (q0 + 64 * QW) / 64, n_iter = (n_tiles + KS - 1) / KS;
  TileFeed<QW> feed(base + d, base + 2 * d, ld, ld, lane, qg, smem + ks * (2 * T64));
  feed.issue(ks < n_tiles ? ks : n_tiles - 1, 0);

  bf16x8 qf[2][4], gf[2][4];
  float lse2[2], Dq[2];
#pragma unroll
  for (int x = 0; x < 2; x++) {
    const int q = qw + 32 * x + (lane & 31);
    const bf16* dorow = d_o + ((int64_t)b * S + q) * d + hd * DH;
    const bf16* orow = o + ((int64_t)b * S + q) * d + hd * DH;
    // D[q] = sum_c dO[q,c] O[q,c]: each lane holds half of its query's row; kept for the dK/dV pass
    float acc = 0.0f;
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
      qf[x][kk] = *reinterpret_cast<const bf16x8*>(base + (int64_t)q * ld + kk * 16 + hf * 8);
      gf[x][kk] = *reinterpret_cast<const bf16x8*>(dorow + kk * 16 + hf * 8);
      const bf16x8 of = *reinterpret_cast<const bf16x8*>(orow + kk * 16 + hf * 8);
#pragma unroll
      for (int e = 0; e < 8; e++) acc += (float)of[e] * (float)gf[x][kk][e];
    }
    lse2[x] = lse[((int64_t)b * h + hd) * S + q] * LOG2E;
    Dq[x] = acc + other_half(acc);
    if (ks == 0 && hf == 0) D[((int64_t)b * h + hd) * S + q] = Dq[x];
  }
  int r_off[4], t_off[2][2];
#pragma unroll
  for (int kk = 0; kk < 4; kk++) r_off[kk] = frag_off(lane, kk);
#pragma unroll
  for (int dt = 0; dt < 2; dt++)
#pragma unroll
    for (int s = 0; s < 2; s++) t_off[dt][s] = tr_frag_off(lane, dt, s);

  f32x16 dq[2][2] = {{zero16(), zero16()}, {zero16(), zero16()}};
  auto tile = [&](const char* Ks, auto diag) {
    constexpr bool DIAG = decltype(diag)::value;
    const char* Vs = Ks + T64;
#pragma unroll
    for (int kt = 0; kt < 2; kt++) {
      bf16x8 kfr[4], vfr[4], ktr[2][2];
#pragma unroll
      for (int kk = 0; kk < 4; kk++) {
        kfr[kk] = lds_direct(Ks + kt * 4096 + r_off[kk]);
        vfr[kk] = lds_direct(Vs + kt * 4096 + r_off[kk]);
      }
      __builtin_amdgcn_sched_barrier(0);
      f32x16 s[2], dp[2];
      auto scores = [&](int x) {
        s[x] = zero16();
        dp[x] = zero16();
#pragma unroll
        for (int kk = 0; kk < 4; kk++) {
          s[x] = MFMA(kfr[kk], qf[x][kk], s[x]);
          dp[x] = MFMA(vfr[kk], gf[x][kk], dp[x]);
        }
      };
      auto grads = [&](int x) {
#pragma unroll
        for (int v = 0; v < 16; v++) {
          float p = fast_exp2(fmaf(s[x][v], scale_log2, -lse2[x]));
          if (DIAG && kt == x && 8 * (v >> 2) + 4 * hf + (v & 3) > (lane & 31)) p = 0.0f;
          s[x][v] = p * (dp[x][v] - Dq[x]);
        }
      };
      auto apply = [&](int x) {
#pragma unroll
        for (int kk = 0; kk < 2; kk++) {
          const bf16x8 dsf = pack8(s[x], kk);
#pragma unroll
          for (int dt = 0; dt < 2; dt++) dq[x][dt] = MFMA(ktr[kk][dt], dsf, dq[x][dt]);
        }
      };
      const bool first = !DIAG || kt == 0;   // block A sees no key of the second half of its diagonal tile
      if (first) scores(0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < 2; kk++)
#pragma unroll
        for (int dt = 0; dt < 2; dt++) {
          const char* p = Ks + (kt * 32 + kk * 16) * 128;
          ktr[kk][dt] = lds_tr2(p + t_off[dt][0], p + t_off[dt][1]);
        }
      scores(1);
      if (first) grads(0);
      __builtin_amdgcn_sched_barrier(0);
      if (first) apply(0);
      grads(1);
      __builtin_amdgcn_sched_barrier(0);
      apply(1);
    }
  };

#pragma unroll
  for (int x = 0; x < 2; x++) { settle(qf[x]); settle(gf[x]); }
  asm volatile("" ::"v"(lse2[0]), "v"(Dq[0]), "v"(lse2[1]), "v"(Dq[1]));
  const int jd = qw / 64;   // the tile with this wavefront's diagonal
  auto next = [&](int it) {   // as in the forward kernel
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const int t = (it + 1) * KS + ks;
    if (it + 1 < n_iter) feed.issue(t < n_tiles ? t : n_tiles - 1, ((it + 1) & 1) * KS);
    return smem + ((it & 1) * KS + ks) * (2 * T64);
  };
  int it = 0;
  for (; it * KS + ks < jd; it++) tile(next(it), std::false_type{});
  for (; it < n_iter; it++) {
    const char* Ks = next(it);
    if (it * KS + ks == jd) tile(Ks, std::true_type{});
  }
  if constexpr (KS == 1) {
#pragma unroll
    for (int x = 0; x < 2; x++)
      store_rows(dqkv + ((int64_t)b * S + qw + 32 * x + (lane & 31)) * ld + hd * DH, dq[x], scale, hf);
  } else {
    add_shares<QW, KS>(smem, wave, lane, &dq[0][0], [&](int part, const f32x4 (&acc)[4]) {
      bf16* dst = dqkv + ((int64_t)b * S + qw + 32 * (part >> 1) + (lane & 31)) * ld + hd * DH + (part & 1) * 32;
      store_quads(dst, acc, scale, hf);
    });
  }
}

// ------------------------------------------------------------------------------------------
// backward, dK and dV: KW KS wavefronts; wavefront (kg, ks) owns 32 keys and every KS-th tile of 64 queries.  Per 32-query half:
//   S = Q K^T ; dP = dO V^T ; P = exp(S - lse) ; dS = P (dP - D) ;
//   dV^T += dO^T P ; dK^T += Q^T dS
// A lane's accumulator holds 16 queries, so that the row statistics would be 32 more values per lane and half, 8 KB of LDS reads
// beside the 16 KB of the operands.  They enter through the matrix cores instead: one more contraction step each, whose A operand holds, per
// query, -lse / scale or -D cut into three bf16 parts of 8 significant bits (their sum is the value, to 2^-133 below 2^-110), and whose
// B operand is ones.  Each has an operand of its own with zeros in the other slots: with both in one, and zeros in B to pick between
// them, a D that is not finite made 0 x infinity = NaN of the scores, and so of the probabilities and of dV, which does not depend on D.
// ------------------------------------------------------------------------------------------
template <int KW, int KS>
__global__ __launch_bounds__(64 * KW * KS, 2) void attn_bwd_dkv_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ d_o,
                                                                       const float* __restrict__ lse, const float* __restrict__ D,
                                                                       bf16* __restrict__ dqkv, int S, int h, int B, float scale) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];   // 2 stages x KS x (Q, dO), then 2 x KS x 64 rows of statistics
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), hf = lane >> 5;
  const int kg = wave % KW, ks = wave / KW;
  const BlockId id = block_id(S / (32 * KW), h, B);  // key block 0 (all queries see it) first
  const int kb0 = id.blk * (32 * KW), hd = id.hd, b = id.b;
  const int d = h * DH;
  const int64_t ld = 3 * (int64_t)d;
  const bf16* base = qkv + (int64_t)b * S * ld + hd * DH;
  const bf16* dobase = d_o + (int64_t)b * S * d + hd * DH;
  const float* lse_b = lse + ((int64_t)b * h + hd) * S;
  const float* D_b = D + ((int64_t)b * h + hd) * S;
  const float scale_log2 = scale * LOG2E, inv_scale = 1.0f / scale;

  const int kw = kb0 + kg * 32;  // this wavefront's first key

  const int t_first = kb0 / 64, n_tiles = S / 64 - t_first, n_iter = (n_tiles + KS - 1) / KS;
  TileFeed<KW> feed(base, dobase, ld, d, lane, kg, smem + ks * (2 * T64));
  // Tile i of this block's into a stage; the statistics through registers of two wavefronts of each share, which cut one kind each.
  char* stats = smem + 4 * KS * T64 + ks * 1024;
  const float* stat_b = kg ? D_b : lse_b;
  const float stat_mul = kg ? -1.0f : -inv_scale;
  float stat = 0.0f;
  auto issue = [&](int i, int stage) {
    i = i < n_tiles ? i : n_tiles - 1;
    if (kg < 2) stat = stat_b[(t_first + i) * 64 + lane];
    feed.issue(t_first + i, stage);
  };
  auto stats_store = [&](int stage) {
    if (kg < 2) {   // three parts of 8 significant bits, an infinity has a first part only
      const float x = stat * stat_mul;
      const auto top = [](float v) { return __builtin_bit_cast(unsigned, v) & 0xffff0000u; };
      const auto real = [](unsigned v) { return __builtin_bit_cast(float, v); };
      const float mid = real(top(x)) == x ? 0.0f : x - real(top(x)), low = mid - real(top(mid));
      *reinterpret_cast<u32x2*>(stats + stage * 1024 + lane * 16 + kg * 8) = (u32x2){top(x) >> 16 | top(mid), top(low) >> 16};
    }
  };
  issue(ks, 0);

  bf16x8 kf[4], vf[4];
  {
    const bf16* row = base + (int64_t)(kw + (lane & 31)) * ld;
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
      kf[kk] = *reinterpret_cast<const bf16x8*>(row + d + kk * 16 + hf * 8);
      vf[kk] = *reinterpret_cast<const bf16x8*>(row + 2 * d + kk * 16 + hf * 8);
    }
  }
  const s16x4 ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const unsigned lower = hf ? 0u : ~0u;   // the parts are contraction slots 0..2; the upper half of the lanes holds slots 4..7
  int r_off[4], t_off[2][2];
#pragma unroll
  for (int kk = 0; kk < 4; kk++) r_off[kk] = frag_off(lane, kk);
#pragma unroll
  for (int dt = 0; dt < 2; dt++)
#pragma unroll
    for (int s = 0; s < 2; s++) t_off[dt][s] = tr_frag_off(lane, dt, s);
  f32x16 acc[2][2] = {{zero16(), zero16()}, {zero16(), zero16()}};   // dK^T, dV^T

  // MODE 0: every query sees every key.  1, 2: the tile with this wavefront's diagonal, in its first or its second half (the first
  // then precedes every key).
  auto tile = [&](const char* Qs, const char* St, auto mode) {
    constexpr int MODE = decltype(mode)::value;
    const char* Gs = Qs + T64;
    f32x16 s[2], dp[2];
    bf16x8 qT[2][2], gT[2][2];   // [16 queries][32 head dimensions]
    auto scores = [&](int qh) {
      bf16x8 qa[4], ga[4];
      const u32x4 sa = *reinterpret_cast<const u32x4*>(St + (qh * 32 + (lane & 31)) * 16);
      const s16x4 sl = __builtin_bit_cast(s16x4, (u32x2){sa[0] & lower, sa[1] & lower}), sd = __builtin_bit_cast(s16x4, (u32x2){sa[2] & lower, sa[3] & lower});
#pragma unroll
      for (int kk = 0; kk < 4; kk++) {
        qa[kk] = lds_direct(Qs + qh * 4096 + r_off[kk]);
        ga[kk] = lds_direct(Gs + qh * 4096 + r_off[kk]);
      }
      s[qh] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(sl, ones, zero16(), 0, 0, 0);
      dp[qh] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(sd, ones, zero16(), 0, 0, 0);
#pragma unroll
      for (int kk = 0; kk < 4; kk++) {
        s[qh] = MFMA(qa[kk], kf[kk], s[qh]);
        dp[qh] = MFMA(ga[kk], vf[kk], dp[qh]);
      }
    };
    auto load_t = [&](int qh) {
#pragma unroll
      for (int kk = 0; kk < 2; kk++)
#pragma unroll
        for (int dt = 0; dt < 2; dt++) {
          const char* p = Qs + (qh * 32 + kk * 16) * 128;
          qT[kk][dt] = lds_tr2(p + t_off[dt][0], p + t_off[dt][1]);
          gT[kk][dt] = lds_tr2(p + T64 + t_off[dt][0], p + T64 + t_off[dt][1]);
        }
    };
    auto grads = [&](int qh) {
#pragma unroll
      for (int v = 0; v < 16; v++) {
        float p = fast_exp2(s[qh][v] * scale_log2);
        if (MODE == qh + 1 && (lane & 31) > 8 * (v >> 2) + 4 * hf + (v & 3)) p = 0.0f;
        s[qh][v] = p;
        dp[qh][v] *= p;
      }
    };
    auto apply = [&](int qh) {
#pragma unroll
      for (int kk = 0; kk < 2; kk++) {
        const bf16x8 pf = pack8(s[qh], kk), dsf = pack8(dp[qh], kk);
#pragma unroll
        for (int dt = 0; dt < 2; dt++) {
          acc[1][dt] = MFMA(gT[kk][dt], pf, acc[1][dt]);
          acc[0][dt] = MFMA(qT[kk][dt], dsf, acc[0][dt]);
        }
      }
    };
    if (MODE != 2) {
      scores(0);
      __builtin_amdgcn_sched_barrier(0);
    }
    scores(1);
    if (MODE != 2) {
      grads(0);
      load_t(0);
      __builtin_amdgcn_sched_barrier(0);
      apply(0);
    }
    grads(1);
    __builtin_amdgcn_sched_barrier(0);
    load_t(1);
    apply(1);
  };

  settle(kf);
  settle(vf);
  const int td = kw / 64 - t_first;   // this block's tile with this wavefront's diagonal
  auto next = [&](int it) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    stats_store((it & 1) * KS);
    __syncthreads();
    if (it + 1 < n_iter) issue((it + 1) * KS + ks, ((it + 1) & 1) * KS);
    return (it & 1) * KS;
  };
  int it = 0;
  for (; it < n_iter && it * KS + ks <= td; it++) {
    const int st = next(it);
    const char* Qs = smem + (st + ks) * (2 * T64);
    if (it * KS + ks == td) {
      if (kg & 1) tile(Qs, stats + st * 1024, std::integral_constant<int, 2>{});
      else tile(Qs, stats + st * 1024, std::integral_constant<int, 1>{});
    }
  }
  for (; it < n_iter; it++) {
    const int st = next(it);
    if (it * KS + ks < n_tiles) tile(smem + (st + ks) * (2 * T64), stats + st * 1024, std::integral_constant<int, 0>{});
  }
  bf16* row = dqkv + ((int64_t)b * S + kw + (lane & 31)) * ld + hd * DH + d;
  if constexpr (KS == 1) {
    store_rows(row, acc[0], scale, hf);
    store_rows(row + d, acc[1], 1.0f, hf);
  } else {
    add_shares<KW, KS>(smem, wave, lane, &acc[0][0], [&](int part, const f32x4 (&a)[4]) {
      store_quads(row + (part >> 1) * d + (part & 1) * 32, a, part >> 1 ? 1.0f : scale, hf);
    });
  }
}

}  // namespace

// Tiles go from memory to LDS 16 bytes at a time, which asks for the alignment of the tensors that they come from (rows are then aligned too).
bool attention_mfma_aligned(const void* qkv, const void* d_o) { return ((uintptr_t)qkv | (uintptr_t)d_o) % 16 == 0; }
bool attention_mfma_supported(int S, int dh, int bf) { return bf && dh == 64 && S >= 128 && S % 128 == 0 && S <= 1024; }

// How many wavefronts share a block of 64 queries (32 keys).  On its own a wavefront takes 1.1 (forward) to 1.5 us for each tile of 64 x 64, so
// sharing pays while SIMDs are without a wavefront.  In us, forward + backward, with 1 / 2 / 4:
//   B 1, S 1024, 14 heads (224 blocks of 64): 22 + 47 / 13 + 31 / 11 + 28     B 2, S 1024, 4 heads (128): 22 + 45 / 13 + 29 / 10 + 26
//   B 8, S 512, 8 heads (512): 12.6 + 29 / 10 + 26 / 12.7 + 34                B 32, S 512, 8 heads (2048): 21 + 63 / 31 + 80 / 49 + 134
//   B 3, S 384, 5 heads (90): 10 + 23 / 7.4 + 17 / 7.4 + 19                   B 4, S 128, 4 heads (32): 5.4 + 13 / 5.0 + 11.5 / 5.9 + 15
// The lines lie below where one call alone gains, since workers run side by side: with 4 at 224 blocks and 2 at 512, rounds of two workers
// took 7706 us (B 1, S 1024, 14 heads) and 3343 (B 32, S 256, 4 heads), with 2 and 1 there 7476 and 3298.  Long rows share up to 384 blocks:
// on its own a block of 16 tiles in one wavefront is a longer chain than the blocks of 32 queries that were there before (B 6, S 1024, 4 heads:
// 66.6 us forward and backward with those, 69.3 / 49.1 with 1 / 2; rounds of 8 heads, B 3, one worker 3688, 3704 / 3480, two 2814, 2815 / 2706, and
// no longer where several contexts overlap: 2328, 2328 / 2323).  At 512 blocks they would lose there (four workers 5531, 5479 / 5706) what one
// worker alone gains (3986, 4010 / 3821); the same from 384 blocks on at S 640 (overlapped 2275, 2266 / 2311) and S 512 (2224, 2206 / 2233).
static int sharing(int B, int S, int h) {
  const int64_t blocks = (int64_t)B * h * (S / 64);
  return blocks <= 128 && S >= 512 ? 4 : blocks <= (S > 768 ? 384 : 256) ? 2 : 1;
}

template <auto Kern, typename... Args>
static int launch(int64_t blocks, int waves, int lds, hipStream_t st, const Args&... args) {
  static std::atomic<bool> attr_set{false};  // the call is idempotent: a race only repeats it
  if (lds > 65536 && !attr_set.load(std::memory_order_acquire)) {
    ALS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(Kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    attr_set.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(Kern, dim3((unsigned)blocks), dim3(64 * waves), lds, st, args...);
  ALS_CHECK_LAUNCH();
  return ALS_OK;
}

int attention_fwd_mfma(const void* qkv, void* o, float* lse, int B, int S, int h, int dh, hipStream_t st) {
  if (!attention_mfma_supported(S, dh, 1) || !attention_mfma_aligned(qkv, nullptr) || B < 1 || h < 1)
    return set_error(ALS_ERR_INVALID, "attention_fwd_mfma: unsupported shape or alignment");
  float scale_log2 = (1.0f / sqrtf((float)dh)) * LOG2E;
#define ALS_FWD(QW, KS) \
  launch<attn_fwd_kernel<QW, KS>>((int64_t)S / (64 * QW) * h * B, QW * KS, KS * 4 * T64, st, (const bf16*)qkv, (bf16*)o, lse, S, h, B, scale_log2)
  const int share = sharing(B, S, h);
  return share == 4 ? ALS_FWD(1, 4) : share == 2 ? ALS_FWD(1, 2) : ALS_FWD(2, 1);
#undef ALS_FWD
}

int attention_bwd_mfma(const void* qkv, const void* o, const void* d_o, const float* lse, float* dscratch,
                       void* dqkv, int B, int S, int h, int dh, hipStream_t st) {
  if (!attention_mfma_supported(S, dh, 1) || !attention_mfma_aligned(qkv, d_o) || B < 1 || h < 1)
    return set_error(ALS_ERR_INVALID, "attention_bwd_mfma: unsupported shape or alignment");
  float scale = 1.0f / sqrtf((float)dh);
#define ALS_DQ(QW, KS) \
  launch<attn_bwd_dq_kernel<QW, KS>>((int64_t)S / (64 * QW) * h * B, QW * KS, KS * 4 * T64, st, (const bf16*)qkv, (const bf16*)o, \
                                     (const bf16*)d_o, lse, dscratch, (bf16*)dqkv, S, h, B, scale)
#define ALS_DKV(KW, KS) \
  launch<attn_bwd_dkv_kernel<KW, KS>>((int64_t)S / (32 * KW) * h * B, KW * KS, KS * (4 * T64 + 2048), st, (const bf16*)qkv, \
                                      (const bf16*)d_o, lse, (const float*)dscratch, (bf16*)dqkv, S, h, B, scale)
  const int share = sharing(B, S, h);
  const int rc = share == 4 ? ALS_DQ(1, 4) : share == 2 ? ALS_DQ(1, 2) : ALS_DQ(2, 1);
  if (rc) return rc;
  return share == 4 ? ALS_DKV(2, 4) : share == 2 ? ALS_DKV(2, 2) : ALS_DKV(4, 1);
#undef ALS_DQ
#undef ALS_DKV
}

}  // namespace als
