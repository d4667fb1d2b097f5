// bf16 GEMM on the matrix cores (v_mfma_f32_32x32x16_bf16, fp32 sums) for any shape and alignment, and for small aligned products: what
// the kernels with fixed tiles of gemm_mfma.hip do not take, or would run on a few CUs.  Layouts and epilogues of the
// worker step: A [m][k] with B [k][n] or [n][k], and X^T dY.
//
// One workgroup owns a BM x BN tile of C and walks K in slices of BK through two LDS buffers; the loads of the slice after
// next are in flight while a slice is multiplied.  A wavefront owns a sub-tile of 32 x 32 blocks and one of WK shares of
// every slice; the shares are added through LDS, in order, on the way out.  An operand is kept in LDS as it lies in memory:
// [row][BK] when the contraction is contiguous, [BK][row], read with the LDS transpose load, when it is strided.  Chunks of
// 8 elements that lie inside the matrix are one 16-byte load at any element address; what lies outside is zero.
//
// What bounds it: for small products the latency of one slice (loads, LDS, barrier), so slices are long (128, 256) and
// few; for ragged ones of ordinary size the same kernels' operand traffic.  Against 64 x 64 tiles in
// vector code (gemm_generic.hip): 600 x 960 x 320 56 us to 6.2, 600 x 320 x 5003 1249 to 25, 3000 x 4000 x 700 389 to 57; error against
// float64 the same or smaller (shares of K are shorter sums).
#include "common.h"
#include "gelu.h"
#include "gemm_launch.h"

#include <atomic>

namespace als {

namespace {

struct __attribute__((packed, aligned(4))) f32x4u { f32x4 v; };
struct __attribute__((packed, aligned(2))) bf16x4u { bf16x4 v; };
struct __attribute__((packed, aligned(2))) bf16x8u { u32x4 v; };

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

__device__ __forceinline__ bf16x8 read_tr(const char* p, int pitch) {   // contraction rows 0..3 and 4..7 from p on
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * pitch));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int BM, int BN, int BK, int WM, int WN, int WK, int AL, int BL>
struct AnyTile {
  static constexpr int NT = 64 * WM * WN * WK;
  static constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  static constexpr int A_PITCH = AL == 0 ? BK * 2 + 16 : BM * 2 + 64, B_PITCH = BL == 1 ? BK * 2 + 16 : BN * 2 + 64;   // bytes
  static constexpr int A_BYTES = A_PITCH * (AL == 0 ? BM : BK), B_BYTES = B_PITCH * (BL == 1 ? BN : BK);
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int O_PITCH = BN + 4;                        // floats: 4-float accesses of neighbouring rows do not collide
  static constexpr int OUT = WK * BM * O_PITCH * 4;             // the partial tiles of the K shares
  static constexpr int LDS_BYTES = 2 * STAGE > OUT ? 2 * STAGE : OUT;
  static constexpr int NA = BM * BK / 8 / NT, NB = BN * BK / 8 / NT;   // 16-byte chunks per thread
  static_assert(NA * 8 * NT == BM * BK && NB * 8 * NT == BN * BK && BK % (16 * WK) == 0, "whole chunks and steps");
};

// One operand's tile: chunk c covers tile row c / (LEN/8), 8 elements from 8 (c % (LEN/8)); LEN is the contiguous direction.
// lim_row, lim_col: how many rows and contiguous elements exist from the tile's origin on.
template <int LEN, int N, int NT>
__device__ __forceinline__ void load_chunks(u32x4 (&r)[N], const bf16* origin, int64_t ld, int lim_row, int lim_col, bool whole) {
#pragma unroll
  for (int i = 0; i < N; i++) {
    const int c = threadIdx.x + i * NT, row = c / (LEN / 8), col = c % (LEN / 8) * 8;
    const bf16* p = origin + row * ld + col;
    if (whole || (row < lim_row && col + 8 <= lim_col)) {
      r[i] = reinterpret_cast<const bf16x8u*>(p)->v;
    } else {
      u32x4 x = {0u, 0u, 0u, 0u};
      if (row < lim_row) {
        const unsigned short* s = reinterpret_cast<const unsigned short*>(p);
#pragma unroll
        for (int e = 0; e < 8; e++)
          if (col + e < lim_col) x[e / 2] |= (unsigned)s[e] << (16 * (e & 1));
      }
      r[i] = x;
    }
  }
}
template <int LEN, int PITCH, int N, int NT>
__device__ __forceinline__ void store_chunks(const u32x4 (&r)[N], char* lds) {
#pragma unroll
  for (int i = 0; i < N; i++) {
    const int c = threadIdx.x + i * NT;
    *reinterpret_cast<u32x4*>(lds + c / (LEN / 8) * PITCH + c % (LEN / 8) * 16) = r[i];
  }
}

// n consecutive results of row m from column `col` on (n = 4 takes the vector form)
template <int N>
__device__ __forceinline__ void any_epilogue(const GemmDesc& g, int m, int col, f32x4 x) {
  const int64_t ci = (int64_t)m * g.ldc + col;
  float aux[4] = {0.f, 0.f, 0.f, 0.f}, y[4];
  if (g.epi == EPI_RESID) {
    const float* p = g.R + (int64_t)m * g.ldr + col;
    if constexpr (N == 4) {
      const f32x4 v = reinterpret_cast<const f32x4u*>(p)->v;
#pragma unroll
      for (int e = 0; e < 4; e++) aux[e] = v[e];
    } else aux[0] = *p;
#pragma unroll
    for (int e = 0; e < N; e++) x[e] += aux[e];
  } else if (g.epi == EPI_DGELU) {
    const bf16* p = reinterpret_cast<const bf16*>(g.U) + ci;
    if constexpr (N == 4) {
      const bf16x4 v = reinterpret_cast<const bf16x4u*>(p)->v;
#pragma unroll
      for (int e = 0; e < 4; e++) aux[e] = (float)v[e];
    } else aux[0] = (float)*p;
#pragma unroll
    for (int e = 0; e < N; e++) x[e] *= aux[e];
  } else if (g.epi == EPI_GELU) {
#pragma unroll
    for (int e = 0; e < N; e++) { y[e] = gelu_tanh_f(x[e]); x[e] = gelu_tanh_grad_f(x[e]); }
  }
  if (!g.c_bf16) {
    float* p = reinterpret_cast<float*>(g.C) + ci;
    if constexpr (N == 4) reinterpret_cast<f32x4u*>(p)->v = x;
    else *p = x[0];
    return;
  }
  bf16* p = reinterpret_cast<bf16*>(g.C) + ci;
  if constexpr (N == 4) reinterpret_cast<bf16x4u*>(p)->v = (bf16x4){(bf16)x[0], (bf16)x[1], (bf16)x[2], (bf16)x[3]};
  else *p = (bf16)x[0];
  if (g.epi == EPI_GELU) {
    bf16* p2 = reinterpret_cast<bf16*>(g.C2) + ci;
    if constexpr (N == 4) reinterpret_cast<bf16x4u*>(p2)->v = (bf16x4){(bf16)y[0], (bf16)y[1], (bf16)y[2], (bf16)y[3]};
    else *p2 = (bf16)y[0];
  }
}

// the tile whose first element is (m0, n0)
template <int BM, int BN, int BK, int WM, int WN, int WK, int AL, int BL>
__device__ __forceinline__ void any_tile(const GemmDesc& g, const int m0, const int n0, char* lds_any) {
  typedef AnyTile<BM, BN, BK, WM, WN, WK, AL, BL> TL;
  constexpr int TM = TL::TM, TN = TL::TN, NS = BK / 16 / WK;   // 16-wide steps of one wavefront per slice
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, hf = lane >> 5, lr = lane & 31;
  const int wk = wave / (WM * WN), wm = wave % (WM * WN) / WN, wn = wave % WN;
  const bf16* A = reinterpret_cast<const bf16*>(g.A) + (AL == 0 ? m0 * g.lda : (int64_t)m0);
  const bf16* B = reinterpret_cast<const bf16*>(g.B) + (BL == 1 ? n0 * g.ldb : (int64_t)n0);
  const int lim_m = g.M - m0, lim_n = g.N - n0;
  const bool whole_mn = lim_m >= BM && lim_n >= BN;

  u32x4 ra[2][TL::NA], rb[2][TL::NB];
  auto load = [&](int k0, u32x4 (&a)[TL::NA], u32x4 (&b)[TL::NB]) {
    const int lim_k = g.K - k0;
    const bool whole = whole_mn && lim_k >= BK;   // uniform
    if constexpr (AL == 0) load_chunks<BK, TL::NA, TL::NT>(a, A + k0, g.lda, lim_m, lim_k, whole);
    else load_chunks<BM, TL::NA, TL::NT>(a, A + (int64_t)k0 * g.lda, g.lda, lim_k, lim_m, whole);
    if constexpr (BL == 1) load_chunks<BK, TL::NB, TL::NT>(b, B + k0, g.ldb, lim_n, lim_k, whole);
    else load_chunks<BN, TL::NB, TL::NT>(b, B + (int64_t)k0 * g.ldb, g.ldb, lim_k, lim_n, whole);
  };
  auto store = [&](char* s, const u32x4 (&a)[TL::NA], const u32x4 (&b)[TL::NB]) {
    store_chunks<(AL == 0 ? BK : BM), TL::A_PITCH, TL::NA, TL::NT>(a, s);
    store_chunks<(BL == 1 ? BK : BN), TL::B_PITCH, TL::NB, TL::NT>(b, s + TL::A_BYTES);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.0f;
  // fragment addresses: lane layouts as in gemm_mfma.hip; products transposed (B first), so that an accumulator holds
  // columns 8 q + 4 hf + 0..3 of one row of C
  const int row0 = wm * TM * 32, col0 = wn * TN * 32, k_tr = hf * 8 + ((lane & 15) >> 2), r_tr = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
  const int a_off = AL == 0 ? (row0 + lr) * TL::A_PITCH + hf * 16 : k_tr * TL::A_PITCH + (row0 + r_tr) * 2;
  const int b_off = TL::A_BYTES + (BL == 1 ? (col0 + lr) * TL::B_PITCH + hf * 16 : k_tr * TL::B_PITCH + (col0 + r_tr) * 2);
  auto compute = [&](const char* s) {
#pragma unroll
    for (int q = 0; q < NS; q++) {
      const int k = (wk * NS + q) * 16;
      bf16x8 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; i++) {
        if constexpr (AL == 0) a[i] = *reinterpret_cast<const bf16x8*>(s + a_off + i * 32 * TL::A_PITCH + k * 2);
        else a[i] = read_tr(s + a_off + k * TL::A_PITCH + i * 64, TL::A_PITCH);
      }
#pragma unroll
      for (int j = 0; j < TN; j++) {
        if constexpr (BL == 1) b[j] = *reinterpret_cast<const bf16x8*>(s + b_off + j * 32 * TL::B_PITCH + k * 2);
        else b[j] = read_tr(s + b_off + k * TL::B_PITCH + j * 64, TL::B_PITCH);
      }
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
    }
  };

  const int nk = (g.K + BK - 1) / BK;
  char* s0 = lds_any;
  char* s1 = lds_any + TL::STAGE;
  load(0, ra[0], rb[0]);
  if (nk > 1) load(BK, ra[1], rb[1]);
  store(s0, ra[0], rb[0]);
  __syncthreads();
  // slice kt is in s0 (s1), slice kt + 1 in registers, slice kt + 2 is requested
  for (int kt = 0; kt < nk; kt += 2) {
    if (kt + 2 < nk) load((kt + 2) * BK, ra[0], rb[0]);
    compute(s0);
    if (kt + 1 < nk) store(s1, ra[1], rb[1]);
    __syncthreads();
    if (kt + 1 < nk) {
      if (kt + 3 < nk) load((kt + 3) * BK, ra[1], rb[1]);
      compute(s1);
      if (kt + 2 < nk) store(s0, ra[0], rb[0]);
      __syncthreads();
    }
  }

  float* out = reinterpret_cast<float*>(lds_any);
  float* mine = out + (wk * BM + row0 + lr) * TL::O_PITCH + col0 + 4 * hf;
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int q = 0; q < 4; q++)
        *reinterpret_cast<f32x4*>(mine + i * 32 * TL::O_PITCH + j * 32 + 8 * q) =
            (f32x4){acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
  __syncthreads();
  for (int e = threadIdx.x; e < BM * BN / 4; e += TL::NT) {
    const int r = e / (BN / 4), c = e % (BN / 4) * 4;
    if (r >= lim_m || c >= lim_n) continue;
    f32x4 x = *reinterpret_cast<const f32x4*>(out + r * TL::O_PITCH + c);
#pragma unroll
    for (int s = 1; s < WK; s++) x += *reinterpret_cast<const f32x4*>(out + (s * BM + r) * TL::O_PITCH + c);
    if (c + 4 <= lim_n) any_epilogue<4>(g, m0 + r, n0 + c, x);
    else
#pragma unroll
      for (int u = 0; u < 3; u++)
        if (c + u < lim_n) any_epilogue<1>(g, m0 + r, n0 + c + u, (f32x4){x[u], 0.f, 0.f, 0.f});
  }
}

// every XCD gets a contiguous run of tiles (columns fastest): neighbours share operand panels in its L2
__device__ __forceinline__ int xcd_tile() {
  const int ntiles = gridDim.x, per = ntiles / 8, id = blockIdx.x;
  return id < per * 8 ? (id % 8) * per + id / 8 : id;
}

template <int BM, int BN, int BK, int WM, int WN, int WK, int AL, int BL>
__global__ __launch_bounds__(64 * WM * WN * WK, 2) void gemm_any_kernel(GemmDesc g, int tiles_n) {
  extern __shared__ __attribute__((aligned(16))) char lds_any[];
  const int tile = xcd_tile();
  any_tile<BM, BN, BK, WM, WN, WK, AL, BL>(g, tile / tiles_n * BM, tile % tiles_n * BN, lds_any);
}

// X^T dY of a list of products
template <int BM, int BN, int BK, int WM, int WN, int WK>
__global__ __launch_bounds__(64 * WM * WN * WK, 2) void gemm_any_dw_list_kernel(DwList list) {
  extern __shared__ __attribute__((aligned(16))) char lds_any[];
  const int id = xcd_tile();
  const DwList::Product& p = list.p[list.find(id)];
  GemmDesc g;
  g.A = p.A; g.B = p.B; g.C = p.C; g.M = p.M; g.N = p.N; g.K = list.K;
  g.lda = p.M; g.ldb = p.N; g.ldc = p.N; g.epi = EPI_STORE; g.c_bf16 = 0;
  g.R = nullptr; g.C2 = nullptr; g.U = nullptr; g.ldr = 0;
  const int tile = id - p.tile0;
  any_tile<BM, BN, BK, WM, WN, WK, 1, 0>(g, tile / p.tiles_n * BM, tile % p.tiles_n * BN, lds_any);
}

template <int BM, int BN, int BK, int WM, int WN, int WK, int AL, int BL>
int launch_any(const GemmDesc& g, hipStream_t st) {
  typedef AnyTile<BM, BN, BK, WM, WN, WK, AL, BL> TL;
  auto kern = gemm_any_kernel<BM, BN, BK, WM, WN, WK, AL, BL>;
  static std::atomic<bool> attr_set{false};  // the call is idempotent: a race only repeats it
  if (!attr_set.load(std::memory_order_acquire)) {
    ALS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS_BYTES));
    attr_set.store(true, std::memory_order_release);
  }
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  return launch_gemm(kern, tiles_m * tiles_n, TL::NT, TL::LDS_BYTES, st, prof_id(PROF_ANY, BM == 32 ? 3 : BM == 64 ? 2 : BN == 64 ? 1 : 0, AL, BL), product_flops(g.M, g.N, g.K),
                     g, tiles_n);
}

template <int BM, int BN, int BK, int WM, int WN, int WK>
int launch_dw_list(const DwProblem* probs, int n, int K, hipStream_t st) {
  typedef AnyTile<BM, BN, BK, WM, WN, WK, 1, 0> TL;
  auto kern = gemm_any_dw_list_kernel<BM, BN, BK, WM, WN, WK>;
  static std::atomic<bool> attr_set{false};  // the call is idempotent: a race only repeats it
  if (!attr_set.load(std::memory_order_acquire)) {
    ALS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS_BYTES));
    attr_set.store(true, std::memory_order_release);
  }
  DwList list;
  for (int i = 0, ntiles; i < n; ) {
    i += list.fill(probs + i, n - i, K, BM, BN, &ntiles);
    int rc = launch_gemm(kern, ntiles, TL::NT, TL::LDS_BYTES, st, prof_id(PROF_ANY_LIST, BM == 32 ? 3 : BM == 64 ? 2 : BN == 64 ? 1 : 0), list_flops(list), list);
    if (rc) return rc;
  }
  return ALS_OK;
}

// Which tile a product (or a list of them, its tiles counted together) takes: 0 for 128 x 128, 1 for 128 x 64 with 2 K shares,
// 2 for 64 x 64 with 2, 3 for 32 x 32 with 8.  In us, in this order (tiles of the first two; of the last two):
//   3000 x 4000 x 700 (768, 1512): 57 / 74 / 99 / 237       1000 x 2001 x 4003, X^T Y (128, 256): 259 / 74 / 132 / 192
//   320 x 5003 x 600, X^T Y (120, 237): 38 / 18 / 23 / 36   600 x 960 x 320 (40, 75; 150, 570): 15 / 8.5 / 6.2 / 11
//   1024 x 896 x 3584 (56, 112; 224, 896): 53 / 32 / 25 / 29    2048 x 256 x 1024 (32, 64; 128, 512): 19 / 11 / 7.9 / 7.1
//   600 x 320 x 5003 (15, 25; 50, 190): 123 / 61 / 45 / 25      512 x 256 x 256 (8, 16; 32, 128): 9.8 / 6.5 / 5.9 / 6.1
template <typename Tiles>
int choose_tile(Tiles tiles, int K) {
  if (tiles(128, 128) >= 256) return 0;
  if (tiles(128, 64) >= 192) return 1;
  return tiles(32, 32) > (K >= 1024 ? 512 : 256) ? 2 : 3;
}
int choose_tile(const GemmDesc& g) {
  return choose_tile([&](int bm, int bn) { return gemm_tiles(g.M, g.N, bm, bn); }, g.K);
}

template <int AL, int BL>
int pick(const GemmDesc& g, hipStream_t st) {
  switch (choose_tile(g)) {
    case 0: return launch_any<128, 128, 64, 2, 2, 1, AL, BL>(g, st);
    case 1: return launch_any<128, 64, 128, 2, 2, 2, AL, BL>(g, st);
    case 2: return launch_any<64, 64, 128, 2, 2, 2, AL, BL>(g, st);
    default: return launch_any<32, 32, 256, 1, 1, 8, AL, BL>(g, st);
  }
}

}  // namespace

bool gemm_mfma_any_supported(const GemmDesc& g) {
  if (!g.in_bf16 || (g.a_layout == 1 && g.b_layout == 1) || (g.a_layout | g.b_layout) & ~1) return false;
  if (g.epi == EPI_GELU && !g.c_bf16) return false;   // writes both outputs in bf16 only
  // fewer than 2^32 threads in the one grid dimension: beyond 256 tiles of 128 x 128, blocks of 256 threads on those; below, fewer blocks than that
  return gemm_tiles(g.M, g.N, 128, 128) < (1 << 24);
}

int gemm_mfma_any(const GemmDesc& g, hipStream_t st) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return set_error(ALS_ERR_INVALID, "gemm: empty shape");
  if (g.epi == EPI_RESID && g.c_bf16) return set_error(ALS_ERR_INVALID, "gemm: residual output must be fp32");
  if (g.a_layout == 1) return pick<1, 0>(g, st);
  return g.b_layout == 0 ? pick<0, 0>(g, st) : pick<0, 1>(g, st);
}

// About what a product takes here, its launch left out: rounds of one workgroup per CU, times K, times what one k of a round was measured to
// take in each tile (64 x 64 and 128 x 64: the median of 500 products of X^T Y with K from 512 to 2048, which lie within 15 %; 32 x 32:
// the slowest of them).
double gemm_mfma_any_us(const GemmDesc& g) {
  static const struct { int bm, bn; double ns; } tile[] = {{128, 128, 27.0}, {128, 64, 9.5}, {64, 64, 6.8}, {32, 32, 4.6}};
  const auto& t = tile[choose_tile(g)];
  return (double)((gemm_tiles(g.M, g.N, t.bm, t.bn) + 255) / 256) * g.K * t.ns * 1e-3;
}

const char* gemm_mfma_any_route(const GemmDesc& g) {
  static const char* const name[] = {"any 128x128", "any 128x64/2", "any 64x64/2", "any 32x32/8"};
  return name[choose_tile(g)];
}

// the tile by the same rule as for one product, on the tiles of all
int gemm_mfma_any_dw_list(const DwProblem* probs, int n, int K, hipStream_t st) {
  if (n <= 0) return ALS_OK;
  switch (choose_tile([&](int bm, int bn) { return dw_list_tiles(probs, n, bm, bn); }, K)) {
    case 0: return launch_dw_list<128, 128, 64, 2, 2, 1>(probs, n, K, st);
    case 1: return launch_dw_list<128, 64, 128, 2, 2, 2>(probs, n, K, st);
    case 2: return launch_dw_list<64, 64, 128, 2, 2, 2>(probs, n, K, st);
    default: return launch_dw_list<32, 32, 256, 1, 1, 8>(probs, n, K, st);
  }
}

}  // namespace als
