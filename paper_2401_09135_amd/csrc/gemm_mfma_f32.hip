// fp32 GEMM on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: whole fp32 products and sums), any shape, any operand
// layout, any alignment, the epilogues of the worker step: the reference mode's products.
//
// One workgroup owns a BM x BN tile of C and walks K in slices of BK through two LDS buffers; the loads of the slice after next
// are in flight while a slice is multiplied.  A wavefront owns a sub-tile of 32 x 32 blocks and, where tiles are few, one of WK shares of
// every slice (the shares are added through LDS at the end, in order).  An operand is kept in LDS as it lies in
// memory: [row][BK] when the contraction is contiguous (a lane's 4 steps of a group of 8 are one 16-byte read), [BK][row] when it is strided.
//   MFMA lane layout (lane l, half hf = l / 32): A row l%32, contraction hf; B column l%32, contraction hf; accumulator
//   element v: row 8 (v/4) + 4 hf + v%4, column l%32.  Step e of a group of 8 takes contraction 4 hf + e.
//
// What bounds it: the fp32 matrix rate, 64 flops per clock and SIMD (157 TFLOP/s at 2.4 GHz), for large products; for small ones the
// latency of the slice loads and of the 64-cycle MFMAs that follow each other in one wavefront, hence the split of K
// inside the workgroup.  Against 64 x 64 tiles in vector code with one element per load
// (gemm_generic.hip): 4096 x 8192 x 512 780 us (44 TFLOP/s) to 307 (112); 1024 x 256 x 1024 163 to 10.4; 256 x 192 x 64 13 to 4.8;
// error against float64 the same or smaller (shares of K are shorter sums).
#include "common.h"
#include "gelu.h"
#include "gemm_launch.h"
#include <atomic>

namespace als {

namespace {

struct __attribute__((packed, aligned(4))) f32x4u { f32x4 v; };   // 16 bytes at any element address

template <int BM, int BN, int BK, int WM, int WN, int WK, int AL, int BL, bool NAT>
struct F32Tile {
  static constexpr int NT = 64 * WM * WN * WK;
  static constexpr int MB = NAT ? 16 : 32;   // rows and columns of a block of the matrix instruction
  static constexpr int TM = BM / WM / MB, TN = BN / WN / MB;
  static constexpr int A_PITCH = AL == 0 ? BK + 4 : BM + 8, B_PITCH = BL == 1 ? BK + 4 : BN + 8;   // floats
  static constexpr int A_SIZE = A_PITCH * (AL == 0 ? BM : BK), B_SIZE = B_PITCH * (BL == 1 ? BN : BK);
  static constexpr int STAGE = A_SIZE + B_SIZE;
  static constexpr int RED = WK > 1 ? WK * BM * BN : 0;   // partial tiles of the K shares
  static constexpr int LDS_BYTES = 4 * (2 * STAGE > RED ? 2 * STAGE : RED);
  static constexpr int NA = BM * BK / 4 / NT, NB = BN * BK / 4 / NT;   // 16-byte chunks per thread
  static_assert(NA * 4 * NT == BM * BK && NB * 4 * NT == BN * BK && BK % (8 * WK) == 0, "whole chunks and groups");
  static_assert(!NAT || WK == 1, "the natural order has no shares");
};

// One operand's tile: chunk c covers tile row c / (LEN/4), 4 elements from 4 (c % (LEN/4)); LEN is the contiguous direction.
// lim_row, lim_col: how many rows and contiguous elements exist from the tile's origin on.
template <int LEN, int N, int NT>
__device__ __forceinline__ void load_chunks(f32x4 (&r)[N], const float* origin, int64_t ld, int lim_row, int lim_col, bool whole) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int i = 0; i < N; i++) {
    const int c = tid + i * NT, row = c / (LEN / 4), col = c % (LEN / 4) * 4;
    const float* p = origin + row * ld + col;
    if (whole) {
      r[i] = reinterpret_cast<const f32x4u*>(p)->v;
    } else {
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 4; e++)
        if (row < lim_row && col + e < lim_col) x[e] = p[e];
      r[i] = x;
    }
  }
}
template <int LEN, int PITCH, int N, int NT>
__device__ __forceinline__ void store_chunks(const f32x4 (&r)[N], float* lds) {
#pragma unroll
  for (int i = 0; i < N; i++) {
    const int c = threadIdx.x + i * NT;
    *reinterpret_cast<f32x4*>(lds + c / (LEN / 4) * PITCH + c % (LEN / 4) * 4) = r[i];
  }
}

__device__ __forceinline__ void f32_epilogue(const GemmDesc& g, int m, int n, float x) {
  if (m >= g.M || n >= g.N) return;
  const int64_t ci = (int64_t)m * g.ldc + n;
  if (g.epi == EPI_RESID) x += g.R[(int64_t)m * g.ldr + n];
  if (g.epi == EPI_DGELU) x *= reinterpret_cast<const float*>(g.U)[ci];
  if (g.epi == EPI_GELU) {
    reinterpret_cast<float*>(g.C2)[ci] = gelu_tanh_f(x);
    x = gelu_tanh_grad_f(x);
  }
  reinterpret_cast<float*>(g.C)[ci] = x;
}

// The tile whose first element is (m0, n0).  NAT: blocks of 16 x 16 (v_mfma_f32_16x16x4_f32: lane l holds row or column l%16 of
// contraction l/16 of a step, accumulator element v is row 4 (l/16) + v), which take the contraction in its natural order, four per step.
template <int BM, int BN, int BK, int WM, int WN, int WK, int AL, int BL, bool NAT>
__device__ __forceinline__ void f32_tile(const GemmDesc& g, const int m0, const int n0, float* lds_f32) {
  typedef F32Tile<BM, BN, BK, WM, WN, WK, AL, BL, NAT> TL;
  constexpr int TM = TL::TM, TN = TL::TN, NG = BK / 8 / WK;   // groups of 8 of one wavefront per slice
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, hf = lane >> 5, lr = lane & 31;
  const int wk = wave / (WM * WN), wm = wave % (WM * WN) / WN, wn = wave % WN;
  const float* A = reinterpret_cast<const float*>(g.A) + (AL == 0 ? m0 * g.lda : (int64_t)m0);
  const float* B = reinterpret_cast<const float*>(g.B) + (BL == 1 ? n0 * g.ldb : (int64_t)n0);
  const int lim_m = g.M - m0, lim_n = g.N - n0;
  const bool whole_mn = lim_m >= BM && lim_n >= BN;

  f32x4 ra[2][TL::NA], rb[2][TL::NB];
  auto load = [&](int k0, f32x4 (&a)[TL::NA], f32x4 (&b)[TL::NB]) {
    const int lim_k = g.K - k0;
    const bool whole = whole_mn && lim_k >= BK;   // uniform
    if constexpr (AL == 0) load_chunks<BK, TL::NA, TL::NT>(a, A + k0, g.lda, lim_m, lim_k, whole);
    else load_chunks<BM, TL::NA, TL::NT>(a, A + (int64_t)k0 * g.lda, g.lda, lim_k, lim_m, whole);
    if constexpr (BL == 1) load_chunks<BK, TL::NB, TL::NT>(b, B + k0, g.ldb, lim_n, lim_k, whole);
    else load_chunks<BN, TL::NB, TL::NT>(b, B + (int64_t)k0 * g.ldb, g.ldb, lim_k, lim_n, whole);
  };
  auto store = [&](float* s, const f32x4 (&a)[TL::NA], const f32x4 (&b)[TL::NB]) {
    store_chunks<(AL == 0 ? BK : BM), TL::A_PITCH, TL::NA, TL::NT>(a, s);
    store_chunks<(BL == 1 ? BK : BN), TL::B_PITCH, TL::NB, TL::NT>(b, s + TL::A_SIZE);
  };

  constexpr int ACC = NAT ? 4 : 16;
  typedef float acc_t __attribute__((ext_vector_type(ACC)));
  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int v = 0; v < ACC; v++) acc[i][j][v] = 0.0f;
  auto compute = [&](const float* s) {
    if constexpr (NAT) {
      const int r = lane & 15, q = lane >> 4;
      const float* As = s + (AL == 0 ? (wm * TM * 16 + r) * TL::A_PITCH + q : q * TL::A_PITCH + wm * TM * 16 + r);
      const float* Bs = s + TL::A_SIZE + (BL == 1 ? (wn * TN * 16 + r) * TL::B_PITCH + q : q * TL::B_PITCH + wn * TN * 16 + r);
#pragma unroll
      for (int k = 0; k < BK; k += 4) {
        float a[TM], b[TN];
#pragma unroll
        for (int i = 0; i < TM; i++) a[i] = AL == 0 ? As[i * 16 * TL::A_PITCH + k] : As[k * TL::A_PITCH + i * 16];
#pragma unroll
        for (int j = 0; j < TN; j++) b[j] = BL == 1 ? Bs[j * 16 * TL::B_PITCH + k] : Bs[k * TL::B_PITCH + j * 16];
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
      }
    } else {
      const float* As = s + (AL == 0 ? (wm * TM * 32 + lr) * TL::A_PITCH + 4 * hf : 4 * hf * TL::A_PITCH + wm * TM * 32 + lr);
      const float* Bs = s + TL::A_SIZE + (BL == 1 ? (wn * TN * 32 + lr) * TL::B_PITCH + 4 * hf : 4 * hf * TL::B_PITCH + wn * TN * 32 + lr);
#pragma unroll
      for (int q = 0; q < NG; q++) {
        const int k = (wk * NG + q) * 8;
        f32x4 a[TM], b[TN];
#pragma unroll
        for (int i = 0; i < TM; i++) {
          if constexpr (AL == 0) a[i] = *reinterpret_cast<const f32x4*>(As + i * 32 * TL::A_PITCH + k);
          else
#pragma unroll
            for (int e = 0; e < 4; e++) a[i][e] = As[(k + e) * TL::A_PITCH + i * 32];
        }
#pragma unroll
        for (int j = 0; j < TN; j++) {
          if constexpr (BL == 1) b[j] = *reinterpret_cast<const f32x4*>(Bs + j * 32 * TL::B_PITCH + k);
          else
#pragma unroll
            for (int e = 0; e < 4; e++) b[j][e] = Bs[(k + e) * TL::B_PITCH + j * 32];
        }
#pragma unroll
        for (int e = 0; e < 4; e++)
#pragma unroll
          for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
      }
    }
  };

  const int nk = (g.K + BK - 1) / BK;
  float* s0 = lds_f32;
  float* s1 = lds_f32 + TL::STAGE;
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

  if constexpr (NAT) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int v = 0; v < 4; v++)
          f32_epilogue(g, m0 + (wm * TM + i) * 16 + 4 * (lane >> 4) + v, n0 + (wn * TN + j) * 16 + (lane & 15), acc[i][j][v]);
  } else if constexpr (WK == 1) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int v = 0; v < 16; v++)
          f32_epilogue(g, m0 + (wm * TM + i) * 32 + 8 * (v >> 2) + 4 * hf + (v & 3), n0 + (wn * TN + j) * 32 + lr, acc[i][j][v]);
  } else {
    float* part = lds_f32 + wk * BM * BN + wm * TM * 32 * BN + wn * TN * 32 + lr;
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) part[(i * 32 + 8 * (v >> 2) + 4 * hf + (v & 3)) * BN + j * 32] = acc[i][j][v];
    __syncthreads();
    for (int e = threadIdx.x; e < BM * BN; e += TL::NT) {
      float x = lds_f32[e];
#pragma unroll
      for (int s = 1; s < WK; s++) x += lds_f32[s * BM * BN + e];
      f32_epilogue(g, m0 + e / BN, n0 + e % BN, x);
    }
  }
}

// every XCD gets a contiguous run of tiles (columns fastest): neighbours share operand panels in its L2
__device__ __forceinline__ int xcd_tile() {
  const int ntiles = gridDim.x, per = ntiles / 8, id = blockIdx.x;
  return id < per * 8 ? (id % 8) * per + id / 8 : id;
}

template <int BM, int BN, int BK, int WM, int WN, int WK, int AL, int BL, bool NAT>
__global__ __launch_bounds__(64 * WM * WN * WK, 2) void gemm_f32_kernel(GemmDesc g, int tiles_n) {
  extern __shared__ __attribute__((aligned(16))) float lds_f32[];
  const int tile = xcd_tile();
  f32_tile<BM, BN, BK, WM, WN, WK, AL, BL, NAT>(g, tile / tiles_n * BM, tile % tiles_n * BN, lds_f32);
}

// X^T dY of a list of products
template <int BM, int BN, int BK, int WM, int WN, int WK, bool NAT>
__global__ __launch_bounds__(64 * WM * WN * WK, 2) void gemm_f32_dw_list_kernel(DwList list) {
  extern __shared__ __attribute__((aligned(16))) float lds_f32[];
  const int id = xcd_tile();
  const DwList::Product& p = list.p[list.find(id)];
  GemmDesc g;
  g.A = p.A; g.B = p.B; g.C = p.C; g.M = p.M; g.N = p.N; g.K = list.K;
  g.lda = p.M; g.ldb = p.N; g.ldc = p.N; g.epi = EPI_STORE; g.c_bf16 = 0;
  g.R = nullptr; g.C2 = nullptr; g.U = nullptr; g.ldr = 0;
  const int tile = id - p.tile0;
  f32_tile<BM, BN, BK, WM, WN, WK, 1, 0, NAT>(g, tile / p.tiles_n * BM, tile % p.tiles_n * BN, lds_f32);
}

template <int BM, int BN, int BK, int WM, int WN, int WK, int AL, int BL, bool NAT = false>
int launch_f32(const GemmDesc& g, hipStream_t st) {
  typedef F32Tile<BM, BN, BK, WM, WN, WK, AL, BL, NAT> TL;
  auto kern = gemm_f32_kernel<BM, BN, BK, WM, WN, WK, AL, BL, NAT>;
  if (TL::LDS_BYTES > 65536) {
    static std::atomic<bool> attr_set{false};  // the call is idempotent: a race only repeats it
    if (!attr_set.load(std::memory_order_acquire)) {
      ALS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS_BYTES));
      attr_set.store(true, std::memory_order_release);
    }
  }
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  return launch_gemm(kern, tiles_m * tiles_n, TL::NT, TL::LDS_BYTES, st, prof_id(PROF_F32, NAT ? 4 : BM == 32 ? (WK == 8 ? 2 : 3) : BM == 64 ? 1 : 0, AL, BL), product_flops(g.M, g.N, g.K),
                     g, tiles_n);
}

template <int BM, int BN, int BK, int WM, int WN, int WK, bool NAT = false>
int launch_dw_list(const DwProblem* probs, int n, int K, hipStream_t st) {
  typedef F32Tile<BM, BN, BK, WM, WN, WK, 1, 0, NAT> TL;
  auto kern = gemm_f32_dw_list_kernel<BM, BN, BK, WM, WN, WK, NAT>;
  static std::atomic<bool> attr_set{false};  // the call is idempotent: a race only repeats it
  if (!attr_set.load(std::memory_order_acquire)) {
    ALS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS_BYTES));
    attr_set.store(true, std::memory_order_release);
  }
  DwList list;
  for (int i = 0, ntiles; i < n; ) {
    i += list.fill(probs + i, n - i, K, BM, BN, &ntiles);
    int rc = launch_gemm(kern, ntiles, TL::NT, TL::LDS_BYTES, st, prof_id(PROF_F32_LIST, NAT ? 4 : BM == 32 ? (WK == 8 ? 2 : 3) : BM == 64 ? 1 : 0), list_flops(list), list);
    if (rc) return rc;
  }
  return ALS_OK;
}

// Which tile a product (or a list of them, its tiles counted together) takes: 0 for 128 x 128, 1 for 64 x 64 with 2 K shares, 2 for
// 32 x 32 with 8, 3 with 4, 4 for 32 x 32 in blocks of 16 x 16 with k in its natural order.
// The largest tile that still gives (almost) every CU a workgroup: a larger tile moves fewer operand bytes per flop, an idle CU
// costs its whole rate.  In us, 128 x 128 / 64 x 64 / 32 x 32 with 8 K shares / with 4 / in natural order:
//   4096 x 8192 x 512 (2048, 8192 tiles): 307 / 347 / 478 / 420 / -     2048 x 1536 x 512 (192, 768): 48 / 39 / 49 / 44 / -
//   1024 x 1024 x 256 (64, 256): 26 / 9.9 / 12 / 10 / -                 256 x 2000 x 1024 (32, 128): 127 / 43 / 26 / 31 / -
//   512 x 512 x 511 (16, 64): 44 / 14 / 6.6 / 8.5 / 9.1                 1024 x 256 x 256 (16, 64): 28 / 8.6 / 5.7 / 5.4 / 5.6
//   1024 x 256 x 511 (16, 64): - / - / - / 7.8 / 8.4                    256 x 64 x 256 (1, 4): - / - / - / 5.2 / 5.2
// Up to K = 256 the natural order costs nothing (1 to 2 % over 260 sizes): the chain of a 16 x 16 block, K/4 instructions of 32
// cycles, is as long as that of a 32 x 32 one with 4 shares of K, which are added at the end.  Its results have the bits of a plain
// loop over k, which keeps short runs of the smallest models within 1e-5 of an fp32 program that adds so (elements with a gradient
// near zero carry rounding into AdamW's direction).  From there on the shares win, 7 % up to 512, and their shorter sums are nearer to
// float64; a short run is then as near to float64 as that program, but no longer to its bits.
template <typename Tiles>
int choose_tile(Tiles tiles, int K) {
  if (tiles(128, 128) >= 256) return 0;
  if (tiles(64, 64) >= 192) return 1;
  return K >= 512 ? 2 : K > 256 ? 3 : 4;
}
int choose_tile(const GemmDesc& g) {
  return choose_tile([&](int bm, int bn) { return gemm_tiles(g.M, g.N, bm, bn); }, g.K);
}

template <int AL, int BL>
int pick(const GemmDesc& g, hipStream_t st) {
  switch (choose_tile(g)) {
    case 0: return launch_f32<128, 128, 32, 2, 2, 1, AL, BL>(g, st);
    case 1: return launch_f32<64, 64, 64, 2, 2, 2, AL, BL>(g, st);
    case 2: return launch_f32<32, 32, 128, 1, 1, 8, AL, BL>(g, st);
    case 3: return launch_f32<32, 32, 64, 1, 1, 4, AL, BL>(g, st);
    default: return launch_f32<32, 32, 64, 2, 2, 1, AL, BL, true>(g, st);
  }
}

}  // namespace

bool gemm_mfma_f32_supported(const GemmDesc& g) {
  if (g.in_bf16 || g.c_bf16 || (g.a_layout | g.b_layout) & ~1) return false;
  // fewer than 2^32 threads in the one grid dimension: beyond 256 tiles of 128 x 128, blocks of 256 threads on those; below, fewer blocks than that
  return gemm_tiles(g.M, g.N, 128, 128) < (1 << 24);
}

int gemm_mfma_f32(const GemmDesc& g, hipStream_t st) {
  if (g.a_layout == 0) return g.b_layout == 0 ? pick<0, 0>(g, st) : pick<0, 1>(g, st);
  return g.b_layout == 0 ? pick<1, 0>(g, st) : pick<1, 1>(g, st);
}

const char* gemm_mfma_f32_route(const GemmDesc& g) {
  static const char* const name[] = {"f32 128x128", "f32 64x64/2", "f32 32x32/8", "f32 32x32/4", "f32 32x32 natural"};
  return name[choose_tile(g)];
}

// the tile by the same rule as for one product, on the tiles of all
int gemm_mfma_f32_dw_list(const DwProblem* probs, int n, int K, hipStream_t st) {
  if (n <= 0) return ALS_OK;
  switch (choose_tile([&](int bm, int bn) { return dw_list_tiles(probs, n, bm, bn); }, K)) {
    case 0: return launch_dw_list<128, 128, 32, 2, 2, 1>(probs, n, K, st);
    case 1: return launch_dw_list<64, 64, 64, 2, 2, 2>(probs, n, K, st);
    case 2: return launch_dw_list<32, 32, 128, 1, 1, 8>(probs, n, K, st);
    case 3: return launch_dw_list<32, 32, 64, 1, 1, 4>(probs, n, K, st);
    default: return launch_dw_list<32, 32, 64, 2, 2, 1, true>(probs, n, K, st);
  }
}

}  // namespace als
