// bf16 GEMM on the matrix cores for aligned products whose 256 x 256 tiles leave much of the chip idle (A [m][k]
// with B [k][n] or [n][k]; M and N multiples of the tile, K of 64).
//
// What bounds such a product is the latency of its operands: with one workgroup per CU, a slice of 64 costs what a load from
// beyond the L2 takes (over 1 us in a chip that is busy) divided by the slices in flight.  So one
// workgroup owns a BM x BN tile and keeps NST - 1 slices (96 KB of the 160 KB of LDS) in flight as loads that go from
// global memory to LDS without registers, and waits for the oldest only (64 x 64 tiles: 64 KB, and two workgroups per CU).  Two wavefronts share every sub-tile, each with half
// of the k of a slice: twice the wavefronts for the latency of LDS and matrix instructions at the same LDS
// traffic.  Their halves are added through LDS, share 0 + share 1, and each then writes half of the rows.
//
// 1024 x 896 x 3584 (224 tiles of 64 x 64): 26 us with operands through registers, two slices ahead, to 17.4 (378 TFLOP/s);
// 3840 x 896 x 3584 (210 of 128 x 128): 69 us in 60 tiles of 256 x 256 to 32 (778).  Which product takes which: gemm_mfma().
//
// Slice kt lies in LDS buffer kt % NST.  One barrier per slice: before it every wavefront waits for its own loads of slice kt
// and for its reads of slice kt - 1; behind it the loads of slice kt + NST - 1 go into the buffer of slice kt - 1.  Chunks are
// permuted inside a tile row on the global side, as in the direct-to-LDS kernel of gemm_pingpong.h, so that the fragment reads
// of rows without padding do not collide:
//   contraction-contiguous, [rows][128 bytes]: row R keeps 16-byte chunk c at position c ^ ((R >> 1) & 7);
//   contraction-strided, [64 k][2 BN bytes]: k row r keeps its 64-byte group q at q ^ (r & 3) (BN = 128) or q ^ ((r >> 1) & 1)
//   (BN = 64): the 4 k rows of a transpose read fall into 4 different quarters of the banks.
#include "common.h"
#include "gemm_launch.h"

#include <atomic>

namespace als {

namespace {

#include "gemm_mfma_common.h"

__device__ __forceinline__ void deep_load_16(const void* base, unsigned voff, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(base) : "memory");
}
// all but the N youngest loads of this wavefront have landed, and its LDS reads are done
template <int N>
__device__ __forceinline__ void deep_wait() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}
template <int LPW, int LEFT>
__device__ __forceinline__ void deep_wait_for(int younger) {   // younger: slices in flight behind the awaited one, at most LEFT
  if constexpr (LEFT == 0) deep_wait<0>();
  else if (younger >= LEFT) deep_wait<LPW * LEFT>();
  else deep_wait_for<LPW, LEFT - 1>(younger);
}

template <int BM, int BN, int NST>
struct DeepTile {
  static constexpr int WM = BM / 64, WN = 2, WK = 2, NW = WM * WN * WK, NT = 64 * NW;
  static constexpr int TM = 2, TN = BN / WN / 32;
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
  static constexpr int LA = A_BYTES / 1024 / NW, LB = B_BYTES / 1024 / NW;   // loads of a wavefront per slice
  static constexpr int XCHG = TN * 16 * 64 * 4;                              // one wavefront's half sub-tile in fp32
  static constexpr int STG = 32 * (TN * 32 * 4 + 16);                        // its epilogue staging
  static constexpr int OUT = NW * (XCHG + STG);
  static constexpr int LDS_BYTES = NST * STAGE > OUT ? NST * STAGE : OUT;
  static_assert(NT == 4 * BM && LA * 1024 * NW == A_BYTES && LB * 1024 * NW == B_BYTES && LDS_BYTES <= 160 * 1024, "whole loads, LDS size");
  static_assert((NST - 2) * (LA + LB) < 64, "the wait counter has 6 bits");
};

template <int BM, int BN, int NST, int BL, int EPI, typename TO>
__global__ __launch_bounds__(4 * BM, 1) void gemm_deep_kernel(MfmaArgs g) {
  typedef DeepTile<BM, BN, NST> TL;
  constexpr int TM = TL::TM, TN = TL::TN, LA = TL::LA, LB = TL::LB;
  extern __shared__ __attribute__((aligned(1024))) char smem_deep[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int share = wave & 1, wn = (wave >> 1) & 1, wm = wave >> 2, hf = lane >> 5;
  // every XCD gets a contiguous run of tiles (columns fastest): neighbours share operand panels in its L2
  const int ntiles = gridDim.x, per = ntiles / 8, id = blockIdx.x;
  const int tile = id < per * 8 ? (id % 8) * per + id / 8 : id;
  const int m0 = tile / g.tiles_n * BM, n0 = tile % g.tiles_n * BN;

  const char* Ag = reinterpret_cast<const char*>(g.A + (int64_t)m0 * g.lda);
  const char* Bg = reinterpret_cast<const char*>(BL == 1 ? g.B + (int64_t)n0 * g.ldb : g.B + n0);
  const int64_t b_step = BL == 1 ? BK * 2 : (int64_t)BK * g.ldb * 2;
  unsigned a_goff[LA], b_goff[LB];
#pragma unroll
  for (int i = 0; i < LA; i++) {
    const int R = 8 * (LA * wave + i) + (lane >> 3);
    a_goff[i] = (unsigned)((int64_t)R * g.lda * 2 + ((lane & 7) ^ ((R >> 1) & 7)) * 16);
  }
#pragma unroll
  for (int i = 0; i < LB; i++) {
    if (BL == 1) {
      const int R = 8 * (LB * wave + i) + (lane >> 3);
      b_goff[i] = (unsigned)((int64_t)R * g.ldb * 2 + ((lane & 7) ^ ((R >> 1) & 7)) * 16);
    } else {
      constexpr int CPR = BN / 8;   // chunks of a k row
      const int kr = 64 / CPR * (LB * wave + i) + lane / CPR;
      const int swz = BN == 128 ? kr & 3 : (kr >> 1) & 1;
      b_goff[i] = (unsigned)((int64_t)kr * g.ldb * 2 + ((lane % CPR) ^ (swz << 2)) * 16);
    }
  }
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)(smem_deep);
  auto issue = [&](int kt, int buf) {
    const char* ap = Ag + kt * (BK * 2);
    const char* bp = Bg + kt * b_step;
    const unsigned dst = lds0 + buf * TL::STAGE;
#pragma unroll
    for (int i = 0; i < LA; i++) deep_load_16(ap, a_goff[i], dst + (LA * wave + i) * 1024);
#pragma unroll
    for (int i = 0; i < LB; i++) deep_load_16(bp, b_goff[i], dst + TL::A_BYTES + (LB * wave + i) * 1024);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.0f;
  // fragment addresses: lane layouts as in gemm_mfma.hip
  const int fx = hf ^ (((lane & 31) >> 1) & 7);
  const int tx = BN == 128 ? (lane >> 2) & 3 : (lane >> 3) & 1;
  const int a_off = (wm * 64 + (lane & 31)) * 128;
  const int b_off = TL::A_BYTES + (BL == 1 ? (wn * TN * 32 + (lane & 31)) * 128
                                           : (hf * 8 + ((lane & 15) >> 2)) * (BN * 2) + ((lane >> 4) & 1) * 32 + (lane & 3) * 8);
  auto compute = [&](const char* s) {
    bf16x8 a[2][TM], b[2][TN];
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const int kk = 2 * share + q, pos = ((kk * 2) ^ fx) * 16;
#pragma unroll
      for (int j = 0; j < TN; j++) {
        if (BL == 1) b[q][j] = lds_read_direct(s + b_off + j * 32 * 128 + pos);
        else b[q][j] = lds_read_tr(s + b_off + kk * 16 * (BN * 2) + (((wn * TN + j) ^ tx) << 6), BN * 2);
      }
#pragma unroll
      for (int i = 0; i < TM; i++) a[q][i] = lds_read_direct(s + a_off + i * 32 * 128 + pos);
    }
#pragma unroll
    for (int q = 0; q < 2; q++)
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[q][j], a[q][i], acc[i][j], 0, 0, 0);
  };

  const int nk = g.K / BK;
#pragma unroll
  for (int s = 0; s < NST - 1; s++)
    if (s < nk) issue(s, s);
  int cur = 0;   // kt % NST
  for (int kt = 0; kt < nk; kt++) {
    deep_wait_for<LA + LB, NST - 2>(nk - 1 - kt);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt + NST - 1 < nk) issue(kt + NST - 1, cur == 0 ? NST - 1 : cur - 1);
    compute(smem_deep + cur * TL::STAGE);
    cur = cur == NST - 1 ? 0 : cur + 1;
  }

  typedef WaveEpilogue<1, TN, TN * 32, EPI, TO, false> EP;
  static_assert(32 * EP::PITCH == TL::STG, "staging");
  EP ep(g, lane, m0 + wm * 64 + share * 32, n0 + wn * TN * 32);
  ep.preload();
  __syncthreads();   // every wavefront is done with the operand buffers
  f32x16 own[1][TN];
  f32x4* give = reinterpret_cast<f32x4*>(smem_deep + wave * TL::XCHG);
  const f32x4* take = reinterpret_cast<const f32x4*>(smem_deep + (wave ^ 1) * TL::XCHG);
#pragma unroll
  for (int j = 0; j < TN; j++) {
    const f32x16 x = share ? acc[0][j] : acc[1][j];
    own[0][j] = share ? acc[1][j] : acc[0][j];
#pragma unroll
    for (int q = 0; q < 4; q++) give[(j * 4 + q) * 64 + lane] = (f32x4){x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < TN; j++)
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const f32x4 x = take[(j * 4 + q) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; e++) own[0][j][4 * q + e] += x[e];
    }
  ep.run(own, smem_deep + TL::NW * TL::XCHG + wave * TL::STG, reinterpret_cast<TO*>(g.C));
}

template <int BM, int BN, int NST, int BL, int EPI, typename TO>
int launch_deep(const MfmaArgs& a, hipStream_t st) {
  typedef DeepTile<BM, BN, NST> TL;
  auto kern = gemm_deep_kernel<BM, BN, NST, BL, EPI, TO>;
  static std::atomic<bool> attr_set{false};  // the call is idempotent: a race only repeats it
  if (!attr_set.load(std::memory_order_acquire)) {
    ALS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS_BYTES));
    attr_set.store(true, std::memory_order_release);
  }
  return launch_gemm(kern, a.tiles_m * a.tiles_n, TL::NT, TL::LDS_BYTES, st,
                     prof_id(PROF_DEEP, BM == 128 ? 0 : 2, 0, BL, EPI, sizeof(TO) == 2), product_flops(a.M, a.N, a.K), a);
}

template <int BM, int BN, int NST>
int run_deep(const GemmDesc& g, hipStream_t st) {
  MfmaArgs a;
  a.A = (const bf16*)g.A; a.B = (const bf16*)g.B; a.lda = g.lda; a.ldb = g.ldb;
  a.M = g.M; a.N = g.N; a.K = g.K; a.tiles_m = g.M / BM; a.tiles_n = g.N / BN;
  a.C = g.C; a.ldc = g.ldc; a.R = g.R; a.ldr = g.ldr; a.C2 = g.C2; a.U = (const bf16*)g.U;
  a.split_stride = 0; a.nsplit = 1;
  if (g.b_layout == 0) {
    if (g.epi == EPI_RESID) return launch_deep<BM, BN, NST, 0, EPI_RESID, float>(a, st);
    if (g.epi == EPI_GELU) return launch_deep<BM, BN, NST, 0, EPI_GELU, bf16>(a, st);
    if (g.c_bf16) return launch_deep<BM, BN, NST, 0, EPI_STORE, bf16>(a, st);
    return launch_deep<BM, BN, NST, 0, EPI_STORE, float>(a, st);
  }
  if (g.epi == EPI_DGELU) return launch_deep<BM, BN, NST, 1, EPI_DGELU, bf16>(a, st);
  if (g.c_bf16) return launch_deep<BM, BN, NST, 1, EPI_STORE, bf16>(a, st);
  return launch_deep<BM, BN, NST, 1, EPI_STORE, float>(a, st);
}

}  // namespace

int gemm_mfma_deep(const GemmDesc& g, int tile, hipStream_t st) {
  if (!gemm_mfma_supported(g) || g.a_layout != 0) return set_error(ALS_ERR_INVALID, "gemm_mfma_deep: unsupported shape or layout");
  return tile == 128 ? run_deep<128, 128, 4>(g, st) : run_deep<64, 64, 5>(g, st);
}

}  // namespace als
