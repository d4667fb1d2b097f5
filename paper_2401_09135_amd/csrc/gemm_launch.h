// Launch of a GEMM kernel, with the events of als_prof_enable around it when those are on (and it is this launch's turn).
#pragma once
#include <atomic>
#include <hip/hip_ext.h>

#include "common.h"

namespace als {

// What als_prof_kernel_name names: the kernels of gemm_mfma.hip have ids of their own below 1 << 13.
enum ProfKind { PROF_DEEP = 1, PROF_ANY, PROF_F32, PROF_ANY_LIST, PROF_F32_LIST };
inline int prof_id(ProfKind kind, int tile, int al = 0, int bl = 0, int epi = 0, int out_bf16 = 0) {
  return kind << 13 | tile | al << 3 | bl << 4 | epi << 5 | out_bf16 << 7;
}

struct ProfRec { hipEvent_t e0, e1; int id; double flops; };
extern std::atomic<bool> g_prof_on;
bool prof_begin(ProfRec* rec);   // false: this launch is not timed
void prof_end(const ProfRec& rec);

template <typename Kernel, typename... Args>
int launch_gemm(Kernel kern, int blocks, int threads, size_t lds, hipStream_t st, int id, double flops, const Args&... args) {
  ProfRec rec;
  rec.id = id;
  rec.flops = flops;
  const bool timed = g_prof_on.load(std::memory_order_relaxed) && prof_begin(&rec);
  // start/stop events attached to the dispatch itself: their difference is the kernel's own execution time, as a profiler
  // reports it
  if (timed) hipExtLaunchKernelGGL(kern, dim3(blocks), dim3(threads), lds, st, rec.e0, rec.e1, 0, args...);
  else hipLaunchKernelGGL(kern, dim3(blocks), dim3(threads), lds, st, args...);
  ALS_CHECK_LAUNCH();
  if (timed) prof_end(rec);
  return ALS_OK;
}
inline double product_flops(int M, int N, int K) { return 2.0 * M * N * (double)K; }
inline double list_flops(const DwList& l) {
  double f = 0.0;
  for (int i = 0; i < l.n; i++) f += product_flops(l.p[i].M, l.p[i].N, l.K);
  return f;
}

}  // namespace als
