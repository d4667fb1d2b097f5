// gelu_tanh and its derivative with the library's tanhf (fp32 mode and the generic GEMM).
#pragma once
#include <hip/hip_runtime.h>

namespace als {

__device__ __forceinline__ float gelu_tanh_f(float u) {
  const float a = 0.7978845608028654f, b = 0.044715f;
  return 0.5f * u * (1.0f + tanhf(a * (u + b * u * u * u)));
}
__device__ __forceinline__ float gelu_tanh_grad_f(float u) {
  const float a = 0.7978845608028654f, b = 0.044715f;
  float th = tanhf(a * (u + b * u * u * u));
  float inner = a * (1.0f + 3.0f * b * u * u);
  return 0.5f * (1.0f + th) + 0.5f * u * (1.0f - th * th) * inner;
}

}  // namespace als
