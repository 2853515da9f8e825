// Definitions shared by the matrix-product kernels (mt_gemm.hip, mt_gemm_small.hip): the kernel
// argument block, vector types and operand conversions.
#pragma once
#include "mt_internal.h"

namespace mt {

template <typename T>
__device__ __forceinline__ T pin_s(T x) {  // keep a uniform value in a scalar register
  asm volatile("" : "+s"(x));
  return x;
}

struct Problems {
  GemmProblem p[2];
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

template <typename T>
__device__ __forceinline__ T bitcast16(const u32x4 &v) {
  T r;
  __builtin_memcpy(&r, &v, 16);
  return r;
}

__device__ __forceinline__ u32x4 pack_bf16x8(const u32x4 &lo, const u32x4 &hi) {
  float a[4], b[4];
  __builtin_memcpy(a, &lo, 16);
  __builtin_memcpy(b, &hi, 16);
  bf16x8 h;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    h[j] = to_bf16(a[j]);
    h[4 + j] = to_bf16(b[j]);
  }
  u32x4 r;
  __builtin_memcpy(&r, &h, 16);
  return r;
}

// Products of few rows (mt_gemm_small.hip); the problems as launch_gemm has checked them
hipError_t launch_gemm_small(int bf16_mma, const Problems &ps, int nprob, Epilogue epi, hipStream_t st);

}  // namespace mt
