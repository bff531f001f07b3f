// mfma.hpp -- the 16x16x4 matrix instructions in both precisions, and the
// workgroup order over the XCDs.
#pragma once
#include <hip/hip_runtime.h>

namespace mp3 {

typedef float mfma_f4 __attribute__((ext_vector_type(4)));
typedef double mfma_d4 __attribute__((ext_vector_type(4)));

template <typename T> struct acc4;
template <> struct acc4<float> { using type = mfma_f4; };
template <> struct acc4<double> { using type = mfma_d4; };

// D += A B over four k: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]
__device__ __forceinline__ mfma_f4 mfma16(float a, float b, mfma_f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ mfma_d4 mfma16(double a, double b, mfma_d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// row of D register i of lane l (column l % 16)
template <typename T> __device__ __forceinline__ int mfma_row(int lane, int i);
template <> __device__ __forceinline__ int mfma_row<float>(int lane, int i) { return 4 * (lane >> 4) + i; }
template <> __device__ __forceinline__ int mfma_row<double>(int lane, int i) { return 4 * i + (lane >> 4); }

// consecutive tasks on one XCD (workgroups are dealt to the 8 XCDs in turn), so that
// neighbouring tiles find each other's halo in that XCD's L2
__device__ __forceinline__ int xcd_order(int i, int n) { return n % 8 == 0 ? (i & 7) * (n / 8) + (i >> 3) : i; }

}  // namespace mp3
