// The real 16 x 16 x 4 matrix instruction of a compute type.  Lane l holds A[l & 15][l >> 4] and
// B[l >> 4][l & 15]; element v of its result is D[row(l, v)][l & 15].
#pragma once

namespace qmg {

template <class C> struct Mm;
template <> struct Mm<float> {
  typedef float V4 __attribute__((ext_vector_type(4)));
  __device__ static V4 mul(float a, float b, V4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row(int lane, int v) { return 4 * (lane >> 4) + v; }  // of element v of the result
};
template <> struct Mm<double> {
  typedef double V4 __attribute__((ext_vector_type(4)));
  __device__ static V4 mul(double a, double b, V4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row(int lane, int v) { return (lane >> 4) + 4 * v; }
};

}  // namespace qmg
