// FP32 / FP64 matrix-core fragments and complex accumulators.
#pragma once
#include "fb_internal.h"

namespace fb {

// ---------------------------------------------------------------- MFMA helpers
// One wave computes 16 rows of a complex product C (NB x T) += A (NB x K) B
// (K x T, in LDS) as three real 16x16x4 MFMAs per complex one (Gauss form,
// see Acc).  Operand fragments: lane l feeds A[l % 16][k + l / 16] and
// B[k + l / 16][l % 16].  Register r of lane l holds the element with the
// first operand's index row(l, r) and the second's l % 16, where row(l, r) =
// 4 (l / 16) + r for the f32 instruction and l / 16 + 4 r for the f64 one
// (both checked on gfx950).
typedef float mf_f4 __attribute__((ext_vector_type(4)));
typedef double mf_d4 __attribute__((ext_vector_type(4)));

template <typename R>
struct MF;
template <>
struct MF<float> {
  using V = mf_f4;
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
  static __device__ __forceinline__ V mma(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct MF<double> {
  using V = mf_d4;
  static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
  static __device__ __forceinline__ V mma(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// Complex accumulator of NC 16 x 16 tiles in Gauss form: the value is
// (p1 - p2) + i (p3 - p1 - p2), so that a complex product takes three real
// MFMA products (p1 += Ar Br, p2 += Ai Bi, p3 += (Ar + Ai)(Br + Bi)).
template <typename R, int NC>
struct Acc {
  typename MF<R>::V p1[NC], p2[NC], p3[NC];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p1[c][r] = (R)0;
        p2[c][r] = (R)0;
        p3[c][r] = (R)0;
      }
  }
  __device__ __forceinline__ cx<R> get(int c, int r) const {
    return mk<R>(p1[c][r] - p2[c][r], p3[c][r] - p1[c][r] - p2[c][r]);
  }
  __device__ __forceinline__ void set(int c, int r, cx<R> v) {
    p1[c][r] = v.x;
    p2[c][r] = (R)0;
    p3[c][r] = v.x + v.y;
  }
};

}  // namespace fb
