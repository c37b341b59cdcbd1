// Several (tile, filter) pairs per lane: N floats that the add networks of sfc_points.hpp treat as one
// value, and the broadcast that hands a lane its dequantization factor.
#pragma once
#include "sfc_points.hpp"

namespace sfc {

template <int N>
struct Floats {
  float v[N];
  Floats() = default;
  __device__ __forceinline__ explicit Floats(float s) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = s;
  }
};
template <int N>
__device__ __forceinline__ Floats<N> operator+(const Floats<N>& a, const Floats<N>& b) {
  Floats<N> r;
#pragma unroll
  for (int i = 0; i < N; ++i) r.v[i] = a.v[i] + b.v[i];
  return r;
}
template <int N>
__device__ __forceinline__ Floats<N> operator-(const Floats<N>& a, const Floats<N>& b) {
  Floats<N> r;
#pragma unroll
  for (int i = 0; i < N; ++i) r.v[i] = a.v[i] - b.v[i];
  return r;
}
template <int N>
__device__ __forceinline__ Floats<N> operator*(const Floats<N>& a, const Floats<N>& b) {
  Floats<N> r;
#pragma unroll
  for (int i = 0; i < N; ++i) r.v[i] = a.v[i] * b.v[i];
  return r;
}
template <int N>
__device__ __forceinline__ Floats<N> operator-(const Floats<N>& a) {
  Floats<N> r;
#pragma unroll
  for (int i = 0; i < N; ++i) r.v[i] = -a.v[i];
  return r;
}
template <int N>
struct Half<Floats<N>> {
  static __device__ __forceinline__ Floats<N> apply(const Floats<N>& a) { return a * Floats<N>(0.5f); }
};
template <int N>
struct Third<Floats<N>> {
  static __device__ __forceinline__ Floats<N> apply(const Floats<N>& a) { return a * Floats<N>(1.0f / 3.0f); }
};
using f4 = Floats<4>;
using f2 = Floats<2>;

// Lane n of the reader's row of 16 lanes (its quarter of the wave), as a DPP row broadcast:
// folds into the instruction that takes the value.
template <int N>
__device__ __forceinline__ float row_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + N, 0xf, 0xf, false));
}

}  // namespace sfc
