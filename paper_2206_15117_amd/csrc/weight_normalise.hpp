// Weight normalisation of a few neighbouring pixels held as one vector.  Floats enter and leave a vector by copy: an array
// of them has a float's alignment, not the vector's.
#pragma once
#include <hip/hip_runtime.h>

namespace pg {

template <typename V>
struct Pixels {
  static constexpr int n = sizeof(V) / 4;
  float at[n];
  __host__ __device__ Pixels() {}
  __host__ __device__ explicit Pixels(const V& v) { __builtin_memcpy(at, &v, sizeof(V)); }
  __host__ __device__ V vector() const {
    V v;
    __builtin_memcpy(&v, at, sizeof(V));
    return v;
  }
};

template <typename V>
__host__ __device__ inline bool any_reaches(const Pixels<V>& weight, float min_weight) {
  bool any = false;
#pragma unroll
  for (int e = 0; e < Pixels<V>::n; ++e) any = any || weight.at[e] >= min_weight;
  return any;
}

// img / weight where the weight reaches min_weight, 0 elsewhere.
template <typename V>
__host__ __device__ inline V over_weight(const Pixels<V>& img, const Pixels<V>& weight, float min_weight) {
  Pixels<V> out;
#pragma unroll
  for (int e = 0; e < Pixels<V>::n; ++e) out.at[e] = weight.at[e] >= min_weight ? img.at[e] / weight.at[e] : 0.0f;
  return out.vector();
}

}  // namespace pg
