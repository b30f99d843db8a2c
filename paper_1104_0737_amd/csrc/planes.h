// Column vectors and the plane-wise link layouts (internal.h) of the kernels
// that hold whole tiles of a domain in LDS.
#pragma once

#include "stencil.h"

namespace mbbs {

// C adjacent columns of one complex component.
template <typename R, int C> struct ColVec { typedef R T __attribute__((ext_vector_type(2 * C))); };
typedef unsigned u4 __attribute__((ext_vector_type(4)));

// Vectors of 16 bytes that hold a link in the domain-plane layout (internal.h).
template <int PR> constexpr int link_vecs() { return PR == P64 ? 9 : 5; }
// The link in direction MU whose first vector (of direction 0) is vector li.
template <int PR, int MU>
__device__ __forceinline__ void plane_link(const u4* __restrict__ U, unsigned li, int Vb, typename RawT<PR>::T* lk) {
  constexpr int NL = link_vecs<PR>(), W = 9 * RawT<PR>::per * (int)sizeof(typename RawT<PR>::T) / 4;
  unsigned w[4 * NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const u4 v = (U + (size_t)(MU * NL + i) * Vb)[li];
    w[4 * i] = v.x; w[4 * i + 1] = v.y; w[4 * i + 2] = v.z; w[4 * i + 3] = v.w;
  }
  __builtin_memcpy(lk, w, 4 * W);
}

// A barrier for what passes through LDS: unlike __syncthreads() it does not
// wait for this wave's global loads and stores in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

}  // namespace mbbs
