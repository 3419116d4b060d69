// cx_device.h -- device helpers shared by the library's kernels: the
// counter-based generator and global-address-space loads.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cx_internal.h"

namespace cx {
namespace {

struct U4 {
  uint32_t x, y, z, w;
};

// Philox4x32-10 (Salmon et al., SC'11).  The key is wave-uniform, so its
// schedule stays in scalar registers.
__device__ __forceinline__ U4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                     uint32_t k1) {
  // keep the round keys from being precomputed (and held in 20 scalar
  // registers) outside the step loop: bumping them costs two scalar adds
  asm volatile("" : "+s"(k0), "+s"(k1));
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // one 32x32->64 multiply per product gives both halves (v_mad_u64_u32)
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    // the two xors of each word in one v_bitop3 (truth table 0x96)
    c0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
    c1 = (uint32_t)p1;
    c2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
    c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return U4{c0, c1, c2, c3};
}

__device__ __forceinline__ float u24(uint32_t w) { return (float)(w >> 8) * 0x1p-24f; }

// Exploring starts: the price day of the episode that began at global step g0,
// (word 0 of Philox (env, g0, 0, DAY) * n_days) >> 32.
__device__ __forceinline__ int episode_day(uint32_t env, uint32_t g0, uint32_t k0, uint32_t k1, int n_days) {
  return (int)__umulhi(philox(env, g0, 0u, kDomDay, k0, k1).x, (uint32_t)n_days);
}

// Loads through the global address space (the tables live in device memory;
// plain pointers from a struct would be generic and compile to flat loads).
template <class T>
__device__ __forceinline__ T gld(const T *p, int64_t i) {
  return ((const __attribute__((address_space(1))) T *)p)[i];
}

// Load through the constant address space: with a wave-uniform address this
// is a scalar load (counted apart from the vector stores in flight, so using it
// does not wait for them).
template <class T>
__device__ __forceinline__ T sld(const T *p, int64_t i) {
  return ((const __attribute__((address_space(4))) T *)p)[i];
}

// Store through the global address space.
template <class T>
__device__ __forceinline__ void gst(T *p, int64_t i, T v) {
  ((__attribute__((address_space(1))) T *)p)[i] = v;
}

// Descriptors and class constants (SegDev, ClassDev) are the same for a whole
// block and never written by a kernel: read through the constant address space
// at a scalar address they are scalar loads into scalar registers.  Read
// through a plain pointer they would be vector loads, one vector register per
// constant for the whole rollout, and every branch on one a divergent branch.
#define CX_KONST const __attribute__((address_space(4)))
template <class T>
__device__ __forceinline__ CX_KONST T *konst(const T *p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (CX_KONST T *)(((uint64_t)hi << 32) | lo);
}

// The same pointer, unknown to the compiler: constants read through it are
// loaded where they are used instead of being held across the step loop (for
// the constants of work that is not done every step).
template <class T>
__device__ __forceinline__ CX_KONST T *reload(CX_KONST T *p) {
  uint64_t v = (uint64_t)p;
  asm volatile("" : "+s"(v));
  return (CX_KONST T *)v;
}

// A value known to be the same in every lane, in a scalar register.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

}  // namespace
}  // namespace cx
