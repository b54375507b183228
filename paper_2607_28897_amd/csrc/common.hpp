// common.hpp -- shared host and device helpers of the batched big-integer
// library (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/bigint_rocm.h"

typedef int v4i __attribute__((ext_vector_type(4)));

namespace bi {

// ---------------------------------------------------------------------------
// Host-side error plumbing
// ---------------------------------------------------------------------------
void set_hip_error(hipError_t e);

#define BI_HIP(call)                                                        \
  do {                                                                      \
    hipError_t e_ = (call);                                                 \
    if (e_ != hipSuccess) {                                                 \
      ::bi::set_hip_error(e_);                                              \
      return BIGINT_EHIP;                                                   \
    }                                                                       \
  } while (0)

#define BI_LAUNCH_CHECK()                                                   \
  do {                                                                      \
    hipError_t e_ = hipGetLastError();                                      \
    if (e_ != hipSuccess) {                                                 \
      ::bi::set_hip_error(e_);                                              \
      return BIGINT_EHIP;                                                   \
    }                                                                       \
  } while (0)

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------------------
// Device helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }
__device__ __forceinline__ int num_waves() { return blockDim.x >> 6; }

// Four limbs at any limb address: one 16-byte access (gfx950 takes 4-byte
// aligned ones; rows of odd length need it on three rows of four)
struct __attribute__((packed, aligned(4))) Limb4 {
  uint32_t x, y, z, w;
};
__device__ __forceinline__ Limb4 load4(const uint32_t* p) { return *reinterpret_cast<const Limb4*>(p); }
__device__ __forceinline__ void store4(uint32_t* p, uint32_t x, uint32_t y, uint32_t z, uint32_t w) {
  *reinterpret_cast<Limb4*>(p) = Limb4{x, y, z, w};
}

// Carry (or borrow) resolution over the 64 lanes of a wave.
//
// Each lane summarises a contiguous run of limbs by (g, p): g = the run emits
// a carry when none enters, p = the run passes an entering carry through
// (g and p are never both set).  This is the carry operator of Section 5.1
// (the pair (overflow, all-ones) combined by an associative operator and
// exclusively scanned).  On a wave the scan is one 64-bit integer addition
// of the ballot masks: with A = G|P and carry-in c, bit i of (A + G + c) ^ A
// ^ G is exactly the carry entering lane i, because a lane with g behaves
// like the bit pair (1,1), p like (1,0) and neither like (0,0).
struct WaveCarry {
  uint64_t G, P;
};

__device__ __forceinline__ WaveCarry wave_carry_masks(bool g, bool p) {
  WaveCarry w;
  w.G = __ballot(g);
  w.P = __ballot(p);
  return w;
}

// Carry into this lane given the carry c entering lane 0 of the wave.
__device__ __forceinline__ uint32_t wave_carry_in(const WaveCarry& w, uint32_t c) {
  const uint64_t A = w.G | w.P;
  const uint64_t S = A + w.G + (uint64_t)c;
  const uint64_t Cin = S ^ A ^ w.G;
  return (uint32_t)((Cin >> lane_id()) & 1ull);
}

// Carry leaving lane 63 given carry-in c.
__device__ __forceinline__ uint32_t wave_carry_out(const WaveCarry& w, uint32_t c) {
  const uint64_t A = w.G | w.P;
  const uint64_t s1 = A + w.G;
  const uint32_t o1 = s1 < A;             // overflow of A + G
  const uint64_t s2 = s1 + (uint64_t)c;
  const uint32_t o2 = s2 < s1;            // overflow of + c
  return o1 | o2;
}

// the carry out of bit 63 and the carries into every bit of g + p bits with
// carry c into bit 0 (p: propagate, g: generate, disjoint)
__device__ __forceinline__ uint64_t carry_bits(uint64_t g, uint64_t p, uint32_t& c) {
  const uint64_t a = g | p, s = a + g + c;
  c = (uint32_t)(g >> 32 | (a >> 32 & ~(s >> 32))) >> 31;
  return s ^ a ^ g;
}

// Work-group wide exclusive carry scan.  Every thread passes the (g, p)
// summary of its own limb run; returns the carry entering that run.  cin is
// the carry entering the whole work-group range.  `scratch` is >= 16 u32 of
// LDS; the function synchronises the work-group twice and leaves scratch
// free for reuse on return.  *cout (optional, all threads) = carry leaving
// the last thread.
__device__ __forceinline__ uint32_t wg_carry_scan(bool g, bool p, uint32_t cin,
                                                  uint32_t* scratch,
                                                  uint32_t* cout) {
  const WaveCarry w = wave_carry_masks(g, p);
  const int wid = wave_id(), nw = num_waves();
  // wave summary for the work-group level: generate with carry-in 0,
  // propagate = every lane propagates
  const uint32_t gw = wave_carry_out(w, 0);
  const uint32_t pw = (w.P == ~0ull);
  if (lane_id() == 0) scratch[wid] = gw | (pw << 1);
  __syncthreads();
  uint32_t c = cin;
  for (int k = 0; k < wid; ++k) {
    const uint32_t s = scratch[k];
    c = (s & 1u) | ((s >> 1) & c);
  }
  if (cout) {
    uint32_t t = c;
    for (int k = wid; k < nw; ++k) {
      const uint32_t s = scratch[k];
      t = (s & 1u) | ((s >> 1) & t);
    }
    *cout = t;
  }
  const uint32_t r = wave_carry_in(w, c);
  __syncthreads();
  return r;
}

// Bits [7k, 7k+7) of the n-limb integer a (0 outside): the k-th 7-bit digit.
__device__ __forceinline__ uint32_t digit7(const uint32_t* __restrict__ a, int n, int k) {
  const int bit = 7 * k;
  const int l = bit >> 5, s = bit & 31;
  if (k < 0 || l >= n) return 0;
  uint32_t v = a[l] >> s;
  if (s > 25 && l + 1 < n) v |= a[l + 1] << (32 - s);
  return v & 127u;
}

// a pointer that is the same in every lane, in scalar registers
template <class T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (T*)(((uint64_t)hi << 32) | lo);
}

// n limbs behind a buffer descriptor: reads past the end give 0 and writes
// there are dropped, with no compare or mask
struct Limbs {
  __amdgpu_buffer_rsrc_t d;
  int n;
  __device__ __forceinline__ Limbs(const uint32_t* p, int n_)
      : d(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p), 0, 4 * n_, 0x00020000)), n(n_) {}
  __device__ __forceinline__ uint32_t operator()(int i) const {
    return __builtin_amdgcn_raw_buffer_load_b32(d, 4 * i, 0, 0);
  }
  __device__ __forceinline__ void put(int i, uint32_t v) const {
    __builtin_amdgcn_raw_buffer_store_b32(v, d, 4 * i, 0, 0);
  }
};

}  // namespace bi
