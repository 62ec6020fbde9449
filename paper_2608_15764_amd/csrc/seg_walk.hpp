// Walking a buffer in 64-lane segments, modulo its size, with the least
// scalar work between two loads.
//
// A wave issues its K loads of a group one after another, and between two of
// them it steps to the next segment and wraps at the buffer's end.  That
// arithmetic is scalar, and the four SIMDs of a CU issue about one scalar
// instruction per clock between them: where the data comes from the caches
// it bounds the rate of loads, and where few waves are resident it spreads
// the K loads of a group in time.  With vector indices in 64 bits a step was
// eleven scalar instructions and a vector compare.
//
//  Near  buffers below 4 GiB.  Byte offsets in 32 bits: compare, select, add;
//        the offset goes into the load (buffer loads) or onto the base
//        (global loads, two instructions more).
//  Far   larger ones.  A 64-bit cursor that counts up to zero from minus the
//        buffer's size, so that the wrap is a test of its sign: nine.
//
// The K sweep of 4-byte loads over 4 MiB (32 cells, 1 GiB read in each, 16
// waves per CU): 4322 -> 3591 us, 8.0 -> 9.6 TB/s (3442 with the loads placed
// ahead, as the plain loop does); 16-byte loads over 1 GiB, bound by HBM, gain
// 1 % at 8 waves per CU.
#pragma once

#include <type_traits>

#include "device.hpp"

namespace ilp {

// Address-space-1 pointers keep a base that went through an integer a global
// (not flat) address.
typedef __attribute__((address_space(1))) const uint8_t* GlobalBytes;

// A segment's address, made here and kept scalar: folded into one 64-bit
// vector address it would cost a vector add and two registers per load, and
// carried as a cursor it would be added up in front of the load.
__device__ __forceinline__ uint64_t scalar_address(uint64_t a) {
  asm("" : "+s"(a));
  return a;
}

// A lane's V bytes at seg + lane_off.
template <int V, int POL>
__device__ __forceinline__ typename Vec<V>::T load_global(uint64_t seg, uint32_t lane_off) {
  typedef typename Vec<V>::T T;
  typedef __attribute__((address_space(1))) const T* P;
  const P p = (P)((GlobalBytes)seg + lane_off);
  if constexpr (POL == SWEEP_CACHE_NT) return __builtin_nontemporal_load(p);
  else return *p;
}

template <int V, int POL>
__device__ __forceinline__ typename Vec<V>::T load_buffer(__amdgpu_buffer_rsrc_t r,
                                                          uint32_t lane_off, uint32_t off) {
  constexpr int aux = POL == SWEEP_CACHE_BYPASS_L1 ? kAuxSc1 : kAuxSc1Nt;
  if constexpr (V == 4) return __builtin_amdgcn_raw_buffer_load_b32(r, lane_off, off, aux);
  else if constexpr (V == 8) return __builtin_amdgcn_raw_buffer_load_b64(r, lane_off, off, aux);
  else return __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, aux);
}

// (o + d) mod n in bytes, for o < n: d and n - d are the walk's constants.
struct NearStep {
  uint32_t d, back;      // step, and n minus the step
  __device__ __forceinline__ NearStep(uint64_t step, uint64_t n)
      : d((uint32_t)step), back((uint32_t)(n - step)) {}
  __device__ __forceinline__ uint32_t operator()(uint32_t o) const {
    return o + (o >= back ? 0u - back : d);
  }
};

template <int V, int POL>
struct NearWalk {
  typedef uint32_t Cursor;
  typedef NearStep Step;
  static constexpr bool kBuffer = POL == SWEEP_CACHE_BYPASS_L1 || POL == SWEEP_CACHE_BYPASS_L1_NT;
  uint64_t base;
  __amdgpu_buffer_rsrc_t r;
  uint32_t lane_off;
  __device__ __forceinline__ NearWalk(const uint8_t* buf, uint64_t n, uint32_t lane)
      : base((uint64_t)buf),
        r(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(buf), 0, (int)(uint32_t)n,
                                            kRsrcWord3)),
        lane_off(lane * V) {}
  __device__ __forceinline__ Step step(uint64_t d, uint64_t n) const { return Step(d, n); }
  __device__ __forceinline__ Cursor at(uint64_t off) const { return (uint32_t)off; }
  // The lane's byte offset in a segment, made anew in each group: hoisted out
  // of the loop as a 64-bit value it could not be a load's 32-bit offset.
  __device__ __forceinline__ uint32_t lane_offset() const {
    uint32_t o = lane_off;
    if constexpr (!kBuffer) asm volatile("" : "+v"(o));
    return o;
  }
  // Where a segment's load starts: its offset in the buffer, or its address.
  typedef std::conditional_t<kBuffer, uint32_t, uint64_t> Start;
  __device__ __forceinline__ Start start(Cursor c) const {
    if constexpr (kBuffer) return c;
    else return scalar_address(base + c);
  }
  __device__ __forceinline__ typename Vec<V>::T load(Start at, uint32_t lo) const {
    if constexpr (kBuffer) return load_buffer<V, POL>(r, lo, at);
    else return load_global<V, POL>(at, lo);
  }
  // for LDS-direct requests, which are global loads under every policy
  __device__ __forceinline__ uint64_t address(Cursor c) const { return base + c; }
  __device__ __forceinline__ uint32_t lds_lane_offset() const {
    uint32_t o = lane_off;
    asm volatile("" : "+v"(o));
    return o;
  }
};

// The cursor is offset - n, in [-n, 0).
struct FarStep {
  int64_t d, n;
  __device__ __forceinline__ FarStep(uint64_t step, uint64_t size)
      : d((int64_t)step), n((int64_t)size) {}
  __device__ __forceinline__ int64_t operator()(int64_t c) const {
    c += d;
    int32_t hi = (int32_t)(c >> 32);
    asm("" : "+s"(hi));       // a scalar compare of the sign, not a 64-bit vector one
    return c - (hi >= 0 ? n : 0);
  }
};

template <int V, int POL>
struct FarWalk {
  typedef int64_t Cursor;
  typedef FarStep Step;
  static constexpr bool kBuffer = NearWalk<V, POL>::kBuffer;
  uint64_t end;
  uint64_t n;
  uint32_t lane;
  __device__ __forceinline__ FarWalk(const uint8_t* buf, uint64_t size, uint32_t l)
      : end((uint64_t)buf + size), n(size), lane(l) {}
  __device__ __forceinline__ Step step(uint64_t d, uint64_t size) const { return Step(d, size); }
  __device__ __forceinline__ Cursor at(uint64_t off) const { return (int64_t)off - (int64_t)n; }
  __device__ __forceinline__ uint32_t lane_offset() const {
    uint32_t o = lane * V;
    if constexpr (!kBuffer) asm volatile("" : "+v"(o));
    return o;
  }
  typedef uint64_t Start;
  __device__ __forceinline__ Start start(Cursor c) const {
    return scalar_address(end + (uint64_t)c);
  }
  __device__ __forceinline__ typename Vec<V>::T load(Start seg, uint32_t lo) const {
    if constexpr (kBuffer) {
      // a buffer of this one segment
      return load_buffer<V, POL>(
          __builtin_amdgcn_make_buffer_rsrc((void*)seg, 0, kWave * V, kRsrcWord3), lo, 0u);
    } else {
      return load_global<V, POL>(seg, lo);
    }
  }
  __device__ __forceinline__ uint64_t address(Cursor c) const { return end + (uint64_t)c; }
  __device__ __forceinline__ uint32_t lds_lane_offset() const {
    uint32_t o = lane * V;
    asm volatile("" : "+v"(o));
    return o;
  }
};

}  // namespace ilp
