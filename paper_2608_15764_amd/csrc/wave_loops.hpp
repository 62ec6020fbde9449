// Wave-level loops shared by the LDS-ring kernels and the two-stream
// kernel.  A wave owns wave-groups q = wid, wid + n_waves, ... below Q; the
// request for load j of group q is the 64-lane segment starting at vector
// (q*D + j)*64 mod n_vec, exactly the plain map with K = D.
//
// At one or two waves per CU these loops are bound by a wave's own
// instruction stream, from a slot's arrival to its refill.  The steps between
// requests are scalar (seg_walk.hpp), the LDS-direct ring refills a slot
// before it folds what it read, and the scheduling barriers keep the requests
// in the order in which the loop waits for them, so that every wait leaves
// D - 1 in flight.  2 GiB, one wave per CU, depth 8 and 16: LDS-direct 590 ->
// 555 and 505 -> 392 us, matched 780 -> 545 and 560 -> 437 under the default
// policy (585 -> 537 and 462 -> 431 with sc1 nt); two streams of 4 waves on
// different CUs at depth 4, 415 -> 336 us.  From 4 waves per CU and depth 8
// on HBM bounds them, as before.
#pragma once

#include <utility>

#include "device.hpp"
#include "seg_walk.hpp"

namespace ilp {

constexpr uint64_t kSegBytes = kWave * 16;   // one 64-lane segment of 16-byte vectors

template <typename F, int... Js>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Js...>) {
  (f(std::integral_constant<int, Js>{}), ...);
}
// f(integral_constant<int, J>) for J = 0 .. N-1, fully unrolled
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// One wave's share of a region: its groups and their addresses, in bytes.
struct Share {
  const uint8_t* buf;
  uint64_t bytes;
  uint64_t stride;      // between two of the wave's groups, mod bytes
  uint32_t wid;
  uint32_t iters;       // groups of this wave
};

// Start of the wave's first group of D segments; most lie inside the region.
template <int D>
__device__ __forceinline__ uint64_t first_group(const Share& a) {
  uint64_t off = (uint64_t)a.wid * (D * kSegBytes);
  if (off >= a.bytes) off %= a.bytes;
  return off;
}

// One 16-byte-per-lane LDS-direct request: lane l's bytes land in
// slot[l] (global_load_lds_dwordx4 writes LDS at M0 + 16*lane).  The last
// builtin operand is the cache policy: 0, nt (2), sc1 (16) or sc1 nt (18).
template <int POL>
__device__ __forceinline__ void lds_issue(uint64_t seg, uint32_t lane_off, u32x4* slot) {
  typedef __attribute__((address_space(3))) void lds_void;
  lds_void* dst = (lds_void*)slot;
  asm("" : "+s"(seg));
  const GlobalBytes src = (GlobalBytes)seg + lane_off;
  if constexpr (POL == SWEEP_CACHE_DEFAULT) {
    __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
  } else if constexpr (POL == SWEEP_CACHE_NT) {
    __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 2);
  } else if constexpr (POL == SWEEP_CACHE_BYPASS_L1) {
    __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 16);
  } else {
    __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 18);
  }
}

// Plain batched loop (K loads, then K folds) over one region.
template <int K, class W>
__device__ __forceinline__ void plain_loop16(const Share& a, uint32_t lane, uint32_t& s,
                                             uint32_t& x) {
  if (a.iters == 0) return;
  const W walk(a.buf, a.bytes, lane);
  const typename W::Step next_load = walk.step(kSegBytes % a.bytes, a.bytes);
  const typename W::Step next_group = walk.step(a.stride, a.bytes);
  typename W::Cursor p = walk.at(first_group<K>(a));
  typename W::Start at[K];      // of the next group, found while one is in flight
  auto place = [&] {
    typename W::Cursor pj = p;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      at[j] = walk.start(pj);
      pj = next_load(pj);
    }
  };
  place();
#pragma unroll 1
  for (uint32_t i = a.iters; i; --i) {
    u32x4 v[K];
    const uint32_t lo = walk.lane_offset();
#pragma unroll
    for (int j = 0; j < K; ++j) v[j] = walk.load(at[j], lo);
    __builtin_amdgcn_sched_barrier(0);
    p = next_group(p);
    place();
    __builtin_amdgcn_sched_barrier(0);   // all K issued before any fold
#pragma unroll
    for (int j = 0; j < K; ++j) fold(v[j], s, x);
  }
}

// LDS-direct ring of depth D: D requests in flight, each slot read as soon
// as it lands (s_waitcnt vmcnt(D-1)) and refilled at once; the read words
// are folded behind the refill, which is what the ring waits for.
template <int D, int POL, class W>
__device__ __forceinline__ void async_ring_loop(const Share& a, uint32_t lane, u32x4* ring,
                                                uint32_t& s, uint32_t& x) {
  if (a.iters == 0) return;
  const W walk(a.buf, a.bytes, lane);
  const typename W::Step next_load = walk.step(kSegBytes % a.bytes, a.bytes);
  const typename W::Step next_group = walk.step(a.stride, a.bytes);
  typename W::Cursor p = walk.at(first_group<D>(a));
  {
    typename W::Cursor pj = p;
    const uint32_t lo = walk.lds_lane_offset();
    static_for<D>([&](auto J) {
      lds_issue<POL>(walk.address(pj), lo, ring + J * kWave);
      __builtin_amdgcn_sched_barrier(0);   // in the order the loop waits for them
      pj = next_load(pj);
    });
  }
#pragma unroll 1
  for (uint32_t i = a.iters - 1; i; --i) {
    p = next_group(p);
    typename W::Cursor pj = p;
    const uint32_t lo = walk.lds_lane_offset();
    static_for<D>([&](auto J) {
      wait_vmcnt<D - 1>();
      const u32x4 v = ring[J * kWave + lane];
      wait_lgkmcnt0();      // the slot's read has returned before refill
      lds_issue<POL>(walk.address(pj), lo, ring + J * kWave);
      fold(v, s, x);
      pj = next_load(pj);
    });
  }
  static_for<D>([&](auto J) {
    wait_vmcnt<D - 1 - J>();
    const u32x4 v = ring[J * kWave + lane];
    fold(v, s, x);
  });
}

// Matched plain ring: the same D requests in flight, loaded into registers,
// then written to the lane's LDS slot and read back before folding.
template <int D, class W>
__device__ __forceinline__ void matched_ring_loop(const Share& a, uint32_t lane, u32x4* ring,
                                                  uint32_t& s, uint32_t& x) {
  if (a.iters == 0) return;
  const W walk(a.buf, a.bytes, lane);
  const typename W::Step next_load = walk.step(kSegBytes % a.bytes, a.bytes);
  const typename W::Step next_group = walk.step(a.stride, a.bytes);
  typename W::Cursor p = walk.at(first_group<D>(a));
  u32x4 v[D];
  {
    typename W::Cursor pj = p;
    const uint32_t lo = walk.lane_offset();
    static_for<D>([&](auto J) {
      v[J] = walk.load(walk.start(pj), lo);
      __builtin_amdgcn_sched_barrier(0);   // in the order the loop waits for them
      pj = next_load(pj);
    });
  }
  auto through_lds = [&](int j) {
    ring[j * kWave + lane] = v[j];
    compiler_fence();       // no store-to-load forwarding through LDS
    const u32x4 r = ring[j * kWave + lane];
    fold(r, s, x);
    asm("" : "+v"(s));      // summed now: summed at the end, D vectors would wait
    compiler_fence();       // the refill below stays after this fold
  };
#pragma unroll 1
  for (uint32_t i = a.iters - 1; i; --i) {
    p = next_group(p);
    typename W::Cursor pj = p;
    const uint32_t lo = walk.lane_offset();
    static_for<D>([&](auto J) {
      through_lds(J);
      v[J] = walk.load(walk.start(pj), lo);
      __builtin_amdgcn_sched_barrier(0);   // before the wait for the next slot
      pj = next_load(pj);
    });
  }
  static_for<D>([&](auto J) { through_lds(J); });
}

}  // namespace ilp
