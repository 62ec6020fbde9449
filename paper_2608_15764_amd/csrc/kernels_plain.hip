// Plain K-load sweep kernel (the hot loop of the method, Section 3 "The
// axis K" and Section 4.2).
//
// One wavefront-iteration issues K independent loads - each one contiguous,
// coalesced 64-lane segment of 64*V bytes, adjacent to each other or (the
// strided layout) Q segments apart - into K distinct register sets,
// and only then folds them, oldest first; nothing from the next iteration is
// in flight meanwhile, so a wave has at most K loads outstanding.  The loop
// itself never stores: the sinks leave the kernel in one record per wave.
#include <array>
#include <utility>

#include "device.hpp"
#include "kernels.hpp"
#include "seg_walk.hpp"

namespace ilp {

template <int K, int V, int POL, template <int, int> class Walk, bool SPACED>
__device__ __forceinline__ void plain_cell(const PlainArgs& a) {
  const uint64_t t0 = wall_ticks();
  const uint32_t lane = lane_id();
  const uint32_t wid = blockIdx.x * (kPlainWgThreads / kWave) + wave_in_wg();

  // Sinks of even and odd loads.  Two chains are no faster than one; they
  // keep the cells that do not reach 8 waves per SIMD what they were, K = 15
  // and 16 with 16-byte loads (66 and 70 registers; one chain would need 64).
  uint32_t s = 0, x = 0, s1 = 0, x1 = 0;
  // this wave's first group and their number (wave-uniform scalars)
  uint64_t q0 = wid;
  uint32_t iters = a.iters + (wid < a.extra ? 1u : 0u);
  if (a.order == SWEEP_ORDER_BLOCKED) {
    q0 = (uint64_t)wid * a.G;
    const uint64_t left = q0 < a.Q ? a.Q - q0 : 0;
    iters = (uint32_t)(left < a.G ? left : a.G);
  }
  if (iters) {
    typedef Walk<V, POL> W;
    const W walk(a.buf, a.bytes, lane);
    const typename W::Step next_load = walk.step(a.jstep, a.bytes);
    const typename W::Step next_group = walk.step(a.stride, a.bytes);
    // the first group's start; most lie inside the buffer
    uint64_t off = q0 * a.gstep;
    if (off >= a.bytes) off %= a.bytes;
    typename W::Cursor p = walk.at(off);
    typename W::Start at[K];
    auto place = [&] {
      typename W::Cursor pj = p;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        at[j] = walk.start(pj);
        pj = next_load(pj);
      }
    };
    // The K loads go into K register sets, all of them before the first is
    // folded (the barrier: without it the scheduler may refill registers
    // early to raise occupancy).  Where the next group's loads start is worked
    // out while this one's are in flight, so that a group goes out at once:
    // 1 GiB in 4-byte loads at 4 waves per CU, K = 2 / 4 / 8 / 14, 891 / 520 /
    // 322 / 228 us with the steps between the loads, 864 / 463 / 275 / 192 with
    // them ahead; 16-byte loads, 4 waves, K = 4, 5460 -> 6150 GB/s.
    place();
#pragma unroll 1
    for (; iters; --iters) {
      typename Vec<V>::T v[K];
      const uint32_t lo = walk.lane_offset();
#pragma unroll
      for (int j = 0; j < K; ++j) {
        v[j] = walk.load(at[j], lo);
        if (SPACED && j + 1 < K) {
          // 16 idle cycles; see the rule at plain_kernel
          __builtin_amdgcn_sched_barrier(0);
          asm volatile("s_nop 15");
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      p = next_group(p);
      place();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < K; ++j) {
        if (j & 1) fold(v[j], s1, x1);
        else fold(v[j], s, x);
      }
    }
    s += s1;
    x ^= x1;
  }
  const uint64_t t1 = wall_ticks();
  wave_epilogue(s, x, t0, t1, wid, a.rec, a.lane_out);
}

template <int K, int V, int POL>
__global__ __launch_bounds__(kPlainWgThreads) void plain_kload(PlainArgs a) {
  plain_cell<K, V, POL, NearWalk, false>(a);
}

// The same cell with a gap between the loads of a group, for cells that
// saturate HBM.
template <int K, int V, int POL>
__global__ __launch_bounds__(kPlainWgThreads) void plain_kload_spaced(PlainArgs a) {
  plain_cell<K, V, POL, NearWalk, true>(a);
}

// The same cells over 4 GiB and more.
template <int K, int V, int POL>
__global__ __launch_bounds__(kPlainWgThreads) void plain_kload_far(PlainArgs a) {
  plain_cell<K, V, POL, FarWalk, false>(a);
}

template <int K, int V, int POL>
__global__ __launch_bounds__(kPlainWgThreads) void plain_kload_far_spaced(PlainArgs a) {
  plain_cell<K, V, POL, FarWalk, true>(a);
}

namespace {

typedef void (*PlainFn)(PlainArgs);

// (of one load there is nothing to space)
template <int K, int V, int POL>
constexpr PlainFn spaced() {
  if constexpr (K == 1) return &plain_kload<K, V, POL>;
  else return &plain_kload_spaced<K, V, POL>;
}
template <int K, int V, int POL>
constexpr PlainFn far_spaced() {
  if constexpr (K == 1) return &plain_kload_far<K, V, POL>;
  else return &plain_kload_far_spaced<K, V, POL>;
}

template <int V, int POL, int... Ks>
constexpr std::array<PlainFn, 4 * sizeof...(Ks)> row(std::integer_sequence<int, Ks...>) {
  return {&plain_kload<Ks + 1, V, POL>..., spaced<Ks + 1, V, POL>()...,
          &plain_kload_far<Ks + 1, V, POL>..., far_spaced<Ks + 1, V, POL>()...};
}

template <int V, int POL>
constexpr auto kRow = row<V, POL>(std::make_integer_sequence<int, kMaxK>{});

// [vector width index][policy][(2 * far + spaced) * kMaxK + K-1]
const PlainFn* table(int vi, int pol) {
  static const std::array<PlainFn, 4 * kMaxK> t[3][kNumPolicies] = {
      {kRow<4, 0>, kRow<4, 1>, kRow<4, 2>, kRow<4, 3>},
      {kRow<8, 0>, kRow<8, 1>, kRow<8, 2>, kRow<8, 3>},
      {kRow<16, 0>, kRow<16, 1>, kRow<16, 2>, kRow<16, 3>},
  };
  return t[vi][pol].data();
}

int width_index(int V) { return V == 4 ? 0 : V == 8 ? 1 : V == 16 ? 2 : -1; }

// Which form a cell takes: a rule on everything but K, so that the loop is one
// and the same along a K curve (a single load has no gap in either form).
// K loads sent at once by many waves reach a saturated HBM as bursts that some
// strides fold onto few channels; a gap between loads spreads them, and costs
// what it delays elsewhere.  So each form wins at some K and loses at others,
// and the line is drawn on the mean over K = 2..16 of ln(time back to back /
// time spaced), in percent, here under the default / nt / sc1 / sc1 nt policy
// with [the least, the most] of the cells:
//  16 bytes, round robin and blocked, from 12 waves per CU on over more than the
//             last-level cache keeps: 256 MiB, 12 waves +0.8 / +0.1 / +0.5 / +0.1
//             [-6 +7], 20 waves +1.0 / +0.1 / +0.8 / +0.8 [-7 +11]; 1 GiB, 12
//             waves +0.5 / 0.0 / +0.9 / +0.1 [-3 +4], 16 waves +0.5 / +0.2 / +0.6
//             / +0.2 [-5 +11]; 4 GiB, 16 waves +0.1 / 0.0 / +0.2 / -0.2 [-3 +8].
//             Not below: 1 GiB, 8 waves +0.6 / -0.1 / 0.0 / 0.0 [-8 +6], 4
//             waves -3.0 / -3.5 / -2.8 / -3.6 [-15 +8]; 64 MiB, 12 waves +0.5 /
//             -0.2 / +0.4 / -0.2 [-9 +5].
//  16 bytes, strided, under any policy but the default, from 12 waves on over
//             one XCD's 4 MiB L2: the loads of a group may all fall on one
//             segment and then miss together where spaced ones hit.  12 waves
//             +0.1 / +1.8 / +2.3 / +1.3 [-8 +17], 28 waves -0.2 / +2.4 / +1.8 /
//             +3.0 [-7 +13].  Not over 16 MiB, 20 waves -0.5 / -0.8 / +0.7 /
//             +0.2 [-16 +11], nor 160 MiB, 28 waves -2.6 / -2.8 / -2.6 / -2.3.
//  4, 8 bytes, strided, at 32 waves over 256 MiB and more: 8 bytes, 256 MiB
//             +2.5 / +1.3 / +2.7 / +1.3 [-2 +10], 4 GiB +2.7 / +4.4 / +3.0 / +4.1
//             [-7 +13]; 4 bytes, 1 GiB +3.1 / +2.8 / +0.3 / -0.3 [-8 +10].  Not
//             at 24 waves: 256 MiB, 8 bytes -1.5 / -1.7 / -1.5 / -1.8, 4 bytes
//             -0.1 / -1.5 / -2.2 / -2.2.
//  4, 8 bytes, other orders: never.  1 GiB, 8 bytes, 16 waves -0.1 / -1.1 / 0.0 /
//             -0.8 [-7 +10], 4 bytes, 8 waves -10.5 / -14.2 / -11.0 / -15.1.
// `resident` is the waves of the launch that a CU holds at a time.
bool spaced_form(int V, int policy, int order, uint64_t resident, uint64_t bytes) {
  if (order != SWEEP_ORDER_STRIDED)
    return V == 16 && resident >= 12 && bytes > (128ull << 20);
  if (V == 16)
    return policy != SWEEP_CACHE_DEFAULT && resident >= 12 && bytes <= (4ull << 20);
  return resident >= 32 && bytes >= (256ull << 20);
}

}  // namespace

const void* plain_kernel(int K, int V, int policy, int order, uint64_t resident,
                         uint64_t bytes) {
  const int vi = width_index(V);
  if (vi < 0 || K < 1 || K > kMaxK || policy < 0 || policy >= kNumPolicies) return nullptr;
  const bool spaced = spaced_form(V, policy, order, resident, bytes);
  const bool far = bytes >= kFarBytes;
  return reinterpret_cast<const void*>(table(vi, policy)[(2 * far + spaced) * kMaxK + K - 1]);
}

}  // namespace ilp
