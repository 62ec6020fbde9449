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

template <int V, int POL, int... Ks>
constexpr std::array<PlainFn, 4 * sizeof...(Ks)> row(std::integer_sequence<int, Ks...>) {
  return {&plain_kload<Ks + 1, V, POL>..., &plain_kload_spaced<Ks + 1, V, POL>...,
          &plain_kload_far<Ks + 1, V, POL>..., &plain_kload_far_spaced<Ks + 1, V, POL>...};
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

// Which form a cell takes.  K loads sent at once by many waves reach a
// saturated HBM as bursts that some strides fold onto few channels; a gap
// between loads spreads them, and costs what it delays elsewhere.  Measured
// over 1 GiB, sc1 nt, GB/s back to back -> spaced:
//  16 bytes   from 8 MiB in flight on, by 8 or more waves per CU or in groups
//             of 16 KiB, over a buffer that the 256 MiB last-level cache does
//             not hold: 16 waves, K = 8 6390 -> 6950, K = 16 5960 -> 6840; 32
//             waves, K = 8 6680 -> 6980; 4 waves, K = 16 6660 -> 6880; most
//             others within 1 %.  Not 4 waves, K = 4 6150 -> 5590, K = 12
//             6890 -> 6680; 64 MiB, 4 waves, K = 16 6840 -> 6260.  At 192 MiB
//             the two are level.
//  4, 8 bytes between 8 and 14 MiB in flight, 4 bytes from 16 waves per CU on,
//             8 from 8; 8 bytes, 16 waves, K = 6 6600 -> 7240, 28 waves, K = 3
//             6160 -> 6930; 4 bytes, 24 waves, K = 8 6120 -> 6890; over 64 to
//             128 MiB the same (28 waves, K = 3 5900 -> 6600).  Not above: 24
//             waves, K = 5 of 8 bytes (15 MiB) 7140 -> 6730, K = 10 of 4 over
//             20 MiB 6950 -> 6780; not below: 4 waves, K = 16 of 8 bytes (8
//             MiB) 7260 -> 6260; 12 waves, K = 12 of 4 bytes 6970 -> 6180.
//  strided, 16 bytes, past the L1: the loads of a group may all fall on one
//             segment of a buffer read more than once, and then miss together
//             where spaced ones hit: above 14 MiB in flight, and from 8 MiB on
//             over 64 MiB and more; 4 MiB, 8 waves, K = 8 16600 -> 19360, K =
//             16 17000 -> 21000; 16 MiB, 16 waves, K = 4 12120 -> 13780; 128
//             MiB, 4 waves, K = 8 5250 -> 5650.  Below, 4 MiB, 8 waves, K = 3
//             11020 -> 9750.
// Gaps of 4 and 8 cycles lift the same cells less.
bool spaced_form(int K, int V, int policy, int order, int waves_per_cu, uint64_t n_waves,
                 uint64_t bytes) {
  const uint64_t group = (uint64_t)K * kWave * V, in_flight = n_waves * group;
  if (V == 16 && order == SWEEP_ORDER_STRIDED && policy >= SWEEP_CACHE_BYPASS_L1 &&
      (in_flight > (14ull << 20) || (in_flight >= (8ull << 20) && bytes >= (64ull << 20))))
    return true;
  if (in_flight <= (8ull << 20)) return false;
  if (V == 16)
    return bytes > (128ull << 20) && (waves_per_cu >= 8 || group >= (16ull << 10));
  return in_flight <= (14ull << 20) && bytes >= (64ull << 20) && waves_per_cu * V >= 64;
}

}  // namespace

const void* plain_kernel(int K, int V, int policy, int order, int waves_per_cu,
                         uint64_t n_waves, uint64_t bytes) {
  const int vi = width_index(V);
  if (vi < 0 || K < 1 || K > kMaxK || policy < 0 || policy >= kNumPolicies) return nullptr;
  const bool spaced = spaced_form(K, V, policy, order, waves_per_cu, n_waves, bytes);
  const bool far = bytes >= kFarBytes;
  return reinterpret_cast<const void*>(table(vi, policy)[(2 * far + spaced) * kMaxK + K - 1]);
}

}  // namespace ilp
