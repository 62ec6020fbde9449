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

template <int K, int V, int POL, template <int, int> class Walk>
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
    // Where the K loads of a group start is worked out while the group
    // before it is in flight, so that they are issued back to back: found
    // between them, K = 2 / 4 / 8 / 14 loads of 4 bytes over 1 GiB at 4 waves
    // per CU (sc1 nt) took 891 / 520 / 322 / 228 us, and take 864 / 463 /
    // 275 / 192.  Cells that HBM bounds do not change.
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
    place();
#pragma unroll 1
    for (; iters; --iters) {
      typename Vec<V>::T v[K];
      const uint32_t lo = walk.lane_offset();
#pragma unroll
      for (int j = 0; j < K; ++j) v[j] = walk.load(at[j], lo);
      __builtin_amdgcn_sched_barrier(0);
      p = next_group(p);
      place();
      // all K loads are issued before the first is consumed: without this
      // barrier the scheduler may refill registers early to raise occupancy
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
  plain_cell<K, V, POL, NearWalk>(a);
}

// The same cell over 4 GiB and more.
template <int K, int V, int POL>
__global__ __launch_bounds__(kPlainWgThreads) void plain_kload_far(PlainArgs a) {
  plain_cell<K, V, POL, FarWalk>(a);
}

namespace {

typedef void (*PlainFn)(PlainArgs);

template <int V, int POL, int... Ks>
constexpr std::array<PlainFn, 2 * sizeof...(Ks)> row(std::integer_sequence<int, Ks...>) {
  return {&plain_kload<Ks + 1, V, POL>..., &plain_kload_far<Ks + 1, V, POL>...};
}

template <int V, int POL>
constexpr auto kRow = row<V, POL>(std::make_integer_sequence<int, kMaxK>{});

// [vector width index][policy][far * kMaxK + K-1]
const PlainFn* table(int vi, int pol) {
  static const std::array<PlainFn, 2 * kMaxK> t[3][kNumPolicies] = {
      {kRow<4, 0>, kRow<4, 1>, kRow<4, 2>, kRow<4, 3>},
      {kRow<8, 0>, kRow<8, 1>, kRow<8, 2>, kRow<8, 3>},
      {kRow<16, 0>, kRow<16, 1>, kRow<16, 2>, kRow<16, 3>},
  };
  return t[vi][pol].data();
}

int width_index(int V) { return V == 4 ? 0 : V == 8 ? 1 : V == 16 ? 2 : -1; }

}  // namespace

const void* plain_kernel(int K, int V, int policy, bool far) {
  const int vi = width_index(V);
  if (vi < 0 || K < 1 || K > kMaxK || policy < 0 || policy >= kNumPolicies) return nullptr;
  return reinterpret_cast<const void*>(table(vi, policy)[(far ? kMaxK : 0) + K - 1]);
}

}  // namespace ilp
