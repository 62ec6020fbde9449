// LDS-ring kernels of the path comparison (Section 4.3) and the
// same-workgroup two-stream kernel (Section 4.4).
//
//  lds_async    loads go straight to LDS (global_load_lds_dwordx4, no
//               destination register), the analogue of cp.async;
//  lds_matched  the same ring through registers (global_load_dwordx4, then
//               ds_write_b128 and ds_read_b128), the matched plain kernel;
//  two_stream   one workgroup per CU whose first waves run the plain
//               batched K-load loop over the first half of the buffer and
//               whose last waves run either the LDS-direct ring or the
//               same plain loop over the second; or, split, half of the
//               workgroups run stream A and the other half stream B, so
//               the two streams share no CU.
// Each wave owns `depth` 1 KiB slots of the workgroup's dynamic LDS.
#include <array>
#include <utility>

#include "kernels.hpp"
#include "wave_loops.hpp"

namespace ilp {

extern __shared__ u32x4 lds_ring[];

template <int KIND, int D, int POL, template <int, int> class Walk>
__device__ __forceinline__ void lds_cell(const LdsArgs& a) {
  typedef Walk<16, POL> W;
  const uint64_t t0 = wall_ticks();
  const uint32_t lane = lane_id();
  const uint32_t wv = wave_in_wg();
  const uint32_t wid = blockIdx.x * a.waves + wv;
  const Share sh{a.buf, a.bytes, a.stride, wid, a.iters + (wid < a.extra ? 1u : 0u)};
  u32x4* ring = lds_ring + wv * (D * kWave);
  uint32_t s = 0, x = 0;
  if constexpr (KIND == SWEEP_KIND_LDS_ASYNC) {
    async_ring_loop<D, POL, W>(sh, lane, ring, s, x);
  } else {
    matched_ring_loop<D, W>(sh, lane, ring, s, x);
  }
  const uint64_t t1 = wall_ticks();
  wave_epilogue(s, x, t0, t1, wid, a.rec, a.lane_out);
}

template <int KIND, int D, int POL>
__global__ __launch_bounds__(1024) void lds_kernel_t(LdsArgs a) {
  lds_cell<KIND, D, POL, NearWalk>(a);
}
template <int KIND, int D, int POL>
__global__ __launch_bounds__(1024) void lds_kernel_far(LdsArgs a) {
  lds_cell<KIND, D, POL, FarWalk>(a);
}

__device__ __forceinline__ Share share_of(const StreamArgs& a, uint32_t wid) {
  return Share{a.buf, a.bytes, a.stride, wid, a.iters + (wid < a.extra ? 1u : 0u)};
}

// Stream B of a two-stream launch: the LDS-direct ring or the plain loop.
template <int D, int POL, class W>
__device__ __forceinline__ void stream_b(const TwoStreamArgs& a, uint32_t wid, uint32_t wb,
                                         uint32_t lane, uint32_t& s, uint32_t& x) {
  const Share sh = share_of(a.b, wid);
  if (a.b_plain) {
    plain_loop16<D, W>(sh, lane, s, x);
  } else {
    u32x4* ring = lds_ring + wb * (D * kWave);
    async_ring_loop<D, POL, W>(sh, lane, ring, s, x);
  }
}

template <int D, int POL, template <int, int> class Walk>
__device__ __forceinline__ void two_streams(const TwoStreamArgs& a) {
  typedef Walk<16, POL> W;
  const uint64_t t0 = wall_ticks();
  const uint32_t lane = lane_id();
  const uint32_t wv = wave_in_wg();
  // Split: workgroups 16m .. 16m+7 run stream A and 16m+8 .. 16m+15 stream B
  // (the grid is a multiple of 16).  Workgroups are dealt to the 8 XCDs
  // in turn, so every XCD holds as many workgroups of A as of B; with one
  // workgroup per CU no CU runs both.  Waves beyond the stream's count
  // leave at once and write no record.  Otherwise a workgroup's first
  // waves_a waves run A and the rest B.
  const uint32_t g = blockIdx.x;
  bool is_a;
  uint32_t idx, wi, n_wg;      // workgroup among its stream's, wave in it, their number
  if (a.split) {
    is_a = ((g >> 3) & 1u) == 0;
    idx = (g >> 4) * 8u + (g & 7u);
    wi = wv;
    n_wg = gridDim.x / 2;
    if (wv >= (is_a ? a.waves_a : a.waves_b)) return;
  } else {
    is_a = wv < a.waves_a;
    idx = g;
    wi = is_a ? wv : wv - a.waves_a;
    n_wg = gridDim.x;
  }
  uint32_t s = 0, x = 0, out;
  if (is_a) {
    out = idx * a.waves_a + wi;
    plain_loop16<D, W>(share_of(a.a, out), lane, s, x);
  } else {
    const uint32_t wid = idx * a.waves_b + wi;
    stream_b<D, POL, W>(a, wid, wi, lane, s, x);
    out = n_wg * a.waves_a + wid;
  }
  const uint64_t t1 = wall_ticks();
  wave_epilogue(s, x, t0, t1, out, a.rec, a.lane_out);
}

template <int D, int POL>
__global__ __launch_bounds__(1024) void two_stream_t(TwoStreamArgs a) {
  two_streams<D, POL, NearWalk>(a);
}
template <int D, int POL>
__global__ __launch_bounds__(1024) void two_stream_far(TwoStreamArgs a) {
  two_streams<D, POL, FarWalk>(a);
}

namespace {

typedef void (*LdsFn)(LdsArgs);
typedef void (*TwoFn)(TwoStreamArgs);

template <int KIND, int POL, int... Ds>
constexpr std::array<LdsFn, 2 * sizeof...(Ds)> lds_row(std::integer_sequence<int, Ds...>) {
  return {&lds_kernel_t<KIND, Ds + 1, POL>..., &lds_kernel_far<KIND, Ds + 1, POL>...};
}
template <int POL, int... Ds>
constexpr std::array<TwoFn, 2 * sizeof...(Ds)> two_row(std::integer_sequence<int, Ds...>) {
  return {&two_stream_t<Ds + 1, POL>..., &two_stream_far<Ds + 1, POL>...};
}
template <int KIND, int POL>
constexpr auto kLdsRow = lds_row<KIND, POL>(std::make_integer_sequence<int, kMaxK>{});
template <int POL>
constexpr auto kTwoRow = two_row<POL>(std::make_integer_sequence<int, kMaxK>{});

}  // namespace

const void* lds_kernel(int kind, int D, int policy, bool far) {
  static const std::array<LdsFn, 2 * kMaxK> t[2][kNumPolicies] = {
      {kLdsRow<SWEEP_KIND_LDS_ASYNC, 0>, kLdsRow<SWEEP_KIND_LDS_ASYNC, 1>,
       kLdsRow<SWEEP_KIND_LDS_ASYNC, 2>, kLdsRow<SWEEP_KIND_LDS_ASYNC, 3>},
      {kLdsRow<SWEEP_KIND_LDS_MATCHED, 0>, kLdsRow<SWEEP_KIND_LDS_MATCHED, 1>,
       kLdsRow<SWEEP_KIND_LDS_MATCHED, 2>, kLdsRow<SWEEP_KIND_LDS_MATCHED, 3>},
  };
  if (D < 1 || D > kMaxK || policy < 0 || policy >= kNumPolicies) return nullptr;
  const int i = (far ? kMaxK : 0) + D - 1;
  if (kind == SWEEP_KIND_LDS_ASYNC) return reinterpret_cast<const void*>(t[0][policy][i]);
  if (kind == SWEEP_KIND_LDS_MATCHED) return reinterpret_cast<const void*>(t[1][policy][i]);
  return nullptr;
}

const void* two_stream_kernel(int D, int policy, bool far) {
  static const std::array<TwoFn, 2 * kMaxK> t[kNumPolicies] = {kTwoRow<0>, kTwoRow<1>,
                                                           kTwoRow<2>, kTwoRow<3>};
  if (D < 1 || D > kMaxK || policy < 0 || policy >= kNumPolicies) return nullptr;
  return reinterpret_cast<const void*>(t[policy][(far ? kMaxK : 0) + D - 1]);
}

}  // namespace ilp
