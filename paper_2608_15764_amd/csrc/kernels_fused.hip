// Fused batch of plain K-load cells (the batched sweep): the points of one
// tuned configuration run as a single persistent launch over their
// concatenated wave-groups, so a small point costs a few groups of the
// running grid instead of a launch of its own.  The loop is the plain
// kernel's: K independent loads issued before the first is consumed, then
// folded oldest first, nothing from the next group in flight, no stores
// inside the loop.  A wave closes a point's record (DPP reduction, one
// store) when its next group belongs to another point, or at the end.
#include <array>
#include <utility>

#include "device.hpp"
#include "kernels.hpp"
#include "seg_walk.hpp"

namespace ilp {

// The point list is read at a wave-uniform index; readfirstlane makes the
// fields scalars, so the buffer descriptors built from them stay scalar.
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// A point's buffer is addressed from the launch's base pointer (a kernel
// argument, so loads through it stay global loads).
struct PointRegs {
  const uint8_t* buf;
  uint64_t bytes, g0, end, stride;
};

// The point list is never written while the kernel runs: read it through
// the constant address space, so the loads are scalar and stay out of the
// vector-memory counter the K loads of a group wait on.
typedef const __attribute__((address_space(4))) FusedPoint* ConstPoints;

__device__ __forceinline__ PointRegs point_regs(const uint8_t* base, const FusedPoint* pts,
                                                uint32_t i) {
  const auto& f = reinterpret_cast<ConstPoints>(reinterpret_cast<uintptr_t>(pts))[i];
  PointRegs r;
  r.buf = base + uniform64(f.off);
  r.bytes = uniform64(f.bytes);
  r.g0 = uniform64(f.g0);
  r.end = r.g0 + uniform64(f.Q);
  r.stride = uniform64(f.stride);
  return r;
}

// Two forms of the loop.  This one steps and wraps a 64-bit offset between two
// loads, which spaces the loads of a group by some 60 clocks; the other one
// below issues them back to back.  Where the batch offers more bytes than HBM
// keeps in flight anyway, spaced loads read 1-2 % faster: 64 points of 1 MiB
// to 2 GiB, 17.5 GiB, K = 8 at 4 waves per CU (8 MiB offered) 2598 against
// 2645 us with nt loads, 2620 against 2642 with sc1 nt; K = 4 at 16 (16 MiB)
// 880 against 895 us for 5.5 GiB.  Below that back to back is faster: K = 3 of
// 8 bytes at 8 waves (3 MiB), 24 points of 4 to 16 MiB, 69 against 64 us; K =
// 3 of 16 bytes at 8 waves (6 MiB) 2680 against 2640 us for the 17.5 GiB.  (The
// choice depends on K, as a plain cell's must not: neighbouring points share
// the launch, so their windows are no K curve.)
template <int K, int V, int POL>
__global__ __launch_bounds__(kPlainWgThreads) void fused_kload(FusedArgs a) {
  const uint32_t lane = lane_id();
  const uint32_t wid = blockIdx.x * (kPlainWgThreads / kWave) + wave_in_wg();
  const uint32_t n_waves = gridDim.x * (kPlainWgThreads / kWave);

  // the wave's current point, cached in scalars (wave-uniform)
  uint32_t pi = 0;
  PointRegs pt = point_regs(a.base, a.pts, 0);
  uint64_t p = 0;               // start of the wave's next group, in bytes
  bool open = false;            // the wave has read a group of point pi
  uint32_t s = 0, x = 0;
  uint64_t t0 = 0;
#pragma unroll 1
  for (uint64_t g = wid; g < a.total_groups; g += n_waves) {
    if (g >= pt.end) {
      if (open) wave_epilogue(s, x, t0, wall_ticks(), pi * n_waves + wid, a.rec, nullptr);
      open = false;
      do {
        ++pi;
        pt = point_regs(a.base, a.pts, pi);
      } while (g >= pt.end);
    }
    if (!open) {
      open = true;
      s = 0;
      x = 0;
      t0 = wall_ticks();
      p = ((g - pt.g0) * (uint64_t)(K * kWave * V)) % pt.bytes;
    }
    typename Vec<V>::T v[K];
    uint64_t pj = p;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      v[j] = load_seg<V, POL>(pt.buf + pj, lane);
      pj += kWave * V;
      if (pj >= pt.bytes) pj -= pt.bytes;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < K; ++j) fold(v[j], s, x);
    p += pt.stride;
    if (p >= pt.bytes) p -= pt.bytes;
  }
  if (open) wave_epilogue(s, x, t0, wall_ticks(), pi * n_waves + wid, a.rec, nullptr);
}

template <int K, int V, int POL>
__global__ __launch_bounds__(kPlainWgThreads) void fused_kload_ahead(FusedArgs a) {
  typedef NearWalk<V, POL> W;       // its points are below kFarBytes each
  const uint32_t lane = lane_id();
  const uint32_t wid = blockIdx.x * (kPlainWgThreads / kWave) + wave_in_wg();
  const uint32_t n_waves = gridDim.x * (kPlainWgThreads / kWave);
  const ConstPoints pts = reinterpret_cast<ConstPoints>(reinterpret_cast<uintptr_t>(a.pts));

  uint64_t g = wid;                 // the wave's next group
  for (uint32_t pi = 0; g < a.total_groups; ++pi) {
    // the point, in scalars, addressed from the launch's base pointer (a
    // kernel argument, so loads through it stay global loads)
    const auto& f = pts[pi];
    const uint64_t bytes = uniform64(f.bytes), g0 = uniform64(f.g0);
    const uint64_t end = g0 + uniform64(f.Q);
    if (g >= end) continue;
    const uint64_t t0 = wall_ticks();
    const W walk(a.base + uniform64(f.off), bytes, lane);
    constexpr uint64_t seg = kWave * V;
    const typename W::Step next_load = walk.step(bytes > seg ? seg : 0, bytes);
    const typename W::Step next_group = walk.step(uniform64(f.stride), bytes);
    uint64_t off = (g - g0) * (K * seg);
    if (off >= bytes) off %= bytes;
    typename W::Cursor p = walk.at(off);
    typename W::Start at[K];        // of the next group, found while one is in flight
    auto place = [&] {
      typename W::Cursor pj = p;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        at[j] = walk.start(pj);
        pj = next_load(pj);
      }
    };
    place();
    uint32_t s = 0, x = 0;
#pragma unroll 1
    do {
      typename Vec<V>::T v[K];
      const uint32_t lo = walk.lane_offset();
#pragma unroll
      for (int j = 0; j < K; ++j) v[j] = walk.load(at[j], lo);
      __builtin_amdgcn_sched_barrier(0);
      p = next_group(p);
      place();
      g += n_waves;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < K; ++j) fold(v[j], s, x);
    } while (g < end);
    wave_epilogue(s, x, t0, wall_ticks(), pi * n_waves + wid, a.rec, nullptr);
  }
}

__global__ __launch_bounds__(256) void clear_records(sweep_wave_rec_t* rec, uint64_t n) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    u32x4* r = reinterpret_cast<u32x4*>(rec + i);
    r[0] = u32x4{0u, 0u, 0u, 0u};
    r[1] = u32x4{0xFFFFFFFFu, 0xFFFFFFFFu, 0u, 0u};
  }
}

hipError_t launch_clear_records(sweep_wave_rec_t* rec, uint64_t n, hipStream_t st) {
  uint64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(clear_records, dim3((uint32_t)blocks), dim3(256), 0, st, rec, n);
  return hipGetLastError();
}

namespace {

// Bytes in flight, of the waves that run at a time, up to which a group's loads
// go out back to back.
constexpr uint64_t kAheadBytes = 6ull << 20;

typedef void (*FusedFn)(FusedArgs);

template <int V, int POL, int... Ks>
constexpr std::array<FusedFn, 2 * sizeof...(Ks)> row(std::integer_sequence<int, Ks...>) {
  return {&fused_kload<Ks + 1, V, POL>..., &fused_kload_ahead<Ks + 1, V, POL>...};
}

template <int V, int POL>
constexpr auto kRow = row<V, POL>(std::make_integer_sequence<int, kMaxK>{});

// [vector width index][policy][ahead * kMaxK + K-1]
const FusedFn* table(int vi, int pol) {
  static const std::array<FusedFn, 2 * kMaxK> t[3][kNumPolicies] = {
      {kRow<4, 0>, kRow<4, 1>, kRow<4, 2>, kRow<4, 3>},
      {kRow<8, 0>, kRow<8, 1>, kRow<8, 2>, kRow<8, 3>},
      {kRow<16, 0>, kRow<16, 1>, kRow<16, 2>, kRow<16, 3>},
  };
  return t[vi][pol].data();
}

int width_index(int V) { return V == 4 ? 0 : V == 8 ? 1 : V == 16 ? 2 : -1; }

}  // namespace

const void* fused_kernel(int K, int V, int policy, uint64_t n_waves, bool far) {
  const int vi = width_index(V);
  if (vi < 0 || K < 1 || K > kMaxK || policy < 0 || policy >= kNumPolicies) return nullptr;
  const bool ahead = !far && n_waves * (uint64_t)(K * kWave * V) <= kAheadBytes;
  return reinterpret_cast<const void*>(table(vi, policy)[(ahead ? kMaxK : 0) + K - 1]);
}

}  // namespace ilp
