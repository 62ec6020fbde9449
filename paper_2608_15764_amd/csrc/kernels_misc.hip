// Buffer fill, per-cell finishing, clock probe and the precision variant's
// streaming FP reduction.
#include <hip/hip_ext.h>

#include "device.hpp"
#include "kernels.hpp"

namespace ilp {

// ------------------------------------------------------------------ fill
// Word i of the buffer is the low half of SplitMix64 output i for state
// `seed`: z = seed + (i+1)*gamma, then the SplitMix64 finaliser
// (Steele, Lea and Flood, 2014), which is splitmix_mix.
constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;

__device__ __forceinline__ uint32_t splitmix_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (uint32_t)z;
}

// One wave writes one chunk of kFillVecs * 64 adjacent 16-byte vectors
// (4 KiB) and leaves; the grid is as large as the buffer.  Bound by HBM
// writes.  8192 workgroups striding through the buffer keep as many write
// fronts open, 32 MiB apart, and took 248 us for 1 GiB (4.3 TB/s);
// dispatched in order, the chip writes one moving front, 184 us (5.8 TB/s;
// 4 MiB to 128 MiB unchanged).  The arithmetic (two 64-bit products per
// word, about 7.5 TB/s by itself) overlaps the stores but for a few percent:
// constant stores in the same shape reach 6.1-6.9 TB/s.  Chunks of 1 to 32
// KiB in workgroups of 64 to 1024 threads are within 5 % of each other.
constexpr int kFillVecs = 4;
constexpr uint64_t kFillChunk = kFillVecs * kWave;   // vectors per wave
constexpr uint64_t kFillMaxGrid = 1u << 24;          // 64 GiB at once, then strides

__global__ __launch_bounds__(kWave) void fill_u32(uint32_t* buf, uint64_t n_words,
                                                  uint64_t seed) {
  const uint64_t n4 = n_words / 4;
  const uint32_t t = threadIdx.x;
  u32x4* b4 = reinterpret_cast<u32x4*>(buf);
  const uint64_t n_chunks = (n_words + 4 * kFillChunk - 1) / (4 * kFillChunk);
  for (uint64_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
    const uint64_t v0 = c * kFillChunk;
    // state of the chunk's word 0, then of this lane's first vector
    const uint64_t z = seed + (v0 * 4 + 1) * kGamma + (uint64_t)(t * 4) * kGamma;
    auto vec = [&](int u) {
      const uint64_t zu = z + (uint64_t)(u * 4 * kWave) * kGamma;
      return u32x4{splitmix_mix(zu), splitmix_mix(zu + kGamma), splitmix_mix(zu + 2 * kGamma),
                   splitmix_mix(zu + 3 * kGamma)};
    };
    if (v0 + kFillChunk <= n4) {
#pragma unroll
      for (int u = 0; u < kFillVecs; ++u) b4[v0 + u * kWave + t] = vec(u);
    } else {
#pragma unroll 1
      for (int u = 0; u < kFillVecs; ++u) {
        const uint64_t v = v0 + u * kWave + t;
        const u32x4 r = vec(u);
        if (v < n4) {
          b4[v] = r;
        } else if (v == n4) {       // the last one to three words
          const uint32_t w[3] = {r.x, r.y, r.z};
#pragma unroll
          for (int k = 0; k < 3; ++k)
            if (n4 * 4 + k < n_words) buf[n4 * 4 + k] = w[k];
        }
      }
    }
  }
}

hipError_t launch_fill(uint32_t* buf, uint64_t n_words, uint64_t seed,
                       hipStream_t st) {
  const uint64_t chunks = (n_words + 4 * kFillChunk - 1) / (4 * kFillChunk);
  const uint32_t blocks = (uint32_t)(chunks < kFillMaxGrid ? chunks : kFillMaxGrid);
  hipLaunchKernelGGL(fill_u32, dim3(blocks), dim3(kWave), 0, st, buf, n_words, seed);
  return hipGetLastError();
}

// ---------------------------------------------------------------- finish
// Workgroup c folds the wave records of cell c, rec[offsets[c] ..
// offsets[c+1]), into the cell's global sinks and its clock window
// [min t0, max t1].
//
// One call waits for this kernel, so it is latency bound: a launch, a read
// of 256 KiB at most per cell (8192 waves) by one CU, a reduction.  256
// threads reading one record at a time made 32 dependent round trips of it
// and an LDS tree of eight barriers; 1024 threads with four records each in
// flight make two, and DPP steps replace the tree.  8192 records: 13.3 ->
// 4.7 us.  The result goes to `out`, which the host-visible callers place
// in pinned memory, so that no copy follows.
constexpr int kFinishThreads = 1024;
constexpr int kFinishBatch = 4;       // records in flight per thread

template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
  return ((uint64_t)dpp<CTRL>((uint32_t)(v >> 32)) << 32) | dpp<CTRL>((uint32_t)v);
}
__device__ __forceinline__ uint64_t readlane64(uint64_t v, int l) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(v >> 32), l) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((uint32_t)v, l);
}
template <class Op>
__device__ __forceinline__ uint64_t wave_fold64(uint64_t v, Op op) {
  v = op(v, dpp64<kDppQuadSwap1>(v));
  v = op(v, dpp64<kDppQuadSwap2>(v));
  v = op(v, dpp64<kDppRowRor4>(v));
  v = op(v, dpp64<kDppRowRor8>(v));
  return op(op(readlane64(v, 0), readlane64(v, 16)), op(readlane64(v, 32), readlane64(v, 48)));
}

// The sinks and the window of a set of records.
struct Window {
  uint32_t s, x;
  uint64_t lo, hi;
};
__device__ __forceinline__ Window no_records() { return Window{0u, 0u, ~0ull, 0ull}; }
__device__ __forceinline__ Window wave_window(Window w) {
  w.s = wave_sum_u32(w.s);
  w.x = wave_xor_u32(w.x);
  w.lo = wave_fold64(w.lo, [](uint64_t p, uint64_t q) { return q < p ? q : p; });
  w.hi = wave_fold64(w.hi, [](uint64_t p, uint64_t q) { return q > p ? q : p; });
  return w;
}

// Folds records [i0, i1) over a workgroup of kFinishThreads threads; thread
// 0 stores the result.  look(i, v, t) sees every record, as its two halves.
template <class Look>
__device__ __forceinline__ void fold_records(const sweep_wave_rec_t* rec, uint64_t i0,
                                             uint64_t i1, CellRes* out, Look look) {
  __shared__ Window part[kFinishThreads / kWave];
  Window w = no_records();
  const u32x4* r = reinterpret_cast<const u32x4*>(rec);
  for (uint64_t b = i0; b < i1; b += kFinishBatch * kFinishThreads) {
    u32x4 v[kFinishBatch], t[kFinishBatch];
    const uint64_t i = b + threadIdx.x;
#pragma unroll
    for (int u = 0; u < kFinishBatch; ++u) {
      uint64_t k = i + u * kFinishThreads;
      k = k < i1 ? k : i1 - 1;          // loads past the end re-read the last record
      v[u] = r[2 * k];
      t[u] = r[2 * k + 1];
    }
#pragma unroll
    for (int u = 0; u < kFinishBatch; ++u) {
      if (i + u * kFinishThreads < i1) {
        w.s += v[u].x;
        w.x ^= v[u].y;
        const uint64_t t0 = ((uint64_t)t[u].y << 32) | t[u].x;
        const uint64_t t1 = ((uint64_t)t[u].w << 32) | t[u].z;
        w.lo = t0 < w.lo ? t0 : w.lo;
        w.hi = t1 > w.hi ? t1 : w.hi;
        look(i + u * kFinishThreads, v[u], t[u]);
      }
    }
  }
  w = wave_window(w);
  const uint32_t lane = lane_id();
  if (lane == 0) part[threadIdx.x / kWave] = w;
  __syncthreads();
  if (threadIdx.x < kWave) {
    w = lane < kFinishThreads / kWave ? part[lane] : no_records();
    w = wave_window(w);
    if (lane == 0) {
      u32x4* o = reinterpret_cast<u32x4*>(out);
      o[0] = u32x4{w.s, 0u, w.x, 0u};
      o[1] = u32x4{(uint32_t)w.lo, (uint32_t)(w.lo >> 32), (uint32_t)w.hi,
                   (uint32_t)(w.hi >> 32)};
    }
  }
}

struct LookAway {
  __device__ __forceinline__ void operator()(uint64_t, u32x4, u32x4) const {}
};

__global__ __launch_bounds__(kFinishThreads) void finish_cells(FinishArgs a) {
  const uint32_t c = blockIdx.x;
  uint64_t i0, i1;
  if (a.offsets) {
    i0 = a.offsets[c];
    i1 = a.offsets[c + 1];
  } else {
    i0 = a.few[c];
    i1 = a.few[c + 1];
  }
  fold_records(a.rec, i0, i1, a.out + c, LookAway());
}

hipError_t launch_finish_cells(const FinishArgs& a, uint32_t n_cells, hipStream_t st) {
  hipLaunchKernelGGL(finish_cells, dim3(n_cells), dim3(kFinishThreads), 0, st, a);
  return hipGetLastError();
}

// One XCD read: the fold, and the first record that is missing (a cleared
// one has t1 = 0) or not from the XCD its number names.  Fetching up to 256 KiB
// of records to check them on the host took 10 to 29 us of a call: 64 MiB by
// six XCDs at 8 waves per CU 62 -> 32 us, 1 GiB by all of them at 16 199 ->
// 180 us.
__global__ __launch_bounds__(kFinishThreads) void finish_xcd(XcdFinishArgs a) {
  __shared__ uint64_t first[kFinishThreads / kWave];
  uint64_t bad = ~0ull;
  fold_records(a.rec, 0, a.n_rec, a.out, [&](uint64_t i, u32x4 v, u32x4 t) {
    const uint32_t slot = ((uint32_t)i / a.run) % a.n_xcds;
    const uint32_t want = (a.xcds >> (4 * slot)) & 0xFu;
    if ((t.z | t.w) == 0u || (v.w & 0xFu) != want) bad = i < bad ? i : bad;
  });
  const auto less = [](uint64_t p, uint64_t q) { return q < p ? q : p; };
  bad = wave_fold64(bad, less);
  const uint32_t lane = lane_id();
  if (lane == 0) first[threadIdx.x / kWave] = bad;
  __syncthreads();
  if (threadIdx.x < kWave) {
    bad = wave_fold64(lane < kFinishThreads / kWave ? first[lane] : ~0ull, less);
    if (lane == 0) a.first_bad[0] = bad;
  }
}

hipError_t launch_finish_xcd(const XcdFinishArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(finish_xcd, dim3(1), dim3(kFinishThreads), 0, st, a);
  return hipGetLastError();
}

// ----------------------------------------------------------------- clock
__global__ void read_clock(uint64_t* out) {
  if (threadIdx.x == 0) out[0] = wall_ticks();
}

hipError_t launch_read_clock(uint64_t* out, hipStream_t st) {
  hipLaunchKernelGGL(read_clock, dim3(1), dim3(64), 0, st, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ gate
// Tickets count up and wrap: one that has been passed stays passed, also where
// a later call's flag is already up when this wave starts.  Every wait ends
// after a.ticks of the clock.
__global__ void gate(GateArgs a) {
  const uint64_t t0 = wall_ticks();
  while ((int32_t)(__hip_atomic_load(a.flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) -
                   a.ticket) < 0 &&
         wall_ticks() - t0 < a.ticks) {
  }
}

hipError_t launch_gate(const GateArgs& a, hipStream_t st, hipEvent_t done) {
  void* args[] = {const_cast<GateArgs*>(&a)};
  return hipExtLaunchKernel(reinterpret_cast<const void*>(&gate), dim3(1), dim3(1), args, 0, st,
                            nullptr, done, 0);
}

// --------------------------------------------------- precision reduction
// Sum2 (Ogita, Rump and Oishi, 2005) per lane: TwoSum (Knuth) is
// error-free, s' + e = s + x exactly; the errors e are summed plainly in c.
struct Pair {
  float s, c;
};

__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e) {
  s = a + b;
  const float bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

__device__ __forceinline__ void add_term(Pair& p, float x) {
  float s, e;
  two_sum(p.s, x, s, e);
  p.s = s;
  p.c += e;
}

// Merge two pairs: TwoSum of the leading parts, the rest summed plainly.
__device__ __forceinline__ Pair merge(Pair a, Pair b) {
  Pair r;
  float e;
  two_sum(a.s, b.s, r.s, e);
  r.c = (a.c + b.c) + e;
  return r;
}

__device__ __forceinline__ float f32_of(uint32_t w) { return __uint_as_float(w); }

// Decode-and-accumulate of one 16-byte vector.
template <int DT>
__device__ __forceinline__ void acc_vec(Pair& p, u32x4 v);

template <>
__device__ __forceinline__ void acc_vec<SWEEP_F32>(Pair& p, u32x4 v) {
  add_term(p, f32_of(v.x));
  add_term(p, f32_of(v.y));
  add_term(p, f32_of(v.z));
  add_term(p, f32_of(v.w));
}

template <>
__device__ __forceinline__ void acc_vec<SWEEP_BF16>(Pair& p, u32x4 v) {
  // element 2k is the low half of word k (little endian)
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    add_term(p, f32_of(w[k] << 16));
    add_term(p, f32_of(w[k] & 0xFFFF0000u));
  }
}

// Plain FP32 sum of the 16 FP8 values of a vector (exact, see below).
__device__ __forceinline__ float fp8_vec_sum(u32x4 v) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  float t = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8(w[k], false);  // bytes 0, 1
    const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8(w[k], true);   // bytes 2, 3
    t += lo[0];
    t += lo[1];
    t += hi[0];
    t += hi[1];
  }
  return t;
}

template <>
__device__ __forceinline__ void acc_vec<SWEEP_FP8_E4M3>(Pair& p, u32x4 v) {
  add_term(p, fp8_vec_sum(v));
}

// Elements per 16-byte vector and bytes per element.
template <int DT> constexpr int elem_bytes() { return DT == SWEEP_F32 ? 4 : DT == SWEEP_BF16 ? 2 : 1; }

template <int DT>
__device__ __forceinline__ float decode_one(const uint8_t* p) {
  if constexpr (DT == SWEEP_F32) {
    uint32_t w = p[0] | (p[1] << 8) | (p[2] << 16) | ((uint32_t)p[3] << 24);
    return f32_of(w);
  } else if constexpr (DT == SWEEP_BF16) {
    uint32_t w = (p[0] | (p[1] << 8)) << 16;
    return f32_of(w);
  } else {
    return __builtin_amdgcn_cvt_pk_f32_fp8((uint32_t)p[0], false)[0];
  }
}

// Accumulates vector j (0, 1, ... in order) of a group.  64 e4m3 values are
// k * 2^-9 with |k| <= 64 * 229376 < 2^24, so their FP32 sum is exact; one
// TwoSum per 64 values (four vectors, whose sum so far is t).
template <int DT>
__device__ __forceinline__ void acc_one(Pair& p, float& t, const u32x4& v, int j) {
  if constexpr (DT == SWEEP_FP8_E4M3) {
    t = (j % 4 ? t : 0.0f) + fp8_vec_sum(v);
    if (j % 4 == 3) add_term(p, t);
  } else {
    acc_vec<DT>(p, v);
  }
}

// A wave-group is NL x 64 lanes x 16 bytes.  AT of its NL loads are asked for
// at a time and added up before the next AT; with AT = 0 a ring instead: a
// vector's place is loaded again as soon as it has been added, so that NL loads
// stay in flight through the arithmetic.  The additions and their order are
// the same for every AT.
template <int DT, int NL, int AT>
__device__ __forceinline__ void reduce_body(const ReduceArgs& a) {
  static_assert(NL % 4 == 0, "FP8 groups of four vectors are summed exactly");
  const uint64_t t0 = wall_ticks();
  const uint32_t lane = lane_id();
  const uint32_t wv = wave_in_wg();
  const uint32_t wid = blockIdx.x * 4 + wv;
  const uint32_t n_waves = gridDim.x * 4;
  Pair p{0.0f, 0.0f};

  const auto load = [&](uint64_t g, int j) {
    return load_seg<16, SWEEP_CACHE_NT>(a.payload + g * (NL * kWave * 16) + j * (kWave * 16),
                                        lane);
  };
  float t = 0.0f;
  if constexpr (AT == 0) {
    if (wid < a.n_groups) {
      u32x4 v[NL];
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        v[j] = load(wid, j);
        __builtin_amdgcn_sched_barrier(0);   // in the order they are waited for
      }
#pragma unroll 1
      for (uint64_t g = (uint64_t)wid + n_waves; g < a.n_groups; g += n_waves) {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          acc_one<DT>(p, t, v[j], j);
          __builtin_amdgcn_sched_barrier(0);
          v[j] = load(g, j);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int j = 0; j < NL; ++j) acc_one<DT>(p, t, v[j], j);
    }
  } else {
    // full wave-groups; AT loads are issued before any is consumed
#pragma unroll 1
    for (uint64_t g = wid; g < a.n_groups; g += n_waves) {
#pragma unroll
      for (int j = 0; j < NL; j += AT) {
        u32x4 v[AT];
#pragma unroll
        for (int k = 0; k < AT; ++k) v[k] = load(g, j + k);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < AT; ++k) acc_one<DT>(p, t, v[k], j + k);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // remaining whole vectors, one per thread of the grid
  const uint64_t gtid = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  const uint64_t first_rem = a.n_groups * (NL * kWave);
  if (first_rem + gtid < a.n_vec) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(a.payload + (first_rem + gtid) * 16);
    acc_vec<DT>(p, v);
  }
  // trailing bytes that do not fill a vector
  if (gtid == 0) {
    for (uint64_t off = a.n_vec * 16; off + elem_bytes<DT>() <= a.n_bytes;
         off += elem_bytes<DT>())
      add_term(p, decode_one<DT>(a.payload + off));
  }

  // wave merge: rotations within 16-lane rows, then the four rows in order
  auto xchg = [](Pair q, auto ctrl) {
    Pair o;
    o.s = __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(q.s), decltype(ctrl)::value, 0xF, 0xF, false));
    o.c = __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(q.c), decltype(ctrl)::value, 0xF, 0xF, false));
    return o;
  };
  p = merge(p, xchg(p, std::integral_constant<int, kDppQuadSwap1>{}));
  p = merge(p, xchg(p, std::integral_constant<int, kDppQuadSwap2>{}));
  p = merge(p, xchg(p, std::integral_constant<int, kDppRowRor4>{}));
  p = merge(p, xchg(p, std::integral_constant<int, kDppRowRor8>{}));
  Pair r[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    r[k].s = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(p.s), 16 * k));
    r[k].c = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(p.c), 16 * k));
  }
  const Pair wsum = merge(merge(r[0], r[1]), merge(r[2], r[3]));

  __shared__ Pair wg[4];
  if (lane == 0) wg[wv] = wsum;
  const uint64_t t1 = wall_ticks();
  if (lane == 0) {
    u32x4* rr = reinterpret_cast<u32x4*>(a.rec + wid);
    rr[0] = u32x4{0u, 0u, hw_id_reg(), xcc_id_reg()};
    rr[1] = u32x4{(uint32_t)t0, (uint32_t)(t0 >> 32), (uint32_t)t1, (uint32_t)(t1 >> 32)};
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const Pair b = merge(merge(wg[0], wg[1]), merge(wg[2], wg[3]));
    a.partials[2 * blockIdx.x] = b.s;
    a.partials[2 * blockIdx.x + 1] = b.c;
  }
}

template <int DT, int NL>
__global__ __launch_bounds__(256) void reduce_fp(ReduceArgs a) {
  reduce_body<DT, NL, NL>(a);
}
// The ring is for BF16 at one or two waves per SIMD.  There the arithmetic of
// a group (eight TwoSums per load of a lane, 64 or 32 a group) takes as long as
// its loads, and no other wave covers either: 4 GiB at 4 waves per CU 5.75 -> 7.25 TB/s, at 8
// 7.25 either way; 1 GiB 5.3 -> 7.0 and 6.9 -> 7.1; 64 MiB 4.3 -> 5.3 and 5.2 ->
// 5.6.  FP32 and FP8 have fewer operations per byte and read 2 % faster in
// batches at 4 waves (7.39 against 7.17 TB/s over 4 GiB); from 12 waves per CU
// on the two forms are within 2 % of each other or the ring loses (BF16 over
// 4 GiB at 32 waves 6.84 against 6.30).
template <int NL>
__global__ __launch_bounds__(256) void reduce_bf16_ring(ReduceArgs a) {
  reduce_body<SWEEP_BF16, NL, 0>(a);
}

// One or two loads at a time, for many waves (reduce_kernel's rule).
template <int DT, int AT>
__global__ __launch_bounds__(256) void reduce_fp_few(ReduceArgs a) {
  reduce_body<DT, 4, AT>(a);
}

template <int NL>
const void* reduce_of(int dtype) {
  switch (dtype) {
    case SWEEP_F32: return reinterpret_cast<const void*>(&reduce_fp<SWEEP_F32, NL>);
    case SWEEP_BF16: return reinterpret_cast<const void*>(&reduce_fp<SWEEP_BF16, NL>);
    case SWEEP_FP8_E4M3: return reinterpret_cast<const void*>(&reduce_fp<SWEEP_FP8_E4M3, NL>);
    default: return nullptr;
  }
}
template <int AT>
const void* reduce_few_of(int dtype) {
  switch (dtype) {
    case SWEEP_F32: return reinterpret_cast<const void*>(&reduce_fp_few<SWEEP_F32, AT>);
    case SWEEP_BF16: return reinterpret_cast<const void*>(&reduce_fp_few<SWEEP_BF16, AT>);
    case SWEEP_FP8_E4M3: return reinterpret_cast<const void*>(&reduce_fp_few<SWEEP_FP8_E4M3, AT>);
    default: return nullptr;
  }
}

// HBM reads fastest with about 6-8 MiB in flight, and four loads of each of
// many waves are 12-32 MiB.  Payloads beyond the 256 MiB last-level cache are
// read one load at a time from 24 MiB on, two from 12 (BF16, whose
// arithmetic needs more cover, from 16).  TB/s, four at a time -> fewer, 4 GiB
// of FP32 / BF16 / FP8: 12 waves per CU 7.07 -> 7.32 / 7.07 -> 6.90, not taken /
// 7.04 -> 7.20; 16 waves 6.99 -> 7.15 / 6.96 -> 7.17 / 6.98 -> 7.02; 20 waves
// 6.73 -> 7.05 / 6.60 -> 7.00 / 6.70 -> 7.00; 24 waves 6.53 -> 7.23 / 6.54 ->
// 7.10 / 6.45 -> 7.11; 32 waves 6.82 -> 7.05 / 6.83 -> 6.98 / 6.84 -> 6.98.  Over
// 512 MiB 32 waves gain nothing (FP32 and BF16 1 % slower), so their line is
// there; over 128 MiB most lose 1-5 %.
const void* reduce_kernel(int dtype, int waves_per_cu, uint64_t n_waves, uint64_t bytes) {
  // (with eight loads BF16 always takes the ring; reduce_of<8> holds it beside
  // the other types for the audit of the loops' assembly)
  const bool ring = dtype == SWEEP_BF16 && waves_per_cu <= 8;
  if (reduce_loads(waves_per_cu) == 8)
    return ring ? reinterpret_cast<const void*>(&reduce_bf16_ring<8>) : reduce_of<8>(dtype);
  if (ring) return reinterpret_cast<const void*>(&reduce_bf16_ring<4>);
  const uint64_t mib = n_waves * (4 * kWave * 16) >> 20;    // four loads of every wave
  if (bytes > (mib >= 32 ? 512ull << 20 : 256ull << 20)) {
    if (mib >= 24) return reduce_few_of<1>(dtype);
    if (mib >= (dtype == SWEEP_BF16 ? 16 : 12)) return reduce_few_of<2>(dtype);
  }
  return reduce_of<4>(dtype);
}

// Workgroup 0 combines the partial pairs in FP64, in a fixed order: thread t
// of 256 sums pairs t, t+256, ... and the 256 totals are added up a fixed
// binary tree.  Workgroup 1 folds the wave records beside it.  Both are
// latency bound, and as two launches of one workgroup each they cost 3.6 and
// 4.9 us and the gap between them; the pairs of a thread are read eight at a
// time.
constexpr int kPairBatch = 8;

__global__ __launch_bounds__(kFinishThreads) void finish_reduce(ReduceFinishArgs a) {
  if (blockIdx.x == 1) {
    fold_records(a.rec, 0, a.n_rec, a.out, LookAway());
    return;
  }
  __shared__ double sd[256];
  const uint32_t t = threadIdx.x;
  if (t >= 256) return;                  // whole waves; the barriers below count the rest
  const float2* pairs = reinterpret_cast<const float2*>(a.partials);
  double acc = 0.0;
  for (uint32_t b = t; b < a.n; b += kPairBatch * 256) {
    float2 p[kPairBatch];
#pragma unroll
    for (int u = 0; u < kPairBatch; ++u) {
      const uint32_t i = b + u * 256;
      p[u] = pairs[i < a.n ? i : a.n - 1];
    }
#pragma unroll
    for (int u = 0; u < kPairBatch; ++u)
      if (b + u * 256 < a.n) acc += (double)p[u].x + (double)p[u].y;
  }
  sd[t] = acc;
  __syncthreads();
  if (t < kWave) {
    // sd[t] + sd[t + 128], then + 64, 32, .. 1: the tree's pairs in its order
    double v = (sd[t] + sd[t + 128]) + (sd[t + 64] + sd[t + 192]);
    for (int h = kWave / 2; h > 0; h >>= 1) v += __shfl_down(v, h);
    if (t == 0) a.sum[0] = v;
  }
}

hipError_t launch_finish_reduce(const ReduceFinishArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(finish_reduce, dim3(2), dim3(kFinishThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace ilp
