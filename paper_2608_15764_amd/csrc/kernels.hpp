// Kernel argument blocks and host-side launch entry points of the gfx950
// kernels.  Each kernel family lives in its own translation unit and is
// reached from the runtime only through the functions declared here.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ilpsweep.h"

namespace ilp {

constexpr int kMaxK = 16;
constexpr int kPlainWgThreads = 256;   // 4 waves, one per SIMD

// Per-cell result reduced on the device from the wave records.
struct alignas(16) CellRes {
  uint64_t sum;   // low 32 bits used
  uint64_t xr;    // low 32 bits used
  uint64_t tmin;
  uint64_t tmax;
};

// Plain K-load cell.  Round robin (and strided): wave w of n_waves handles
// wave-groups q = w, w + n_waves, ... below Q, iters of them and one more if
// w < extra; blocked: q = w*G .. w*G + G - 1.  All steps are in bytes: load j
// of group q reads the 64 vectors starting at (q*gstep + j*jstep) mod bytes:
// gstep = K segments, jstep = 1 (adjacent segments, (q*K + j) segments), or
// in the strided layout gstep = 1 segment, jstep = Q segments ((j*Q + q)
// segments).  `stride` is the step between a wave's consecutive groups, mod
// bytes: n_waves*gstep (round robin, strided) or gstep (blocked).
struct PlainArgs {
  const uint8_t* buf;
  uint64_t bytes;
  uint64_t Q;
  uint64_t stride;
  sweep_wave_rec_t* rec;
  uint32_t* lane_out;
  uint64_t G;          // groups per wave in blocked order
  uint32_t order;      // SWEEP_ORDER_*
  uint32_t iters;      // Q / n_waves
  uint32_t extra;      // Q mod n_waves
  uint64_t gstep;
  uint64_t jstep;      // mod bytes
};

// Buffers of this many bytes and more are walked with 64-bit cursors.
constexpr uint64_t kFarBytes = 1ull << 32;

// Fused batch of plain cells that share K, vector width, cache policy and
// launch shape: one persistent launch over their concatenated wave-groups.
// Point p owns global groups [g0, g0 + Q); wave w of n_waves handles global
// groups w, w + n_waves, ... (round robin over the concatenation), reading
// load j of its point's local group q at segment (q*K + j) mod the point's
// size.  Steps and sizes are in bytes; `stride` = n_waves*K segments, mod
// `bytes`, lies between two of a wave's groups inside one point.  Wave w's record for point p is
// rec[p*n_waves + w]; records of points a wave never reaches are left as
// they are (cleared once, before the first launch, to "empty").
struct FusedPoint {
  uint64_t off;            // the point's buffer: FusedArgs::base + off
  uint64_t bytes;
  uint64_t Q;
  uint64_t g0;
  uint64_t stride;
};
struct FusedArgs {
  const uint8_t* base;     // the lowest point buffer of the launch
  const FusedPoint* pts;   // device, n_pts entries
  uint64_t total_groups;   // sum of Q over the points
  sweep_wave_rec_t* rec;   // n_pts * n_waves records
};

// LDS-ring cell (async or matched), `waves` waves per workgroup; steps and
// iteration counts as in PlainArgs, round robin.
struct LdsArgs {
  const uint8_t* buf;
  uint64_t bytes;
  uint64_t stride;        // n_waves groups of D segments, mod bytes
  sweep_wave_rec_t* rec;
  uint32_t* lane_out;
  uint32_t iters, extra;
  uint32_t waves;         // waves per workgroup
};

// Two co-resident streams: A (plain K = D) on region A, B (LDS-async ring
// of depth D) on region B.  Records of A come first (n_waves_a of them),
// then those of B.
struct StreamArgs {
  const uint8_t* buf;
  uint64_t bytes, stride;
  uint32_t iters, extra;
};
struct TwoStreamArgs {
  StreamArgs a, b;
  sweep_wave_rec_t* rec;   // n_waves_a + n_waves_b records
  uint32_t* lane_out;      // lanes of A then lanes of B, or null
  uint32_t waves_a, waves_b;  // per workgroup
  uint32_t b_plain;           // 1: stream B runs the plain loop as well
  uint32_t split;             // 1: each workgroup runs one stream only
};

// Precision variant: full wave-groups of 4 or 8 loads x 64 lanes x 16 bytes,
// then the ragged remainder (whole 16-byte vectors, then the last bytes).
struct ReduceArgs {
  const uint8_t* payload;
  uint64_t n_groups;        // full wave-groups (loads x 1 KiB each)
  uint64_t n_vec;           // whole 16-byte vectors
  uint64_t n_bytes;         // payload bytes
  float* partials;          // 2 floats (s, c) per workgroup
  sweep_wave_rec_t* rec;
};

// Its finish: `n` partial pairs into *sum, `n_rec` wave records into *out;
// both results are device or pinned host memory.
struct ReduceFinishArgs {
  const float* partials;
  uint32_t n;
  double* sum;
  const sweep_wave_rec_t* rec;
  uint64_t n_rec;
  CellRes* out;
};

// Pointer chase: buf[idx] holds the next index (32-bit words); `out`
// receives {final index, wall t0, wall t1, shader-clock t0, shader-clock t1}.
constexpr uint32_t kMaxChaseSamples = 4096;
struct ChaseArgs {
  const uint32_t* buf;
  uint32_t n_bytes;        // buffer bytes (< 4 GiB)
  uint32_t start;
  uint32_t warm;           // untimed hops
  uint32_t steps;          // timed hops
  uint32_t n_samples;      // per-hop cycle samples (first hops), <= 4096
  uint32_t* samples;       // device [n_samples] or null if n_samples == 0
  uint64_t* out;           // device [5]
};

// Several dependent-chain walkers at once, one single-lane wave per
// workgroup; walker b starts at starts[b] and writes out[4b .. 4b+3] =
// final index, wall clock at the start and end of its timed hops, XCC_ID.
constexpr uint32_t kMaxWalkers = 64;
struct WalkArgs {
  const uint32_t* buf;
  uint32_t n_bytes;        // buffer bytes (< 4 GiB)
  uint32_t warm;           // untimed hops per walker
  uint32_t steps;          // timed hops per walker
  uint32_t n_walkers;      // 1..kMaxWalkers (= the grid)
  uint32_t starts[kMaxWalkers];
  uint64_t* out;           // device [4 * n_walkers]
};

// Streaming read by the workgroups of chosen XCDs only (sweep_xcd_subset).
// Workgroup b belongs to XCD b mod 8; the active waves, numbered densely,
// read groups of kXcdK adjacent 64-lane segments of 16-byte vectors dealt
// round robin: group i * n_act + w goes to active wave w.
constexpr int kXcdK = 8;
struct XcdArgs {
  const uint8_t* buf;
  uint64_t groups;         // groups per active wave
  uint64_t n_act;          // active waves
  uint32_t mask;           // bit x set: workgroups on XCD x work
  uint32_t pop;            // set bits in mask
  sweep_wave_rec_t* rec;   // device [n_act]
};

// Static split weighted per XCD (sweep_xcd_split): XCD x reads groups
// [starts[x], starts[x+1]) of kXcdK segments, dealt round robin over its own
// waves; waves are numbered (rank of the XCD among those with a share,
// wave within the XCD).
struct XcdSplitArgs {
  const uint8_t* buf;
  uint64_t starts[9];      // group prefix sums per XCD
  uint32_t per_xcd;        // waves per XCD
  uint32_t mask;           // XCDs with a nonzero share
  sweep_wave_rec_t* rec;   // device [popcount(mask) * per_xcd]
};

// Folding of wave records into cell results: cell c owns records
// [offsets[c], offsets[c+1]).  The offsets of up to kFewCells cells travel in
// the argument block (`offsets` null); those of more lie where the device can
// read them.  `out` is device or pinned host memory.
constexpr size_t kFewCells = 64;
struct FinishArgs {
  const sweep_wave_rec_t* rec;
  const uint64_t* offsets;
  CellRes* out;
  uint32_t few[kFewCells + 1];
};

// Its finish: the fold of the n_rec records (below 2^32) into *out, and the
// index of the first record that was not written, or not by the XCD it
// should be from, into *first_bad (all ones if there is none).  Records come
// in runs of `run` per XCD, going round the n_xcds XCDs of `xcds` (four bits
// each, the first one lowest).
struct XcdFinishArgs {
  const sweep_wave_rec_t* rec;
  uint64_t n_rec;
  CellRes* out;
  uint64_t* first_bad;
  uint32_t run, n_xcds, xcds;
};

// ---- static scratch of the allocation-free entry point (static_scratch.hip)
// Layout: per-wave records, then the cell result.  512 KiB + 256 bytes per
// device.
constexpr uint64_t kStaticRecords = 16384;
constexpr uint64_t kStaticResOffset = kStaticRecords * sizeof(sweep_wave_rec_t);
constexpr uint64_t kStaticScratchBytes = kStaticResOffset + 256;
// Device address of the calling thread's current device's copy of the
// static scratch (resolved once per device, with that device current).
hipError_t static_scratch(int ordinal, uint8_t** ptr);

// ---- kernel lookup: the host launches these with their one argument
// struct (PlainArgs, LdsArgs, TwoStreamArgs, ReduceArgs); nullptr for an
// unknown combination.
// plain (kernels_plain.hip), in the form for `resident` waves on a CU at a
// time over `bytes`
const void* plain_kernel(int K, int V, int policy, int order, uint64_t resident,
                         uint64_t bytes);
// fused plain batch (kernels_fused.hip), in the form for n_waves waves at a
// time; `far` if a point has kFarBytes or more
const void* fused_kernel(int K, int V, int policy, uint64_t n_waves, bool far);
const void* xcd_kernel(int policy);
const void* xcd_split_kernel(int policy);
// Set `n` records to "empty" (zero sinks, t0 = all ones, t1 = 0), which
// the finishing kernel's min / max ignore.
hipError_t launch_clear_records(sweep_wave_rec_t* rec, uint64_t n, hipStream_t st);

// ---- LDS paths (kernels_lds.hip)
const void* lds_kernel(int kind, int D, int policy, bool far);
const void* two_stream_kernel(int D, int policy, bool far);

// ---- pointer chase (kernels_chase.hip)
const void* chase_kernel(int policy);
hipError_t launch_chase(int policy, hipStream_t st, const ChaseArgs& a);
hipError_t launch_walkers(int policy, hipStream_t st, const WalkArgs& a);

// ---- fill, finishing, clock, reduction (kernels_misc.hip)
hipError_t launch_fill(uint32_t* buf, uint64_t n_words, uint64_t seed,
                       hipStream_t st);
// One workgroup per cell.
hipError_t launch_finish_cells(const FinishArgs& a, uint32_t n_cells, hipStream_t st);
hipError_t launch_finish_xcd(const XcdFinishArgs& a, hipStream_t st);
// One wave that leaves when `*flag` has come to `ticket`, or after `ticks` of
// the wall clock; `done` is stamped with its end.
struct GateArgs {
  const uint32_t* flag;   // pinned host memory
  uint32_t ticket;
  uint32_t ticks;
};
constexpr double kGateSeconds = 200e-6;   // a host that takes longer is timed with the dispatch
hipError_t launch_gate(const GateArgs& a, hipStream_t st, hipEvent_t done);
hipError_t launch_read_clock(uint64_t* out, hipStream_t st);
// 16-byte loads of a lane's group: 8 at one wave per SIMD, 4 above, so that
// the forms that ask for a whole group at a time, or keep one in flight, have
// at least 8 MiB in flight at every occupancy of the default grid.  (Those for
// many waves ask for one or two loads at a time, 6 MiB and more.)
constexpr int reduce_loads(int waves_per_cu) { return waves_per_cu == 4 ? 8 : 4; }
// in the form for n_waves waves over `bytes`
const void* reduce_kernel(int dtype, int waves_per_cu, uint64_t n_waves, uint64_t bytes);
hipError_t launch_finish_reduce(const ReduceFinishArgs& a, hipStream_t st);

}  // namespace ilp
