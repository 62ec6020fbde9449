// A HIP runtime without a device, for tests of the host runtime: one gfx950
// of 256 CUs whose memory is the host's, whose kernels do nothing and whose
// launches are listed.  Loaded in front of the library, under the real
// runtime's name.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Launch {
  std::string kernel;
  uint64_t args[8];           // the head of the kernel's argument struct
  void *start, *stop;         // the events that it was launched with
};
struct Event {
  unsigned flags;
};

std::map<const void*, std::string> g_names;
std::vector<Launch> g_launches;
size_t g_pinned = SIZE_MAX;   // an allocation of more pinned bytes fails
int g_fail = -1;              // the launch that fails, counted from the last reset
std::vector<void*> g_from;    // start events of the intervals asked for
dim3 g_grid, g_block;
size_t g_lds = 0;
hipStream_t g_stream = nullptr;

hipError_t allocate(void** p, size_t n) {
  *p = std::calloc(1, n);
  return hipSuccess;
}

hipError_t launch(const void* fn, void** args, void* start = nullptr, void* stop = nullptr) {
  Launch l;
  l.kernel = g_names.at(fn);
  l.start = start;
  l.stop = stop;
  std::memset(l.args, 0, sizeof(l.args));
  // the structs whose pointers the tests look at
  if (l.kernel.find("finish_") != std::string::npos) std::memcpy(l.args, args[0], 48);
  if (l.kernel.find("gate") != std::string::npos) std::memcpy(l.args, args[0], 16);
  g_launches.push_back(l);
  return (int)g_launches.size() - 1 == g_fail ? hipErrorLaunchFailure : hipSuccess;
}

}  // namespace

extern "C" {

// ---- the tests' side
void fake_reset() {
  g_launches.clear();
  g_from.clear();
  g_fail = -1;
}
void fake_fail_launch(int i) { g_fail = i; }
void fake_limit_pinned(size_t bytes) { g_pinned = bytes; }
int fake_launches() { return (int)g_launches.size(); }
const char* fake_kernel(int i) { return g_launches[(size_t)i].kernel.c_str(); }
uint64_t fake_arg(int i, int k) { return g_launches[(size_t)i].args[k]; }
// Which launch ended with the event that interval i was measured from, or -1.
int fake_interval_from(int i) {
  for (size_t k = 0; (size_t)i < g_from.size() && k < g_launches.size(); ++k)
    if (g_launches[k].stop && g_launches[k].stop == g_from[(size_t)i]) return (int)k;
  return -1;
}

// ---- registration and launches
void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) {
  g_grid = grid;
  g_block = block;
  g_lds = lds;
  g_stream = st;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) {
  *grid = g_grid;
  *block = g_block;
  *lds = g_lds;
  *st = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3, dim3, void** args, size_t, hipStream_t) {
  return launch(fn, args);
}
hipError_t hipExtLaunchKernel(const void* fn, dim3, dim3, void** args, size_t, hipStream_t,
                              hipEvent_t start, hipEvent_t stop, int) {
  return launch(fn, args, start, stop);
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) {
  std::memset(a, 0, sizeof(*a));
  a->numRegs = 64;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 8;
  return hipSuccess;
}

// ---- the device
hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  p->maxSharedMemoryPerMultiProcessor = 160 << 10;
  p->sharedMemPerBlock = 160 << 10;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 100000;
  return hipSuccess;
}

// ---- memory
hipError_t hipMalloc(void** p, size_t n) { return allocate(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  return n > g_pinned ? hipErrorOutOfMemory : allocate(p, n);
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyWithStream(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static char scratch[(512 << 10) + 256];
  *p = scratch;
  return hipSuccess;
}

// ---- events, streams, graphs
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags) {
  *e = reinterpret_cast<hipEvent_t>(new Event{flags});
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, hipEventDefault); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete reinterpret_cast<Event*>(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t start, hipEvent_t) {
  g_from.push_back(start);
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(new int(0));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  delete reinterpret_cast<int*>(s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = reinterpret_cast<hipGraph_t>(new int(0));
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *x = reinterpret_cast<hipGraphExec_t>(new int(0));
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete reinterpret_cast<int*>(g);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  delete reinterpret_cast<int*>(x);
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake"; }

}  // extern "C"
