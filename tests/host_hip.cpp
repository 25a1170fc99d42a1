// A stand-in for the HIP runtime, for CPU tests of the library's host code:
// device memory is host memory, copies are done at once, launches are only
// written down.  Loaded with RTLD_GLOBAL before libsdeliver.so, its functions
// take the place of the runtime's.  It refuses what the runtime refuses (an
// event recorded on another device's stream, a wait on a stream that is being
// captured) and what a test tells it to (pinned memory).
#define __HIP_PLATFORM_AMD__ 1
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "../paper_2109_12855_amd/csrc/sd_internal.h"

namespace {
struct Stream { int device; bool capturing; };
struct Event { int device; };
struct Launch { int64_t f[8]; };
std::mutex mu;
std::map<const void*, std::string> names;
std::vector<Launch> launches;
Stream null_stream{0, false};
int device = 0;
bool no_pinned = false, end_early = false, record = false;
int64_t n_pinned = 0, n_recorded = 0;
struct { dim3 grid, block; size_t lds; hipStream_t s; } config;

Stream* of(hipStream_t s) { return s ? (Stream*)s : &null_stream; }
bool is(const std::string& n, const char* k) { return n.find(k) != std::string::npos; }

void note(const void* fn, void** args, hipStream_t s) {
  const std::string n = names.count(fn) ? names[fn] : std::string();
  Launch l{};
  l.f[1] = (int64_t)s;
  if (is(n, "k_persist")) {
    const auto* p = (const sd::PersistArgs*)args[0];
    l.f[0] = 1;
    l.f[2] = p->S;
    l.f[3] = p->epoch0;
    l.f[4] = p->a.seg_lanes;
    if (end_early) {
      *p->ended = p->serial;
      *p->a.overflow |= 16;
    }
    // two blocks' rasters as a slow second block leaves them: its spikes of a
    // slice (neuron 64) after the first block's of the next one (neuron 0)
    if (record)
      for (int k = 0; k <= p->S; ++k)
        for (int b = 0; b < 2; ++b) {
          if (k - b < 0 || k - b >= p->S) continue;
          const int64_t t = p->t0 + (int64_t)(k - b) * p->a.Dmin;
          p->a.rec[(*p->a.rec_n)++] = make_uint2((uint32_t)t, 64u * b);
        }
  } else if (is(n, "k_slice1")) {
    const auto* a = (const sd::SliceArgs*)args[0];
    l.f[0] = 2;
    l.f[4] = a->seg_lanes;
  } else if (is(n, "k_fill") && !is(n, "k_fill_sm")) {
    const auto* b = (const sd::BuildArgs*)args[0];  // the table's size, as the scan leaves it
    b->row[b->n_src * b->NB] = (uint32_t)(b->N * b->K);
    return;
  } else {
    return;
  }
  std::lock_guard<std::mutex> lock(mu);
  launches.push_back(l);
}
}  // namespace

extern "C" {
// ---- what a test sees and sets ----------------------------------------------
int64_t host_launches() { return (int64_t)launches.size(); }
void host_launch(int64_t i, int64_t* out) { std::memcpy(out, launches[(size_t)i].f, sizeof(Launch)); }
void host_clear() { launches.clear(); }
void host_no_pinned(int on) { no_pinned = on; }
void host_end_early(int on) { end_early = on; }  // persistent launches to come
void host_record(int on) { record = on; }
int64_t host_pinned() { return n_pinned; }
int64_t host_recorded() { return n_recorded; }
void host_capture(void* s, int on) { of((hipStream_t)s)->capturing = on; }
void host_device(int d) { device = d; }
void* host_stream(int d) { return new Stream{d, false}; }

// ---- the runtime --------------------------------------------------------------
void** __hipRegisterFatBinary(const void*) {
  static void* h = nullptr;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  names[fn] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  config = {g, b, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = config.grid;
  *b = config.block;
  *lds = config.lds;
  *s = config.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t s) {
  note(f, args, s);
  return hipSuccess;
}
hipError_t hipLaunchCooperativeKernel(const void* f, dim3, dim3, void** args, unsigned,
                                      hipStream_t s) {
  note(f, args, s);
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount          ? 256
       : a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024
                                                           : 1;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { return *d = device, hipSuccess; }
hipError_t hipSetDevice(int d) { return device = d, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof *p);
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { return (*p = std::calloc(n, 1)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = nullptr;
  if (no_pinned) return hipErrorOutOfMemory;
  ++n_pinned;
  *p = std::calloc(n, 1);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemcpy2D(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind) {
  return hipErrorNotSupported;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  if (of(st)->capturing) ++n_recorded;
  else std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  return std::memset(d, v, n), hipSuccess;
}
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t) new Stream{device, false};
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  return of(s)->capturing ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
  *c = of(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  return of(s)->capturing = true, hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  return of(s)->capturing = false, *g = nullptr, hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipErrorNotSupported;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t) new Event{device};
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete (Event*)e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  return ((Event*)e)->device == of(s)->device ? hipSuccess : hipErrorInvalidHandle;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0.f, hipSuccess; }
}
