// A stand-in for the HIP runtime and the kernel launchers, so that the host side of
// the library (slh_api.cpp) runs without a GPU: device memory is host memory, events
// complete at once, and every call that matters to the order of the work is written
// to a log, one per line, as "name stream ..." (streams and events as numbers).
#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include "slh_internal.h"

namespace {
std::string g_log;
std::map<void*, size_t> g_mem;
long g_events = 0;
int g_groups = -1;                    // distinct rows that launch_group reports (-1: none taken)
int g_resident = 0;                   // blocks per window of the resident kernel (0: streaming)
int g_fail_resident = 0;              // launches of it that fail
int g_fail_events = 0;                // event records and waits that fail
void* g_capturing = nullptr;          // stream under the caller's capture
bool g_capture_on = false;
long g_own_capture = 0;               // the library's own capture

void log(const char* fmt, ...) {
  char b[256];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(b, sizeof b, fmt, ap);
  va_end(ap);
  g_log += b;
  g_log += '\n';
}
long id(const void* p) { return (long)(intptr_t)p; }
hipError_t launched(const char* name, hipStream_t s, long arg = 0) {
  log("%s %ld %ld", name, id(s), arg);
  return hipSuccess;
}
}  // namespace

extern "C" {
const char* stub_log() { return g_log.c_str(); }
void stub_clear() { g_log.clear(); }
void stub_groups(int n) { g_groups = n; }
void stub_resident(int nb) { g_resident = nb; }
void stub_fail_resident(int n) { g_fail_resident = n; }
void stub_fail_events(int n) { g_fail_events = n; }
void stub_capture(void* s, int on) {
  g_capturing = s;
  g_capture_on = on != 0;
}

hipError_t hipMalloc(void** p, size_t n) {
  if (g_capture_on) return hipErrorStreamCaptureUnsupported;
  *p = calloc(1, n);
  g_mem[*p] = n;
  log("malloc 0 %zu", n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  if (g_capture_on) return hipErrorStreamCaptureUnsupported;
  log("free 0 %zu", g_mem[p]);
  g_mem.erase(p);
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset((void*)p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return launched("device_sync", nullptr); }
hipError_t hipStreamSynchronize(hipStream_t s) { return launched("stream_sync", s); }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)(intptr_t)(1000000 + ++g_events);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = g_capture_on && (void*)s == g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)(intptr_t)++g_events;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  return g_fail_events > 0 ? (--g_fail_events, hipErrorInvalidHandle) : launched("record", s, id(e));
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  return g_fail_events > 0 ? (--g_fail_events, hipErrorInvalidHandle) : launched("wait", s, id(e));
}
hipError_t hipEventQuery(hipEvent_t e) { return launched("query", nullptr, id(e)); }
hipError_t hipEventSynchronize(hipEvent_t e) { return launched("event_sync", nullptr, id(e)); }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  ++g_own_capture;
  return launched("begin_capture", s);
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  *g = (hipGraph_t)(intptr_t)g_own_capture;
  return launched("end_capture", s);
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)g;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) { return launched("graph_launch", s, id(e)); }
}  // extern "C"

namespace slh {
hipError_t launch_rownorm(const void*, int, int64_t, int64_t, int, int, int, double*, double*, double*,
                          float*, uint16_t*, hipStream_t s) {
  return launched("rownorm", s);
}
hipError_t launch_gather_windows(double*, const double*, const int*, int64_t, int, hipStream_t s) {
  return launched("gather", s);
}
hipError_t launch_group(const GroupWS& w, const uint16_t*, int64_t, int, hipStream_t s) {
  for (int a = 0; a < w.n_act; ++a) w.n_out[a] = g_groups;
  return launched("group", s);
}
hipError_t launch_group_expand(const GroupWS&, const double*, int64_t, int64_t, int64_t, int, double*,
                               int64_t, int64_t, int64_t, hipStream_t s) {
  return launched("expand", s);
}
hipError_t launch_group_copy(const GroupWS&, const void*, int64_t, int, void*, hipStream_t s) {
  return launched("group_copy", s);
}
hipError_t launch_featmap(const FeatmapArgs& a, int, hipStream_t s, hipEvent_t, hipEvent_t) {
  return launched("featmap", s, (long)a.n_rows);
}
hipError_t launch_lanczos(const LanczosWS&, const double*, hipStream_t s, const hipEvent_t*,
                          const hipEvent_t*) {
  return launched("lanczos", s);
}
hipError_t launch_lanczos_passes(const LanczosWS&, int, int, hipStream_t s) { return launched("passes", s); }
int lanczos_resident_blocks(const LanczosWS&, int) { return g_resident; }
int lanczos_resident_most_blocks(const LanczosWS&) { return 256; }
size_t lanczos_resident_bar_words() { return (size_t)LZ_BAR_ERR + 32; }
hipError_t launch_lanczos_resident(const LanczosWS&, const double*, unsigned*, int, hipStream_t s,
                                   hipEvent_t, hipEvent_t) {
  if (g_fail_resident > 0) {
    --g_fail_resident;
    return hipErrorUnknown;
  }
  return launched("resident", s);
}
hipError_t launch_eigh_ritz(const double*, const double*, const int*, int, int, int, double*, double*,
                            const double*, int, int, double*, int, hipStream_t s) {
  return launched("eigh_ritz", s);
}
hipError_t launch_simhash(const double*, int, const GroupWS*, const double*, const int*, int, int, int, int,
                          uint32_t*, double*, hipStream_t s) {
  return launched("simhash", s);
}
bool local_supported(int L, int n_it, int) { return L <= 32 && n_it <= L; }
hipError_t launch_local(const float*, int, int, int, int, int, double, const double*, double*, double*,
                        double*, int*, double*, double*, hipStream_t s) {
  return launched("local", s);
}
int normalise_groups(int n_act, int L, int m, int n_cu) { return (L + 63) / 64; }
hipError_t launch_normalise(float*, const double*, int64_t, int, int, int, int, double*, double*, double*,
                            hipStream_t s) {
  return launched("normalise", s);
}
hipError_t launch_energy(const float*, const double*, int64_t, const double*, int, int, int, int, double*,
                         double*, hipStream_t s) {
  return launched("energy", s);
}
hipError_t launch_purity(const void*, int, int64_t, int, const int*, const int*, const double*, int64_t,
                         const int*, int, double, unsigned long long*, hipStream_t s) {
  return launched("purity", s);
}
hipError_t launch_fill_u32(uint32_t*, int64_t, uint32_t, hipStream_t s) { return launched("fill", s); }
int merge_nchunks(int64_t N, int CH) { return (int)((N + CH - 1) / CH); }
int64_t merge_tiled_ws(int, int64_t, int, int*, MergeWS*) { return 0; }
int merge_chunk(int64_t, int64_t, int) { return 16; }
hipError_t launch_merge(const MergeWS&, const void*, int, int64_t, float*, const MergeOut&, hipStream_t s) {
  return launched("merge", s);
}
hipError_t launch_merge_tail(const void*, int, int64_t, int, int64_t, int, const int*, int, float*, int*,
                             int*, hipStream_t s) {
  return launched("merge_tail", s);
}
int route_slices(int) { return 1; }
int route_norm_groups(int, int) { return 0; }
hipError_t launch_route_norm_scores(const void*, int, int64_t, int, int, int, int, int, double*, double*,
                                    double*, float*, uint16_t*, double*, double*, double*, hipStream_t s) {
  return launched("route", s);
}
hipError_t launch_route_scores(const void*, int, int64_t, const double*, int, int, int, double*, double*,
                               hipStream_t s) {
  return launched("route", s);
}
}  // namespace slh
