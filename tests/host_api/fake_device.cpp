// A stand-in for the device side of libpnerf, on the CPU: the HIP runtime calls
// and the kernel launchers that api.hip uses.  Linked with api.hip's host pass
// it runs the library's own host code -- workspaces, chunk plans, what a failed
// call leaves behind -- without a GPU.  "Device" memory is reserved host memory;
// launchers note what they were given and fill in the few words that the host
// reads back.
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <cstdlib>
#include <cstring>
#include <map>

#include "../../paper_2210_10108_amd/csrc/pnerf_internal.h"

using namespace pnerf;

namespace {
std::map<void*, size_t> g_mem;  // device allocations
size_t g_bytes = 0, g_peak = 0;
size_t g_limit = (size_t)-1;    // hipMalloc fails above this many bytes in all
int g_samples = 0;              // samples of every hypothesis
int g_calls = 0;                // counted batches marched
int g_inspected = 0;            // inspection kernels launched
int g_encodes = 0;              // encoding kernels launched
DevField g_field;               // the field of the last one
}  // namespace

extern "C" {
void fake_reset() { g_limit = (size_t)-1; g_samples = g_calls = g_inspected = g_encodes = 0; g_peak = g_bytes; }
void fake_limit(size_t bytes) { g_limit = bytes; }
void fake_samples(int per_hypothesis) { g_samples = per_hypothesis; }
size_t fake_bytes() { return g_bytes; }
size_t fake_peak() { return g_peak; }
int fake_inspected() { return g_inspected; }
int fake_encodes() { return g_encodes; }
// the queues of the last encoding: first levels [n_queue + 1], levels [L]
int fake_queues(int* first, int* level, int* n_hashed) {
  std::memcpy(first, g_field.q_first, sizeof(int) * (g_field.n_queue + 1));
  std::memcpy(level, g_field.q_level, sizeof(int) * g_field.L);
  *n_hashed = g_field.n_hashed_queue;
  return g_field.n_queue;
}

// ------------------------------------------------------------- HIP runtime
hipError_t hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (g_bytes + n > g_limit) return hipErrorOutOfMemory;
  void* m = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return hipErrorOutOfMemory;
  g_mem[m] = n;
  g_bytes += n;
  if (g_bytes > g_peak) g_peak = g_bytes;
  *p = m;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  auto it = g_mem.find(p);
  if (it == g_mem.end()) return hipErrorInvalidValue;
  munmap(p, it->second);
  g_bytes -= it->second;
  g_mem.erase(it);
  return hipSuccess;
}
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return hipMalloc(p, n); }
hipError_t hipFreeAsync(void* p, hipStream_t) { return hipFree(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)std::malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free((void*)s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void*)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
}  // extern "C"

// --------------------------------------------------------------- launchers
namespace pnerf {
hipError_t launch_march_count(const DevField&, const DevBatch& b, const DevWork& w, bool,
                              int* raw_blocks, hipStream_t) {
  *raw_blocks = 0;
  for (int k = 0; k < b.K; ++k) w.hyp_total[k] = g_samples;
  w.rrec[0].x = (float)++g_calls;  // the ray records are this call's from here on
  *w.total = b.K * g_samples;
  return hipSuccess;
}
hipError_t launch_march_write(const DevField&, const DevBatch& b, const DevWork&, const DevWork& wc,
                              int, int, int, int, int32_t*, hipStream_t) {
  *wc.total = b.K * g_samples;
  wc.t[0] = wc.rrec[0].x;
  return hipSuccess;
}
// what 3 reads the ray records beside the sample buffer: dst[0] is the call the
// sample buffer is from, dst[1] the call the records are from
hipError_t launch_inspect(const DevField&, const DevBatch&, const DevWork& w, int what, float* dst,
                          int64_t, hipStream_t) {
  ++g_inspected;
  dst[0] = w.t[0];
  dst[1] = what == 3 && w.rrec ? w.rrec[0].x : -1.0f;
  return hipSuccess;
}
hipError_t launch_encode(const DevField& f, const DevWork&, int64_t, int, int, int, hipStream_t) {
  ++g_encodes;
  g_field = f;
  return hipSuccess;
}
hipError_t launch_mlp_fwd(const DevField&, const DevBatch&, const DevWork&, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_composite(const DevField&, const DevBatch&, const DevWork&, int, float*, hipStream_t) { return hipSuccess; }
hipError_t launch_mlp_bwd(const DevField&, const DevBatch&, const DevWork&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_reduce(const DevField&, const DevBatch&, const DevWork&, float*, float*, hipStream_t) { return hipSuccess; }
hipError_t launch_ray_bwd(const DevField&, const DevBatch&, const DevWork&, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_reduce_rays(const DevBatch&, const DevWork&, float*, float*, hipStream_t) { return hipSuccess; }
hipError_t launch_occupancy(const DevField&, uint32_t*, int, float, hipStream_t) { return hipSuccess; }
hipError_t launch_copy_samples(const float*, const int32_t*, float*, int32_t*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_offsets_i64(const int32_t*, int64_t*, int, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_step_momentum(int, float*, float*, const float*, float, float, hipStream_t) { return hipSuccess; }
hipError_t launch_step_adam(int, float*, float*, const float*, double, double, double, double, double,
                            int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_resample(int, float*, float*, int, const float*, int, float, float, uint64_t,
                           uint32_t, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t resample_scratch(int, int32_t**, int*) { return hipErrorUnknown; }
int mlp_fwd_blocks_per_cu(int, int) { return 4; }
int mlp_bwd_blocks_per_cu(int, int, int) { return 4; }
int ray_bwd_blocks_per_cu(int, int, int) { return 2; }
int encode_blocks_per_cu(const DevField&) { return 7; }
}  // namespace pnerf
