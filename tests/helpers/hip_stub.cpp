// A stand-in for the HIP runtime on a machine without a GPU, for tests of the
// library's host code: every runtime function that libmetricgraph.so calls,
// over host memory, with a log of the calls.  Loaded into the global symbol
// scope before the library.  Of the kernels only the two that carry results
// to the host run (their copies, at the time of the launch); the others leave
// their memory as it is, so sets stay as allocated (zeros: particle on edge 0,
// position 0).  A call can be made to fail by name.
#include <dlfcn.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "../../paper_2512_02175_amd/csrc/mg_internal.h"

namespace {
struct Block {
  size_t bytes;
  int device;
  bool host;
};
std::map<char *, Block> g_mem;
std::map<const void *, std::string> g_kernel;
std::string g_log;
std::string g_fail;
int g_skip = 0, g_count = 0, g_device = 0, g_blocks_per_cu = 4;
bool g_capturing = false;
int g_fast = -1;

void log(const char *fmt, ...) __attribute__((format(printf, 1, 2)));
void log(const char *fmt, ...) {
  char line[1024];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(line, sizeof line, fmt, ap);
  va_end(ap);
  g_log += line;
  g_log += '\n';
}
// whether this call is one that was asked to fail
bool fails(const char *name) {
  if (g_fail != name || g_count == 0) return false;
  if (g_skip > 0) {
    --g_skip;
    return false;
  }
  --g_count;
  return true;
}
hipError_t alloc(void **p, size_t bytes, bool host) {
  *p = aligned_alloc(256, (bytes + 255) / 256 * 256);
  std::memset(*p, 0, bytes);
  g_mem[(char *)*p] = {bytes, g_device, host};
  return hipSuccess;
}
const Block *find(const void *p) {
  auto it = g_mem.upper_bound((char *)p);
  if (it == g_mem.begin()) return nullptr;
  --it;
  return (const char *)p < it->first + it->second.bytes ? &it->second : nullptr;
}
std::string args_of(const mg::StepArgs &a) {
  char b[256];
  snprintf(b, sizeof b, " nsteps=%u kernel=%d idle=%d refill=%d pool_cap=%u claim=%u", a.nsteps,
           a.kernel, a.idle, a.refill, a.pool_cap, a.claim_chunk);
  return b;
}
void run(const std::string &k, void **args) {
  if (k.find("k_copy_out") != std::string::npos) {
    const auto &c = *(const mg::CopyOut *)args[0];
    for (int i = 0; i < c.n; ++i) std::memcpy(c.dst[i], c.src[i], 4 * (size_t)c.words[i]);
  } else if (k.find("k_read") != std::string::npos) {
    const auto &g = *(const mg::GraphDev *)args[0];
    const auto &s = *(const mg::SetDev *)args[1];
    const uint32_t first = *(uint32_t *)args[2], count = *(uint32_t *)args[3];
    int32_t *edge = *(int32_t **)args[4];
    double *pos = *(double **)args[5];
    uint8_t *alive = *(uint8_t **)args[6];
    uint64_t *hash = *(uint64_t **)args[7];
    uint32_t *hits = *(uint32_t **)args[8];
    for (uint32_t i = 0; i < count; ++i) {
      const uint32_t ef = s.ef[first + i];
      const int32_t e = (int32_t)(ef & mg::kEdgeMask);
      if (edge) edge[i] = e;
      if (alive) alive[i] = !(ef & mg::kDeadBit);
      if (pos && s.x64) pos[i] = s.x64[first + i];
      if (pos && !s.x64) {
        const double y = (double)s.y32[first + i].x + (double)s.y32[first + i].y;
        pos[i] = (ef & mg::kSideBit) ? g.e64[e].L - y : y;
      }
      if (hash) hash[i] = s.seqhash[first + i];
      if (hits) hits[i] = s.hits[first + i];
    }
  }
}
}  // namespace

// The library's own allocations can be made to fail too ("new").
void *operator new(size_t bytes) {
  if (g_count > 0 && g_fail == "new") {
    Dl_info at;
    if (dladdr(__builtin_return_address(0), &at) && strstr(at.dli_fname, "libmetricgraph") &&
        fails("new"))
      throw std::bad_alloc();
  }
  if (void *p = malloc(bytes ? bytes : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

extern "C" {

// ------------------------------------------------------------- controls --
void stub_fail(const char *name, int skip, int count) {
  g_fail = name;
  g_skip = skip;
  g_count = count;
}
void stub_device(int d) { g_device = d; }
void stub_capture(int on) { g_capturing = on != 0; }
// Timings are 1 ms, but for the k-th from now.
void stub_fast(int k) { g_fast = k; }
void stub_blocks_per_cu(int n) { g_blocks_per_cu = n; }
void *stub_device_block(size_t bytes) {
  void *p;
  alloc(&p, bytes, false);
  return p;
}
// The log so far, which is then emptied.
const char *stub_log(void) {
  static std::string out;
  out = g_log;
  g_log.clear();
  return out.c_str();
}

// -------------------------------------------------------------- runtime --
void **__hipRegisterFatBinary(const void *) {
  static void *h;
  return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
  g_kernel[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

struct Config {
  dim3 grid, block;
  size_t shm;
  hipStream_t st;
};
static std::vector<Config> g_cfg;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shm, hipStream_t st) {
  g_cfg.push_back({grid, block, shm, st});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shm, hipStream_t *st) {
  const Config c = g_cfg.back();
  g_cfg.pop_back();
  *grid = c.grid;
  *block = c.block;
  *shm = c.shm;
  *st = c.st;
  return hipSuccess;
}
static hipError_t g_last = hipSuccess;
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t shm,
                           hipStream_t st) {
  const std::string &k = g_kernel[f];
  const bool step = k.find("k_pool") != std::string::npos || k.find("k_step") != std::string::npos;
  const bool bad = fails("hipLaunchKernel");
  log("launch%s %s grid=%u shm=%zu stream=%p device=%d%s", bad ? "-failed" : "", k.c_str(),
      grid.x, shm, (void *)st, g_device,
      step ? args_of(*(const mg::StepArgs *)args[2]).c_str() : "");
  if (bad) return g_last = hipErrorLaunchFailure;
  run(k, args);
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t) { return "an error of the stand-in"; }

hipError_t hipMalloc(void **p, size_t bytes) {
  log("malloc %zu device=%d", bytes, g_device);
  return fails("hipMalloc") ? hipErrorOutOfMemory : alloc(p, bytes, false);
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
  log("host_malloc %zu device=%d", bytes, g_device);
  return fails("hipHostMalloc") ? hipErrorOutOfMemory : alloc(p, bytes, true);
}
static hipError_t release(void *p) {
  g_mem.erase((char *)p);
  free(p);
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  log("free");
  return release(p);
}
hipError_t hipHostFree(void *p) {
  log("host_free");
  return release(p);
}
hipError_t hipMemcpy(void *d, const void *s, size_t bytes, hipMemcpyKind) {
  std::memcpy(d, s, bytes);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t bytes, hipMemcpyKind, hipStream_t st) {
  log("copy %zu stream=%p", bytes, (void *)st);
  if (fails("hipMemcpyAsync")) return hipErrorUnknown;
  std::memcpy(d, s, bytes);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t bytes, hipStream_t st) {
  log("memset %zu stream=%p", bytes, (void *)st);
  std::memset(d, v, bytes);
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  const Block *b = find(p);
  if (!b) return hipErrorInvalidValue;
  std::memset(a, 0, sizeof *a);
  a->type = b->host ? hipMemoryTypeHost : hipMemoryTypeDevice;
  a->device = b->device;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidSymbol; }

hipError_t hipGetDevice(int *d) {
  *d = g_device;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  g_device = d;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 0;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t shm) {
  *n = shm ? std::max(1, std::min(g_blocks_per_cu, (int)(163840 / shm))) : g_blocks_per_cu;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) {
  log("sync_device");
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st) {
  log("sync stream=%p", (void *)st);
  return fails("hipStreamSynchronize") ? hipErrorUnknown : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t *s) { return alloc((void **)s, 1, true); }
hipError_t hipStreamDestroy(hipStream_t s) { return release((void *)s); }

struct Event {
  int device;
};
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  *e = (hipEvent_t) new Event{g_device};
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete (Event *)e;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
  log("record event_device=%d stream=%p", ((Event *)e)->device, (void *)st);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = g_fast-- == 0 ? 0.5f : 1.0f;
  return hipSuccess;
}

hipError_t hipGraphCreate(hipGraph_t *g, unsigned) { return alloc((void **)g, 1, true); }
hipError_t hipGraphDestroy(hipGraph_t g) { return release((void *)g); }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  return alloc((void **)e, 1, true);
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { return release((void *)e); }
hipError_t hipGraphAddKernelNode(hipGraphNode_t *n, hipGraph_t, const hipGraphNode_t *,
                                 size_t deps, const hipKernelNodeParams *p) {
  static char node[1 << 16];
  static size_t next = 0;
  *n = (hipGraphNode_t)&node[next++ % sizeof node];
  const std::string &k = g_kernel[p->func];
  const bool step = k.find("batch_reset") == std::string::npos;
  log("node %s grid=%u shm=%u after=%zu%s", k.c_str(), p->gridDim.x, p->sharedMemBytes, deps,
      step ? args_of(*(const mg::StepArgs *)p->kernelParams[3]).c_str() : "");
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t st) {
  log("graph stream=%p", (void *)st);
  return hipSuccess;
}

}  // extern "C"
