#include "fake_hip.h"

#include <cstdlib>
#include <cstring>
#include <map>

using namespace mona;

namespace fake {
std::function<void(const Launch&)> on_launch;
bool capturing = false;
std::string fail;
int capability_major = 256, capability_minor = 256;
int device = 0, queries = 0;
namespace {
std::map<const void*, std::string> names;
std::vector<std::function<void()>> recorded;
hipError_t last = hipSuccess;
struct Config { dim3 grid, block; size_t shmem; hipStream_t stream; };
std::vector<Config> configs;

bool failing(const std::string& what) {
  if (fail.empty() || what.find(fail) == std::string::npos) return false;
  fail.clear();
  return true;
}
bool is_captured(hipStream_t s) { return capturing && s != nullptr; }

// sizes of the arguments of the kernels whose arguments this file or a test looks at: they are kept for a replay
std::vector<size_t> argument_sizes(const std::string& name) {
  if (name.find("write_dyn_kernel") != std::string::npos) return {sizeof(DynTable), sizeof(int), sizeof(void*)};
  if (name.find("state_update_kernel") != std::string::npos) return {sizeof(void*), sizeof(void*)};
  return {};
}

void carry_out(const Launch& l) {
  if (l.name.find("write_dyn_kernel") != std::string::npos) {
    const DynTable& t = *static_cast<const DynTable*>(l.args[0]);
    std::memcpy(*static_cast<MatDynamic**>(l.args[2]), t.v, sizeof(MatDynamic) * *static_cast<int*>(l.args[1]));
  }
  if (on_launch) on_launch(l);
}
}  // namespace

std::vector<Array>& arrays() { static std::vector<Array> all; return all; }
void replay() { for (auto& f : recorded) f(); }
void clear_recorded() { recorded.clear(); }
}  // namespace fake

using namespace fake;

extern "C" {
// (a source of the library has a module of its own: its arrays take device memory when something of it is used first)
void** __hipRegisterFatBinary(const void*) { static void* handles[64] = {}; static int n = 0; return &handles[n++]; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void** module, void*, char*, char*, int, size_t bytes, int, int) {
  arrays().push_back({module, bytes});
}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t s) {
  configs.push_back({grid, block, shmem, s});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* s) {
  const Config c = configs.back();
  configs.pop_back();
  *grid = c.grid; *block = c.block; *shmem = c.shmem; *s = c.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t s) {
  const std::string name = names.at(f);
  if (failing(name)) return last = hipErrorLaunchFailure;
  if (!is_captured(s)) { carry_out({name, grid.x, block.x, args}); return hipSuccess; }
  std::vector<std::vector<char>> kept;
  const std::vector<size_t> sizes = argument_sizes(name);
  for (size_t i = 0; i < sizes.size(); ++i)
    kept.emplace_back(static_cast<char*>(args[i]), static_cast<char*>(args[i]) + sizes[i]);
  recorded.push_back([=]() mutable {
    std::vector<void*> a;
    for (auto& k : kept) a.push_back(k.data());
    carry_out({name, grid.x, block.x, a.data()});
  });
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t s) {
  if (failing("copy")) return last = hipErrorInvalidValue;
  auto copy = [=] { std::memcpy(dst, src, n); };
  if (is_captured(s)) recorded.push_back(copy); else copy();
  return hipSuccess;
}
hipError_t hipGetLastError(void) { const hipError_t e = last; last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "a failure of the test's making"; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* out) {
  *out = is_captured(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return capturing ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipExtStreamCreateWithCUMask(hipStream_t* s, uint32_t, const uint32_t*) { return hipStreamCreateWithFlags(s, 0); }
hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipGetDevice(int* d) { ++queries; *d = device; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  ++queries;
  if (failing("attribute")) return last = hipErrorNotInitialized;
  *v = a == hipDeviceAttributeComputeCapabilityMajor ? capability_major
       : a == hipDeviceAttributeComputeCapabilityMinor ? capability_minor : 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static char* scratch = static_cast<char*>(std::aligned_alloc(256, (size_t)32 << 20));
  *p = scratch;
  return hipSuccess;
}
}
