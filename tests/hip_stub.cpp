// A HIP runtime for host-logic tests on a machine without a GPU: device memory is host memory,
// copies are memcpy, kernels do nothing (a value handed to the waiting host arrives, unless held
// back or late) and every launch is logged by name.  Failures of chosen calls are injected.
#include <chrono>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <thread>

namespace {
struct Dim3 {
  uint32_t x, y, z;
};
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::string log_text;
int last_error = 0;
// calls until one fails, < 0: none
int fail_malloc = -1, fail_host_malloc = -1;
std::string fail_kernel;   // a launch whose name contains it fails, once
int hold_values = 0, late_ms = 0;
std::chrono::steady_clock::time_point done;   // when the stream's work has ended
int syncs = 0, null_writes = 0;
int dirty_counts = 0;   // histograms begun on counts that were not clear
Dim3 cfg_grid, cfg_block;
size_t cfg_shmem;
void* cfg_stream;

bool due(int& n) { return n >= 0 && n-- == 0; }
bool bad(const void* p) { return reinterpret_cast<uintptr_t>(p) < (1u << 20); }
}  // namespace

extern "C" {
// ---- control
void stub_fail_malloc(int n) { fail_malloc = n; }
void stub_fail_host_malloc(int n) { fail_host_malloc = n; }
void stub_fail_kernel(const char* name) { fail_kernel = name; }
void stub_hold_values(int on) { hold_values = on; }
void stub_late_values(int ms) { late_ms = ms; }
int stub_syncs() { return syncs; }
int stub_null_writes() { return null_writes; }
int stub_dirty_counts() { return dirty_counts; }
const char* stub_log() { return log_text.c_str(); }
void stub_clear_log() { log_text.clear(); }

// ---- runtime
int hipMalloc(void** p, size_t n) {
  if (due(fail_malloc)) return last_error = 2;
  *p = std::calloc(1, n ? n : 1);
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
  if (due(fail_host_malloc)) return last_error = 2;
  *p = std::calloc(1, n ? n : 1);
  return 0;
}
int hipFree(void* p) {
  std::free(p);
  return 0;
}
int hipHostFree(void* p) {
  std::free(p);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  if (bad(d) || bad(s)) {
    ++null_writes;
    return last_error = 1;
  }
  std::memmove(d, s, n);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void*) {
  return hipMemcpy(d, s, n, kind);
}
int hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void*) { return hipMemset(d, v, n); }
int hipMemGetInfo(size_t* f, size_t* t) {
  *f = *t = size_t{1} << 32;
  return 0;
}
int hipGetLastError() {
  const int e = last_error;
  last_error = 0;
  return e;
}
const char* hipGetErrorString(int e) { return e ? "injected" : "no error"; }
int hipStreamSynchronize(void*) {
  ++syncs;
  std::this_thread::sleep_until(done);
  return 0;
}
int hipDeviceSynchronize() { return 0; }
int hipStreamQuery(void*) { return std::chrono::steady_clock::now() < done ? 600 : 0; }
int hipStreamIsCapturing(void*, int* c) {
  *c = 0;
  return 0;
}
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipEventCreate(void** e) {
  *e = std::malloc(1);
  return 0;
}
int hipEventDestroy(void* e) {
  std::free(e);
  return 0;
}
int hipEventRecord(void*, void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 0;
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  *p = std::calloc(1, 1 << 20);
  return 0;
}
void** __hipRegisterFatBinary(const void*) {
  static void* h = nullptr;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shmem, void* stream) {
  cfg_grid = g;
  cfg_block = b;
  cfg_shmem = shmem;
  cfg_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* shmem, void** stream) {
  *g = cfg_grid;
  *b = cfg_block;
  *shmem = cfg_shmem;
  *stream = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3, void** args, size_t, void*) {
  const std::string& name = names()[f];
  const auto is = [&](const char* k) { return name.find(k) != std::string::npos; };
  const auto pointer = [&](int i) { return *static_cast<char**>(args[i]); };
  if (!fail_kernel.empty() && is(fail_kernel.c_str())) {
    log_text += "failed " + name + "\n";
    fail_kernel.clear();
    return last_error = 1;
  }
  log_text += name + "\n";
  // the bin counts: a histogram starts from zeros and leaves some, the bin sort clears them
  const int counts = is("hist_kernel") ? 1 : (is("kick_drift_kernel") ? 11 : -1);
  if (counts >= 0 && pointer(counts)) {
    uint32_t* c = reinterpret_cast<uint32_t*>(pointer(counts));
    if (c[0] != 0) ++dirty_counts;
    c[0] = 1;
  }
  if (is("bin_sort_gather_kernel")) reinterpret_cast<uint32_t*>(pointer(5))[0] = 0;
  if (is("fill_kernel")) {   // p, v, count
    char* p = pointer(0);
    if (bad(p)) {
      ++null_writes;
    } else {
      float v = *static_cast<float*>(args[1]);
      const long long n = *static_cast<long long*>(args[2]);
      for (long long i = 0; i < n; ++i) std::memcpy(p + 4 * i, &v, 4);
    }
  }
  if ((is("reduce_kernel") || is("reduce_to_host_kernel")) && (bad(pointer(0)) || bad(pointer(3))))
    ++null_writes;   // in, count, stride, out
  if (is("reduce_to_host_kernel") && !hold_values) {           // in, count, stride, out, seq
    char* out = pointer(3);
    const uint64_t seq = *static_cast<uint64_t*>(args[4]);
    done = std::chrono::steady_clock::now() + std::chrono::milliseconds(late_ms);
    const auto arrive = [out, seq, n = grid.x] {
      std::this_thread::sleep_until(done - std::chrono::milliseconds(20));
      for (uint32_t v = 0; v < n; ++v) {
        const double one = 1.0;
        std::memcpy(out + 16 * v, &one, 8);
        __atomic_store_n(reinterpret_cast<uint64_t*>(out + 16 * v + 8), seq, __ATOMIC_RELEASE);
      }
    };
    if (late_ms)
      std::thread(arrive).detach();
    else
      arrive();
  }
  return 0;
}
}
