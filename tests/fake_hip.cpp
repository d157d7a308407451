// Stand-in for the HIP runtime: "device" memory is host memory, a kernel
// launch does nothing but leave a line in the log.  Loaded into a process with
// RTLD_GLOBAL before libgwl.so, it takes the library's HIP calls, so that the
// host side (allocation, growth, failure paths, choice of kernels and launch
// arguments) can be tested without a GPU.  Results are meaningless.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 {
  unsigned x, y, z;
};
std::map<const void*, std::string> kernels;
std::map<void*, size_t> blocks;  // live allocations
std::string log_text;
long n_malloc = 0, fail_malloc = -1, n_event = 0, fail_event = -1;
size_t live = 0, limit = SIZE_MAX;
bool unsynced = false;  // a fill on the null stream that nothing has waited for
int last_error = 0;
Dim3 cfg_grid, cfg_block;
size_t cfg_shmem;
void* cfg_stream;
std::string watch_kernel;
int watch_arg = -1;
long watch_n = 0;
double watch_max = -1.0;
int error(int e) { return last_error = e; }
}  // namespace

extern "C" {
// ---- controls
void fake_reset() {
  log_text.clear();
  n_malloc = n_event = 0;
  fail_malloc = fail_event = -1;
  limit = SIZE_MAX;
  watch_max = -1.0;
}
void fake_fail_malloc(long k) { fail_malloc = n_malloc + k; }  // the k-th from now on (0 = next)
void fake_fail_event(long k) { fail_event = n_event + k; }
void fake_limit(size_t bytes) { limit = bytes; }
size_t fake_live() { return live; }
long fake_mallocs() { return n_malloc; }
int fake_unsynced() { return unsynced; }
const char* fake_log() { return log_text.c_str(); }
// largest |value| among the first n doubles behind pointer argument `arg` at the launches of `kernel`
void fake_watch(const char* kernel, int arg, long n) {
  watch_kernel = kernel;
  watch_arg = arg;
  watch_n = n;
  watch_max = -1.0;
}
double fake_watched() { return watch_max; }

// ---- memory
int hipMalloc(void** p, size_t n) {
  *p = nullptr;
  const long k = n_malloc++;
  if (k == fail_malloc || live + n > limit) return error(2);  // hipErrorOutOfMemory
  *p = aligned_alloc(256, (n + 255) / 256 * 256);
  blocks[*p] = n;
  live += n;
  return 0;
}
int hipFree(void* p) {
  auto it = blocks.find(p);
  if (it == blocks.end()) return error(1);
  live -= it->second;
  blocks.erase(it);
  free(p);
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
int hipHostFree(void* p) { return hipFree(p); }
int hipMemset(void* p, int v, size_t n) {
  if (!p) return error(1);
  memset(p, v, n);
  unsynced = true;
  return 0;
}
int hipMemsetAsync(void* p, int v, size_t n, void*) {
  if (!p) return error(1);
  memset(p, v, n);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  if (n && (!d || !s)) return error(1);
  memmove(d, s, n);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void*) { return hipMemcpy(d, s, n, k); }
int hipPointerGetAttributes(void* a, const void*) {
  memset(a, 0, 32);  // type 0: hipMemoryTypeUnregistered
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  static std::vector<char> sym(64 << 20);
  *p = sym.data();
  return 0;
}

// ---- device, streams, events
int hipGetDevice(int* d) { return *d = 0; }
int hipDeviceSynchronize() {
  unsynced = false;
  return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) {
  *s = malloc(1);
  return 0;
}
int hipStreamDestroy(void* s) {
  free(s);
  return 0;
}
int hipStreamSynchronize(void*) { return 0; }
int hipEventCreateWithFlags(void** e, unsigned) {
  if (n_event++ == fail_event) return error(2);
  *e = malloc(1);
  return 0;
}
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void* e) {
  free(e);
  return 0;
}
int hipEventRecord(void* e, void*) { return e ? 0 : error(400); }  // hipErrorInvalidHandle
int hipEventSynchronize(void* e) { return e ? 0 : error(400); }
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 1.0f;
  return 0;
}
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) {
  *g = malloc(1);
  return 0;
}
int hipGraphInstantiate(void** x, void*, void*, char*, size_t) {
  *x = malloc(1);
  return 0;
}
int hipGraphDestroy(void* g) {
  free(g);
  return 0;
}
int hipGraphExecDestroy(void* g) {
  free(g);
  return 0;
}
int hipGraphLaunch(void*, void*) { return 0; }
int hipGetLastError() {
  const int e = last_error;
  last_error = 0;
  return e;
}
const char* hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }

// ---- kernels
void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t sh, void* st) {
  cfg_grid = g;
  cfg_block = b;
  cfg_shmem = sh;
  cfg_stream = st;
  return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* sh, void** st) {
  *g = cfg_grid;
  *b = cfg_block;
  *sh = cfg_shmem;
  *st = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void** args, size_t, void*) {
  const std::string& name = kernels[f];
  log_text += name + " " + std::to_string(g.x) + " " + std::to_string(g.y) + " " + std::to_string(b.x);
  const bool pd = name.find("gemm2_pd_kernel") != std::string::npos;
  if (pd || name.find("gemm2_f64m_kernel") != std::string::npos ||
      name.find("gemm2_f16_n") != std::string::npos) {  // split, points per part
    const int k = pd ? 5 : 2;
    log_text += " split " + std::to_string(*(int*)args[k]) + " " + std::to_string(*(int*)args[k + 1]);
  }
  log_text += unsynced ? " unsynced\n" : "\n";
  if (!watch_kernel.empty() && name.find(watch_kernel) != std::string::npos) {
    const double* p = *(const double**)args[watch_arg];
    for (long i = 0; i < watch_n; ++i) {
      const double v = p[i] < 0 ? -p[i] : p[i];
      if (v > watch_max) watch_max = v;
    }
  }
  return 0;
}
}
