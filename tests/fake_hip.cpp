// A stand-in for the HIP runtime, for host-side tests of libnnp.so on a machine without
// a GPU: device memory is host memory, launches do nothing but what the host's control
// flow turns on (clearing and comparing of the flags, copies of the inputs, gates), and
// a test can make the next allocation, event wait or launch of a named kernel fail.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim3 { uint32_t x, y, z; };
struct Gate { const int* flags; int cap, lcap; };
std::map<const void*, std::string> names;
std::string fail_launch;  // a launch of a kernel of this name fails, once
int fail_malloc = -1, fail_event = -1;  // this many more succeed before one fails (-1: none fails)
int last_error = 0;
std::map<std::string, long> launches;
std::map<std::string, size_t> lds;  // of a kernel's last launch
int* flags = nullptr;               // the handle's pinned flags (the one allocation of 16 bytes)
int rows = 0;                       // longest neighbour row that a build reports
struct Config { Dim3 g, b; size_t lds; void* s; } config;

template <class X> X arg(void** a, int i) { return *static_cast<X*>(a[i]); }
bool once(int& n) { return n >= 0 && n-- == 0; }
}  // namespace

extern "C" {
void fake_fail_launch(const char* name) { fail_launch = name; }
void fake_fail_malloc(int after) { fail_malloc = after; }
void fake_fail_event(int after) { fail_event = after; }
void fake_rows(int n) { rows = n; }
size_t fake_lds(const char* name) {
  for (auto& x : lds)
    if (x.first.find(name) != std::string::npos) return x.second;
  return 0;
}
long fake_launches(const char* name) {
  long n = 0;
  for (auto& x : launches)
    if (x.first.find(name) != std::string::npos) n += x.second;
  return n;
}

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void* s) { config = {g, b, lds, s}; return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* lds, void** s) {
  *g = config.g, *b = config.b, *lds = config.lds, *s = config.s;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3, Dim3, void** a, size_t shared, void*) {
  const std::string& k = names[f];
  auto is = [&](const char* name) { return k.find(name) != std::string::npos; };
  if (!fail_launch.empty() && is(fail_launch.c_str())) {
    fail_launch.clear();
    return last_error = 719;
  }
  ++launches[k];
  lds[k] = shared;
  if (is("k_max_count") || is("k_mlp")) flags[2] = rows;
  if (is("k_sort_small")) std::memset(arg<int*>(a, 14), 0, 5 * sizeof(int));
  if (is("k_copy_inputs")) {  // FP64
    const int64_t n = arg<int64_t>(a, 0);
    std::memcpy(arg<void*>(a, 3), arg<void*>(a, 1), n * 24);
    std::memcpy(arg<void*>(a, 4), arg<void*>(a, 2), n * 4);
  }
  if (is("k_same_inputs")) {
    const int64_t n = arg<int64_t>(a, 0);
    if (std::memcmp(arg<void*>(a, 1), arg<void*>(a, 2), n * 24) || std::memcmp(arg<void*>(a, 3), arg<void*>(a, 4), n * 4))
      *arg<int*>(a, 5) = *arg<int*>(a, 6) = 1;
  }
  if (is("k_wgrad_final")) {
    const Gate g = arg<Gate>(a, 7);
    const bool closed = g.flags && (((g.flags[0] & 7) | g.flags[3]) != 0 || g.flags[1] > g.cap || g.flags[2] > g.lcap);
    if (!closed)
      for (int64_t i = 0; i < arg<int64_t>(a, 0); ++i) arg<double*>(a, 6)[i] = 1.0;
  }
  return 0;
}

int hipMalloc(void** p, size_t n) {
  if (once(fail_malloc)) return 2;
  return (*p = std::calloc(n, 1)) ? 0 : 2;
}
int hipFree(void* p) { std::free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(n, 1);
  if (n == 16) flags = static_cast<int*>(*p);
  return *p ? 0 : 2;
}
int hipHostFree(void* p) { std::free(p); return 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { std::memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { std::memcpy(d, s, n); return 0; }
int hipGetSymbolAddress(void** p, const void*) { static char c[16]; *p = c; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 160 * 1024; return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipEventCreate(void** e) { *e = std::malloc(1); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void* e) { std::free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return once(fail_event) ? 719 : 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0.f; return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "forced by the test"; }
}
