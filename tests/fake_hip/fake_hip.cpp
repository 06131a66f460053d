// A stand-in for the HIP runtime calls that a forward call makes, for tests of
// the host side on machines without a GPU: no kernel runs and no device memory
// exists.  Loaded with RTLD_GLOBAL before libsats.so, it takes the calls that it
// defines; every one of them is written to a log, a line each.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim {
  uint32_t x, y, z;
};
constexpr int kOutOfMemory = 2, kCaptureUnsupported = 900;
std::map<const void *, std::string> g_kernels;  // host function -> device name
std::map<void *, size_t> g_live;
std::string g_log;
size_t g_limit = SIZE_MAX, g_held = 0;
uintptr_t g_next = (uintptr_t)1 << 40;
int g_capturing = 0, g_device_queries = 0;
Dim g_grid, g_block;
size_t g_shared;
void *g_stream;

void line(const char *what, unsigned long long a = 0, unsigned long long b = 0) {
  char s[160];
  snprintf(s, sizeof s, "%s %llx %llu\n", what, a, b);
  g_log += s;
}
// `launch NAME GRIDxGRIDy` and the first argument's bytes from offset 0 on, as hex pointers of 8 bytes
int launch(const void *f, Dim grid) {
  const auto it = g_kernels.find(f);
  g_log += "launch " + (it == g_kernels.end() ? std::string("?") : it->second) + " " + std::to_string(grid.x) + "x" +
           std::to_string(grid.y) + "\n";
  return 0;
}
}  // namespace

extern "C" {
// control
void fake_limit(size_t bytes) { g_limit = bytes; }
void fake_capture(int on) { g_capturing = on; }
size_t fake_held() { return g_held; }
int fake_queries() { return g_device_queries; }
const char *fake_log() { return g_log.c_str(); }
void fake_clear() {
  g_log.clear();
  g_device_queries = 0;
}

// registration of the library's kernels
void **__hipRegisterFatBinary(const void *) {
  static void *h;
  return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
  g_kernels[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

// launches
int __hipPushCallConfiguration(Dim grid, Dim block, size_t shared, void *stream) {
  g_grid = grid, g_block = block, g_shared = shared, g_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *shared, void **stream) {
  *grid = g_grid, *block = g_block, *shared = g_shared, *stream = g_stream;
  return 0;
}
int hipLaunchKernel(const void *f, Dim grid, Dim, void **, size_t, void *) { return launch(f, grid); }
int hipExtLaunchKernel(const void *f, Dim grid, Dim, void **, size_t, void *, void *, void *, int) {
  return launch(f, grid);
}

// device and memory
int hipGetDevice(int *d) {
  *d = 0;
  return 0;
}
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int *v, int, int) {
  ++g_device_queries;
  *v = 256;  // compute units
  return 0;
}
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "fake"; }
int hipMalloc(void **p, size_t n) {
  *p = nullptr;
  if (g_capturing || g_held + n > g_limit) {
    line("malloc-failed", 0, n);
    return g_capturing ? kCaptureUnsupported : kOutOfMemory;
  }
  *p = reinterpret_cast<void *>(g_next);
  g_next += (n + 4095) / 4096 * 4096;
  g_live[*p] = n;
  g_held += n;
  line("malloc", (unsigned long long)*p, n);
  return 0;
}
int hipFree(void *p) {
  const auto it = g_live.find(p);
  if (it == g_live.end()) return 1;
  line("free", (unsigned long long)p, it->second);
  g_held -= it->second;
  g_live.erase(it);
  return 0;
}
int hipStreamSynchronize(void *) {
  line("sync");
  return g_capturing ? kCaptureUnsupported : 0;
}
int hipDeviceSynchronize() {
  line("device-sync");
  return 0;
}
int hipStreamIsCapturing(void *, int *st) {
  *st = g_capturing;
  return 0;
}
int hipMemsetAsync(void *p, int, size_t n, void *) {
  line("memset", (unsigned long long)p, n);
  return 0;
}
int hipGetSymbolAddress(void **p, const void *) {
  *p = reinterpret_cast<void *>((uintptr_t)1 << 36);
  return 0;
}
}
