// Stands in for the HIP runtime and the range markers in a process that has no
// GPU: every call the library makes is taken down, in order, and nothing runs.
// Device memory is host memory; kernels are known by the names they are
// registered under.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim3 {
  uint32_t x, y, z;
};
std::map<const void *, std::string> &kernels() {
  static std::map<const void *, std::string> m;
  return m;
}
FILE *out() {
  static FILE *f = fopen(getenv("HOST_TRACE"), "w");
  return f;
}
void say(const char *what, const char *arg = "") {
  fprintf(out(), "%s %s\n", what, arg);
  fflush(out());
}
Dim3 g_grid, g_block;
size_t g_shared;
void *g_stream;
}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
  kernels()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream) {
  g_grid = grid, g_block = block, g_shared = shared, g_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream) {
  *grid = g_grid, *block = g_block, *shared = g_shared, *stream = g_stream;
  return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3, void **, size_t, void *) {
  if (grid.x == 0) return 1;
  say("launch", kernels()[f].c_str());
  return 0;
}
int hipGetDeviceCount(int *n) { return *n = 1, 0; }
int hipGetDevice(int *d) { return *d = 0, 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, 0; }
int hipDeviceSynchronize() { return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "error"; }
int hipMalloc(void **p, size_t n) { return *p = calloc(1, n ? n : 1), 0; }
int hipFree(void *p) { return free(p), 0; }
int hipMemset(void *p, int v, size_t n) { return memset(p, v, n), 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { return memcpy(d, s, n), 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { return memcpy(d, s, n), 0; }
int hipGetSymbolAddress(void **p, const void *) {
  static char *mem = static_cast<char *>(calloc(1, 80u << 20));
  return *p = mem, 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  return *n = 4, 0;
}
int hipStreamCreateWithFlags(void **s, unsigned) { return say("stream"), *s = malloc(1), 0; }
int hipStreamDestroy(void *s) { return free(s), 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipEventCreate(void **e) { return *e = malloc(1), 0; }
int hipEventCreateWithFlags(void **e, unsigned) { return say("event"), *e = malloc(1), 0; }
int hipEventDestroy(void *e) { return free(e), 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { return *ms = 0.001f, 0; }
int roctxRangePushA(const char *name) { return say("push", name), 0; }
int roctxRangePop() { return say("pop"), 0; }
void hostTraceMark(const char *what) { say("mark", what); }
}
