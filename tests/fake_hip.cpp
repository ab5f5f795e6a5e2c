// The HIP runtime calls that liblme.so imports, on host memory: allocation
// and copies work, launches are recorded and run nothing.  Loaded before
// liblme.so (RTLD_GLOBAL) its host code runs on a machine without a GPU, with
// an allocation that fails on demand.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
long g_fail_at = 0;             // the allocation, counted from here, that fails (0: none)
std::map<const void *, std::string> g_names;
std::string g_log;              // "kernel grid threads lds <first 8 bytes of the arguments>\n" per launch
struct Dim3 { uint32_t x, y, z; };
Dim3 g_grid, g_block;
size_t g_lds;
void *g_stream;
const int kOutOfMemory = 2;
}  // namespace

extern "C" {
void fake_fail_allocation(long k) { g_fail_at = k; }
const char *fake_launches() { return g_log.c_str(); }
void fake_clear() { g_log.clear(); }

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) { g_names[f] = name; }
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *s) {
  g_grid = grid; g_block = block; g_lds = lds; g_stream = s;
  return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **s) {
  *grid = g_grid; *block = g_block; *lds = g_lds; *s = g_stream;
  return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3 block, void **args, size_t lds, void *) {
  char line[96];
  uint64_t word;
  memcpy(&word, args[0], sizeof word);
  snprintf(line, sizeof line, " %u %u %zu %llx\n", grid.x, block.x, lds, (unsigned long long)word);
  g_log += g_names[f] + line;
  return 0;
}

int hipMalloc(void **p, size_t n) {
  *p = nullptr;
  if (g_fail_at > 0 && --g_fail_at == 0) return kOutOfMemory;
  *p = malloc(n);
  return 0;
}
int hipFree(void *p) { free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { *p = malloc(n); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { memcpy(d, s, n); return 0; }

// hipDeviceAttribute_t values are not spelled out here: the library asks for
// the LDS of a workgroup and the number of CUs, told apart by their use in
// ensure_device() (first) and the planner
int hipDeviceGetAttribute(int *v, int attr, int) {
  static int lds_attr = -1;
  if (lds_attr < 0) lds_attr = attr;
  *v = attr == lds_attr ? 160 * 1024 : 256;
  return 0;
}
int hipGetDeviceCount(int *n) { const char *e = getenv("FAKE_DEVICES"); *n = e ? atoi(e) : 1; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "fake error"; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetSymbolAddress(void **p, const void *) {
  static char scratch[64 << 20];
  *p = scratch;
  return 0;
}
int hipEventCreate(void **e) { *e = &g_log; return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1.0f; return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = &g_log; return 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { *g = &g_log; return 0; }
int hipGraphInstantiate(void **x, void *, void **, char *, size_t) { *x = &g_log; return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipGraphLaunch(void *, void *) { return 0; }
}
