/* A stand-in for the HIP runtime on a machine without a GPU: every call libtrack makes
 * succeeds without doing anything, is written to a log, and can be made to fail as the
 * runtime fails (the status returned and left as the last error).  Loaded with global
 * visibility before libtrack.so, whose calls then bind to it. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef int hipError_t;
typedef struct { uint32_t x, y, z; } dim3_t;

static char* g_log;
static size_t g_len, g_cap;
static struct { const void* fn; const char* name; } g_fns[4096];
static int g_nfns;
static hipError_t g_last;
static char g_fail_name[64];
static int g_fail_count, g_handles;

static void say(const char* op, const char* what, const void* where) {
  const size_t need = g_len + strlen(op) + strlen(what) + 64;
  if (need > g_cap) {
    g_cap = 2 * need;
    g_log = (char*)realloc(g_log, g_cap);
  }
  g_len += (size_t)sprintf(g_log + g_len, "%s %s %lx\n", op, what, (unsigned long)where);
}

const char* fake_log(void) { return g_log ? g_log : ""; }
void fake_clear(void) {
  g_len = 0;
  if (g_log) g_log[0] = 0;
}
/* the next `count` calls of `name` fail */
void fake_fail(const char* name, int count) {
  snprintf(g_fail_name, sizeof(g_fail_name), "%s", name);
  g_fail_count = count;
}

static hipError_t status(const char* name) {
  if (g_fail_count > 0 && strcmp(name, g_fail_name) == 0) {
    --g_fail_count;
    return g_last = 1;
  }
  return 0;
}
static void* handle(void) { return (void*)(uintptr_t)(0x1000 + 16 * ++g_handles); }

void* __hipRegisterFatBinary(const void* p) { return (void*)p; }
void __hipUnregisterFatBinary(void* p) { (void)p; }
void __hipRegisterFunction(void* m, const void* host, char* dev, const char* name, unsigned lim, void* a, void* b,
                           void* c, void* d, int* w) {
  if (g_nfns < 4096) {
    g_fns[g_nfns].fn = host;
    g_fns[g_nfns++].name = name;
  }
}
void __hipRegisterVar(void* m, void* v, char* h, char* d, int e, size_t s, int c, int g) {}

static struct { dim3_t g, b; size_t sh; void* st; } g_cfg;
hipError_t __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void* st) {
  g_cfg.g = g, g_cfg.b = b, g_cfg.sh = sh, g_cfg.st = st;
  return 0;
}
hipError_t __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* sh, void** st) {
  *g = g_cfg.g, *b = g_cfg.b, *sh = g_cfg.sh, *st = g_cfg.st;
  return 0;
}
hipError_t hipLaunchKernel(const void* fn, dim3_t g, dim3_t b, void** args, size_t sh, void* st) {
  const char* name = "?";
  for (int i = 0; i < g_nfns; ++i)
    if (g_fns[i].fn == fn) name = g_fns[i].name;
  say("launch", name, st);
  if (g.x > 0x7fffffffu || g.y > 65535 || g.z > 65535 || (uint64_t)g.x * b.x > 0xffffffffu) return g_last = 9;
  return status("hipLaunchKernel");
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return status("hipGetDevice");
}
hipError_t hipDeviceGetAttribute(int* v, int attr, int dev) {
  *v = 256;
  return 0;
}
hipError_t hipDeviceSynchronize(void) { return 0; }
hipError_t hipGetLastError(void) {
  const hipError_t e = g_last;
  g_last = 0;
  return e;
}
const char* hipGetErrorString(hipError_t e) { return e ? "made to fail" : "no error"; }
hipError_t hipEventCreate(void** e) {
  *e = handle();
  return status("hipEventCreate");
}
hipError_t hipEventCreateWithFlags(void** e, unsigned f) {
  const hipError_t st = status("hipEventCreateWithFlags");
  if (!st) *e = handle();
  return st;
}
hipError_t hipEventDestroy(void* e) { return 0; }
hipError_t hipEventElapsedTime(float* ms, void* a, void* b) {
  *ms = 0;
  return 0;
}
hipError_t hipEventRecord(void* e, void* st) {
  say("record", "-", st);
  return status("hipEventRecord");
}
hipError_t hipStreamWaitEvent(void* st, void* e, unsigned f) {
  say("wait", "-", st);
  return status("hipStreamWaitEvent");
}
hipError_t hipStreamCreateWithFlags(void** st, unsigned f) {
  const hipError_t e = status("hipStreamCreateWithFlags");
  if (!e) *st = handle();
  return e;
}
hipError_t hipStreamDestroy(void* st) { return 0; }
hipError_t hipStreamIsCapturing(void* st, int* s) {
  *s = 0;
  return status("hipStreamIsCapturing");
}
hipError_t hipStreamSynchronize(void* st) {
  say("sync", "-", st);
  return status("hipStreamSynchronize");
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) {
  say("copy", "-", d);
  return status("hipMemcpyAsync");
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned f) {
  const hipError_t e = status("hipHostMalloc");
  say("hostmalloc", "-", 0);
  if (!e) *p = calloc(1, n);
  return e;
}
hipError_t hipHostFree(void* p) {
  free(p);
  return 0;
}
hipError_t hipGetSymbolAddress(void** p, const void* sym) {
  *p = handle();
  return 0;
}
