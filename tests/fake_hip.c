/* A HIP runtime of two devices for CPU tests of the library's host code: memory
 * is the host's, kernels do nothing, and every call is checked for the device it
 * is made on.  Loaded (RTLD_GLOBAL) before the library, whose calls then come
 * here.  Streams are the numbers kStream + device; the null stream is the
 * current device's. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

enum { kStream = 0x1000, kOk = 0, kError = 1, kMaxKernels = 256, kLog = 1 << 16 };
typedef struct { unsigned x, y, z; } Dim3;
typedef struct { int device; } Event;

static _Thread_local int current;
static _Thread_local struct { Dim3 grid, block; size_t shared; void *stream; } call;
static struct { const void *fn; const char *name; } kernels[kMaxKernels];
static int n_kernels, n_wrong, n_pinned;
static char launches[kLog], wrong[256];

static int device_of(void *stream) { return stream ? (int)((intptr_t)stream - kStream) : current; }
static void expect(int device, void *stream, const char *what) {
  if (device == device_of(stream)) return;
  __atomic_add_fetch(&n_wrong, 1, __ATOMIC_RELAXED);
  snprintf(wrong, sizeof wrong, "%s: device %d, stream of device %d", what, device, device_of(stream));
}

/* for the tests */
void fake_reset(void) { n_wrong = n_pinned = 0; launches[0] = 0; }
int fake_wrong(void) { return n_wrong; }
const char *fake_wrong_what(void) { return wrong; }
int fake_pinned(void) { return n_pinned; }
const char *fake_launches(void) { return launches; }

/* what the compiler's launch stubs call */
void **__hipRegisterFatBinary(void *image) { static void *handle; handle = image; return &handle; }
void __hipUnregisterFatBinary(void **handle) { (void)handle; }
void __hipRegisterVar(void **h, void *var, char *a, char *b, int c, size_t d, int e, int f) {
  (void)h; (void)var; (void)a; (void)b; (void)c; (void)d; (void)e; (void)f;
}
void __hipRegisterFunction(void **h, const void *fn, char *a, const char *name, unsigned b, void *c,
                           void *d, void *e, void *f, int *g) {
  (void)h; (void)a; (void)b; (void)c; (void)d; (void)e; (void)f; (void)g;
  if (n_kernels < kMaxKernels) { kernels[n_kernels].fn = fn; kernels[n_kernels++].name = name; }
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream) {
  call.grid = grid; call.block = block; call.shared = shared; call.stream = stream;
  return kOk;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream) {
  *grid = call.grid; *block = call.block; *shared = call.shared; *stream = call.stream;
  return kOk;
}
int hipLaunchKernel(const void *fn, Dim3 grid, Dim3 block, void **args, size_t shared, void *stream) {
  (void)args; (void)shared;
  const char *name = "?";
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].fn == fn) name = kernels[i].name;
  expect(current, stream, name);
  static int lock;
  while (__atomic_exchange_n(&lock, 1, __ATOMIC_ACQUIRE)) {}
  const size_t at = strlen(launches);
  if (at + 256 < kLog)
    snprintf(launches + at, kLog - at, "%.200s %u %u %u\n", name, grid.x, grid.y, block.x);
  __atomic_store_n(&lock, 0, __ATOMIC_RELEASE);
  return kOk;
}

/* the runtime calls of the library */
int hipGetDevice(int *d) { *d = current; return kOk; }
int hipSetDevice(int d) { current = d; return kOk; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return kOk; }
int hipGetDevicePropertiesR0600(void *p, int d) { (void)p; (void)d; return kError; }
int hipDeviceSynchronize(void) { return kOk; }
int hipMalloc(void **p, size_t n) { *p = calloc(1, n); return *p ? kOk : kError; }
int hipFree(void *p) { free(p); return kOk; }
int hipHostMalloc(void **p, size_t n, unsigned f) {
  (void)f;
  __atomic_add_fetch(&n_pinned, 1, __ATOMIC_RELAXED);
  return hipMalloc(p, n);
}
int hipHostFree(void *p) { free(p); return kOk; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) {
  (void)k; (void)st;
  memcpy(d, s, n);
  return kOk;
}
int hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)st; memset(d, v, n); return kOk; }
int hipStreamSynchronize(void *s) { (void)s; return kOk; }
int hipEventCreateWithFlags(Event **e, unsigned f) {
  (void)f;
  *e = malloc(sizeof(Event));
  (*e)->device = current;
  return kOk;
}
int hipEventCreate(Event **e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(Event *e) { free(e); return kOk; }
int hipEventRecord(Event *e, void *stream) { expect(e->device, stream, "event"); return kOk; }
int hipEventSynchronize(Event *e) { (void)e; return kOk; }
int hipEventElapsedTime(float *ms, Event *a, Event *b) { (void)a; (void)b; *ms = 0.f; return kOk; }
int hipGetLastError(void) { return kOk; }
const char *hipGetErrorString(int e) { return e ? "error" : "no error"; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; return hipMalloc(p, 1 << 16); }
int hipGraphDestroy(void *g) { (void)g; return kOk; }
int hipGraphExecDestroy(void *g) { (void)g; return kOk; }
