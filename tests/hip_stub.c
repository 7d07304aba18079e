/* A host stand-in for the HIP calls libvla.so makes: "device" memory is host memory, kernels do nothing, and the
 * calls that order work on the device are logged, one per line.  Loaded before the library, with global symbols,
 * it lets the host code's order of launches, events and synchronisations be read without a GPU. */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;
typedef int (*sync_fn)(void);

static char log_buf[1 << 20];
static size_t log_len;
static int n_events;
static int capture_status, capture_error;   /* what hipStreamIsCapturing reports */
static int device;
static sync_fn on_sync;                     /* called once, inside the next hipDeviceSynchronize */

static void note(const char* what, void* stream, void* event) {
  if (log_len + 64 < sizeof log_buf)
    log_len += (size_t)snprintf(log_buf + log_len, sizeof log_buf - log_len, "%s %lx %lx\n", what, (long)stream, (long)event);
}

const char* stub_log(void) { return log_buf; }
void stub_clear(void) { log_len = 0; log_buf[0] = 0; }
void stub_capture(int status, int error) { capture_status = status; capture_error = error; }
void stub_device(int d) { device = d; }
void stub_on_sync(sync_fn f) { on_sync = f; }

int hipMalloc(void** p, size_t n) { *p = aligned_alloc(256, (n + 255) / 256 * 256); return *p ? 0 : 2; }
int hipFree(void* p) { free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; return hipMalloc(p, n); }
int hipHostFree(void* p) { return hipFree(p); }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) {
  (void)d; (void)s; (void)n; (void)k; (void)st;   /* the error word of a kernel that did not run */
  return 0;
}
int hipMemcpy2D(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, int k) {
  (void)k;
  for (size_t i = 0; i < h; ++i) memcpy((char*)d + i * dp, (const char*)s + i * sp, w);
  return 0;
}
int hipMemset(void* p, int v, size_t n) { memset(p, v, n); return 0; }
int hipMemsetAsync(void* p, int v, size_t n, void* st) { (void)st; return hipMemset(p, v, n); }
int hipGetLastError(void) { return 0; }
int hipGetDevice(int* d) { *d = device; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t l) {
  (void)f; (void)b; (void)l;
  *n = 1;
  return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = (void*)0x5; return 0; }
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipStreamIsCapturing(void* s, int* st) { (void)s; *st = capture_status; return capture_error; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = (void*)(long)(0xe0 + n_events++); return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* s) { note("record", s, e); return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)f; note("wait", s, e); return 0; }
int hipDeviceSynchronize(void) {
  note("sync", 0, 0);
  if (on_sync) {
    sync_fn f = on_sync;
    on_sync = 0;
    return f();
  }
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds, void* s) {
  (void)f; (void)args; (void)block;
  /* the persistent kernel: a workgroup for every compute unit, most of its LDS */
  note(grid.x * grid.y * grid.z == 256 && lds >= (100u << 10) ? "persist" : "kernel", s, 0);
  return 0;
}
static struct { dim3_t grid, block; size_t lds; void* s; } cfg;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* s) {
  cfg.grid = grid; cfg.block = block; cfg.lds = lds; cfg.s = s;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** s) {
  *grid = cfg.grid; *block = cfg.block; *lds = cfg.lds; *s = cfg.s;
  return 0;
}
