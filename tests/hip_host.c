/* A HIP runtime without a device for CPU tests of the library's host paths: device memory is host memory,
 * kernels do nothing, streams and events complete at once.  Loaded globally before libcopse.so, its functions
 * stand in for the runtime's.  It counts what the tests ask about: kernel launches, device bytes, and copies
 * between device and pageable host memory since the last wait for a stream.  Limits are set from the test. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef int err;
enum { OK = 0, OUT_OF_MEMORY = 2 };
typedef struct { uint32_t x, y, z; } dim;

static size_t live, peak, limit = (size_t)-1;
static int launches, pending, no_pinned;
static void (*pause_in_event_wait)(void);

void host_set_limit(size_t bytes) { limit = bytes; }
void host_set_no_pinned(int on) { no_pinned = on; }
void host_set_event_wait(void (*f)(void)) { pause_in_event_wait = f; }
size_t host_live(void) { return live; }
size_t host_peak(int reset) {
  size_t p = peak;
  if (reset) peak = live;
  return p;
}
int host_launches(void) { return launches; }
int host_pending(void) { return pending; }

/* every block carries its size in front of it; pinned blocks lie in a list of few */
static struct { char *p; size_t n; } pinned[64];
static int is_pinned(const void *p) {
  for (int i = 0; i < 64; ++i)
    if (pinned[i].p && (const char *)p >= pinned[i].p && (const char *)p < pinned[i].p + pinned[i].n) return 1;
  return 0;
}

err hipMalloc(void **p, size_t n) {
  *p = NULL;
  if (live + n > limit) return OUT_OF_MEMORY;
  size_t *b = calloc(1, n + 64);
  if (!b) return OUT_OF_MEMORY;
  *b = n;
  *p = (char *)b + 64;
  live += n;
  if (live > peak) peak = live;
  return OK;
}
err hipFree(void *p) {
  if (!p) return OK;
  size_t *b = (size_t *)((char *)p - 64);
  live -= *b;
  free(b);
  return OK;
}
err hipHostMalloc(void **p, size_t n, unsigned flags) {
  (void)flags;
  *p = NULL;
  if (no_pinned) return OUT_OF_MEMORY;
  for (int i = 0; i < 64; ++i)
    if (!pinned[i].p) {
      *p = pinned[i].p = calloc(1, n);
      pinned[i].n = n;
      return OK;
    }
  return OUT_OF_MEMORY;
}
err hipHostFree(void *p) {
  for (int i = 0; i < 64; ++i)
    if (p && pinned[i].p == p) pinned[i].p = NULL;
  free(p);
  return OK;
}
err hipMemcpy(void *d, const void *s, size_t n, int kind) {
  (void)kind;
  memcpy(d, s, n);
  return OK;
}
err hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
  (void)st;
  memcpy(d, s, n);
  if ((kind == 1 && !is_pinned(s)) || (kind == 2 && !is_pinned(d))) ++pending;
  return OK;
}
err hipMemsetAsync(void *d, int v, size_t n, void *st) {
  (void)st;
  memset(d, v, n);
  return OK;
}
err hipStreamSynchronize(void *s) {
  (void)s;
  pending = 0;
  return OK;
}
err hipEventSynchronize(void *e) {
  (void)e;
  if (pause_in_event_wait) pause_in_event_wait();
  return OK;
}
err hipLaunchKernel(const void *f, dim g, dim b, void **args, size_t lds, void *s) {
  (void)f, (void)g, (void)b, (void)args, (void)lds, (void)s;
  ++launches;
  return OK;
}

static dim call_grid, call_block;
static size_t call_lds;
static void *call_stream;
err __hipPushCallConfiguration(dim g, dim b, size_t lds, void *s) {
  call_grid = g, call_block = b, call_lds = lds, call_stream = s;
  return OK;
}
err __hipPopCallConfiguration(dim *g, dim *b, size_t *lds, void **s) {
  *g = call_grid, *b = call_block, *lds = call_lds, *s = call_stream;
  return OK;
}
static char handle[64];
err hipGetSymbolAddress(void **p, const void *sym) { (void)sym; *p = handle; return OK; }
err hipEventCreate(void **e) { *e = handle; return OK; }
err hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = handle; return OK; }
err hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = handle; return OK; }
err hipEventElapsedTime(float *ms, void *a, void *b) { (void)a, (void)b; *ms = 0; return OK; }
err hipEventDestroy(void *e) { (void)e; return OK; }
err hipEventQuery(void *e) { (void)e; return OK; }
err hipEventRecord(void *e, void *s) { (void)e, (void)s; return OK; }
err hipStreamDestroy(void *s) { (void)s; return OK; }
err hipSetDevice(int d) { (void)d; return OK; }
err hipGetLastError(void) { return OK; }
const char *hipGetErrorString(err e) { return e == OUT_OF_MEMORY ? "out of memory" : "no error"; }
