/* A HIP runtime without a device, for tests of the library's host code: loaded
 * with its symbols global before libpasur.so, whose calls it then takes.  Device
 * memory is host memory, kernels do nothing, and work counts as pending on the
 * device from a launch to the next wait.  What a test sets and reads is in
 * `fake`. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } Dim3;

enum { MAX_EVENTS = 65536 };
struct {
  int free_status;      /* what hipFree returns, freeing nothing unless 0 */
  int sync_status;      /* what hipStreamSynchronize returns */
  int last_error;       /* what the next hipGetLastError returns */
  int failing_mallocs;  /* so many hipMallocs fail */
  int failing_after;    /* after so many that don't */
  int device;           /* the current device */
  int capturing;        /* what hipStreamIsCapturing reports */
  int pending;          /* launches since the last wait */
  int freed_pending;    /* hipFrees of memory while work was pending */
  int mallocs, frees, host_mallocs, syncs, launches, mallocs_async, frees_async;
  int unfinished;       /* events have not ended yet */
  int event_waits;      /* hipStreamWaitEvents */
  int64_t free_bytes[2], total_bytes[2];  /* per device */
  const void *copy_from;  /* where copies of copy_bytes bytes to the host come from */
  int64_t copy_bytes;
  int64_t words[31];    /* what the kernels report in the library's host words */
  void (*in_sync)(void);  /* called before a wait ends */
  void (*in_free)(void);  /* called by hipFree */
} fake;

static int64_t *host_words[64];
static int n_host_words;

int hipMalloc(void **p, size_t bytes) {
  *p = 0;
  if (fake.failing_mallocs > 0 && fake.failing_after-- <= 0) {
    fake.failing_after = 0;
    --fake.failing_mallocs;
    fake.last_error = 2;
    return 2;
  }
  ++fake.mallocs;
  *p = aligned_alloc(4096, (bytes + 4095) / 4096 * 4096);
  if (*p) memset(*p, 0, bytes);
  return *p ? 0 : 2;
}
int hipFree(void *p) {
  if (fake.in_free) fake.in_free();
  if (fake.free_status) return fake.free_status;
  if (fake.pending) ++fake.freed_pending;
  fake.pending = 0;
  ++fake.frees;
  free(p);
  return 0;
}
int hipMallocAsync(void **p, size_t bytes, void *s) {
  (void)s;
  ++fake.mallocs_async;
  *p = aligned_alloc(4096, (bytes + 4095) / 4096 * 4096);
  return *p ? 0 : 2;
}
int hipFreeAsync(void *p, void *s) {
  (void)s;
  ++fake.frees_async;
  free(p);
  return 0;
}
int hipHostMalloc(void **p, size_t bytes, unsigned flags) {
  (void)flags;
  ++fake.host_mallocs;
  *p = calloc(1, bytes);
  if (n_host_words < 64) host_words[n_host_words++] = *p;
  return *p ? 0 : 2;
}
int hipStreamSynchronize(void *s) {
  (void)s;
  ++fake.syncs;
  if (fake.in_sync) fake.in_sync();
  if (fake.sync_status) return fake.sync_status;
  fake.pending = 0;
  for (int i = 0; i < n_host_words; ++i) memcpy(host_words[i], fake.words, sizeof(fake.words));
  return 0;
}
int hipGetLastError(void) {
  const int e = fake.last_error;
  fake.last_error = 0;
  return e;
}
const char *hipGetErrorString(int e) { return e == 2 ? "out of memory" : "fake error"; }
int hipGetDevice(int *d) {
  *d = fake.device;
  return 0;
}
int hipSetDevice(int d) {
  fake.device = d;
  return 0;
}
int hipMemGetInfo(size_t *f, size_t *t) {
  *f = (size_t)fake.free_bytes[fake.device & 1];
  *t = (size_t)fake.total_bytes[fake.device & 1];
  return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int kind) {
  (void)kind;
  memcpy(d, s, n);
  return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
  (void)st;
  if (kind == 2 && fake.copy_from && (int64_t)n == fake.copy_bytes) s = fake.copy_from;
  memcpy(d, s, n);
  return 0;
}
int hipStreamIsCapturing(void *s, int *status) {
  (void)s;
  *status = fake.capturing;
  return 0;
}
int hipFuncSetAttribute(const void *f, int a, int v) {
  (void)f;
  (void)a;
  (void)v;
  return 0;
}
int hipEventCreate(void **e) {
  *e = malloc(1);
  return 0;
}
int hipEventCreateWithFlags(void **e, unsigned flags) {
  (void)flags;
  return hipEventCreate(e);
}
int hipEventDestroy(void *e) {
  free(e);
  return 0;
}
int hipEventQuery(void *e) {
  (void)e;
  return fake.unfinished ? 600 : 0;
}
int hipStreamWaitEvent(void *s, void *e, unsigned flags) {
  (void)s;
  (void)e;
  (void)flags;
  ++fake.event_waits;
  return 0;
}
int hipEventRecord(void *e, void *s) {
  (void)e;
  (void)s;
  return 0;
}
int hipEventSynchronize(void *e) {
  (void)e;
  return 0;
}
int hipEventElapsedTime(float *ms, void *a, void *b) {
  (void)a;
  (void)b;
  *ms = 0;
  return 0;
}
static struct { Dim3 g, b; size_t shm; void *s; } cfg;
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shm, void *s) {
  cfg.g = g;
  cfg.b = b;
  cfg.shm = shm;
  cfg.s = s;
  return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *shm, void **s) {
  *g = cfg.g;
  *b = cfg.b;
  *shm = cfg.shm;
  *s = cfg.s;
  return 0;
}
int hipLaunchKernel(const void *f, Dim3 g, Dim3 b, void **args, size_t shm, void *s) {
  (void)f;
  (void)g;
  (void)b;
  (void)args;
  (void)shm;
  (void)s;
  ++fake.launches;
  ++fake.pending;
  return 0;
}
void *__hipRegisterFatBinary(void *d) { return d; }
void __hipRegisterFunction(void *m, const void *h, char *n, const char *dn, unsigned t, void *a,
                           void *b, void *c, void *d, int *w) {
  (void)m, (void)h, (void)n, (void)dn, (void)t, (void)a, (void)b, (void)c, (void)d, (void)w;
}
void __hipUnregisterFatBinary(void *m) { (void)m; }
