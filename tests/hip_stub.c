/* A HIP runtime without a device, for tests of the library's host code: loaded with RTLD_GLOBAL before
 * the library, its functions stand in for the runtime's.  Device memory is host memory reserved by
 * mmap, bounded by stub_limit; what has been freed is never handed out again (unless stub_reuse asks
 * for one address, whenever it is free, with memory of zeros), and an upload whose
 * words point into it is counted (stub_stale).  Launches are recorded by kernel name and run nothing;
 * the time between two events is shortest when the watched kernel ran with the grid of stub_fastest. */
#define _GNU_SOURCE
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

enum { OK = 0, INVALID = 1, NOMEM = 2, FAILED = 719 };
typedef struct { unsigned x, y, z; } dim3;

struct range { char *p; size_t n; int live; };
static struct range ranges[4096];
static int nranges, last_error, stale, nkernels, nlaunches;
static size_t live_bytes, peak_bytes, limit = (size_t)1 << 46;
static struct { const void *f; char name[256]; } kernels[4096];
static int launched[65536];
static const char *fail_name, *watched;
static long watched_grid, fastest_grid;
static char *reused;
static double read_value;

void stub_limit(size_t n) { limit = n; }
size_t stub_live(void) { return live_bytes; }
size_t stub_peak(void) { size_t p = peak_bytes; peak_bytes = live_bytes; return p; }
int stub_stale(void) { return stale; }
void stub_fail(const char *name) { fail_name = name; }
void stub_watch(const char *name) { watched = name; }
long stub_grid(void) { return watched_grid; }
void stub_fastest(long grid) { fastest_grid = grid; }
void stub_clear(void) { nlaunches = 0; }
/* Launches since stub_clear of kernels whose mangled name holds `name`. */
int stub_launches(const char *name) {
  int n = 0;
  for (int q = 0; q < nlaunches; ++q) n += strstr(kernels[launched[q]].name, name) != NULL;
  return n;
}

static const size_t kReused = (size_t)1 << 32;
void stub_reuse(int on) {
  reused = on ? mmap(NULL, kReused, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0) : NULL;
}
/* What copies to the host return. */
void stub_read(double v) { read_value = v; }

static int err(int e) {
  if (e) last_error = e;
  return e;
}
static struct range *find(const void *p) {
  for (int q = nranges - 1; q >= 0; --q)
    if ((char *)p >= ranges[q].p && (char *)p < ranges[q].p + ranges[q].n) return &ranges[q];
  return NULL;
}

int hipMalloc(void **p, size_t n) {
  if (live_bytes + n > limit || nranges == 4096) return err(NOMEM);
  n = (n + 4095) / 4096 * 4096;
  struct range *last = reused ? find(reused) : NULL;
  if (reused && n <= kReused && !(last && last->live)) {
    if (last) last->n = 0;
    mmap(reused, kReused, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE | MAP_FIXED, -1, 0);
    ranges[nranges++] = (struct range){reused, n, 1};
    live_bytes += n;
    *p = reused;
    return OK;
  }
  char *m = mmap(NULL, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return err(NOMEM);
  ranges[nranges++] = (struct range){m, n, 1};
  live_bytes += n;
  if (live_bytes > peak_bytes) peak_bytes = live_bytes;
  *p = m;
  return OK;
}
int hipFree(void *p) {
  struct range *r = p ? find(p) : NULL;
  if (!p) return OK;
  if (!r || !r->live || r->p != p) return err(INVALID);
  r->live = 0;
  live_bytes -= r->n;
  mprotect(r->p, r->n, PROT_NONE);
  return OK;
}
int hipHostMalloc(void **p, size_t n, unsigned flags) { (void)flags; return (*p = malloc(n)) ? OK : err(NOMEM); }
int hipHostFree(void *p) { free(p); return OK; }
int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *stream) {
  (void)kind; (void)stream;
  struct range *r = find(dst);
  if (find(src)) {
    for (size_t q = 0; q + 8 <= n; q += 8) memcpy((char *)dst + q, &read_value, 8);
    return OK;
  }
  if (!r || !r->live || (char *)dst + n > r->p + r->n) return err(INVALID);
  for (size_t q = 0; q + 8 <= n; q += 8) {
    const void *w;
    memcpy(&w, (const char *)src + q, 8);
    struct range *o = find(w);
    if (o && !o->live) ++stale;
  }
  memcpy(dst, src, n);
  return OK;
}
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t smem, void *stream) {
  (void)args; (void)stream;
  if (!g.x || !g.y || !g.z || b.x * b.y * b.z > 1024 || !b.x || smem > 160 * 1024) return err(INVALID);
  for (int q = 0; q < nkernels; ++q) {
    if (kernels[q].f != f) continue;
    if (fail_name && strstr(kernels[q].name, fail_name)) return err(FAILED);
    if (watched && strstr(kernels[q].name, watched)) watched_grid = (long)g.x * g.y * g.z;
    if (nlaunches < 65536) launched[nlaunches++] = q;
    return OK;
  }
  return err(INVALID);
}
static dim3 cfg_g, cfg_b;
static size_t cfg_s;
static void *cfg_t;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void *t) { cfg_g = g; cfg_b = b; cfg_s = s; cfg_t = t; return OK; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, void **t) { *g = cfg_g; *b = cfg_b; *s = cfg_s; *t = cfg_t; return OK; }
void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **m, const void *f, char *dev, const char *name, unsigned n, void *a, void *b, void *c,
                           void *d, int *e) {
  (void)m; (void)dev; (void)n; (void)a; (void)b; (void)c; (void)d; (void)e;
  if (nkernels == 4096) return;
  kernels[nkernels].f = f;
  strncpy(kernels[nkernels].name, name, 255);
  ++nkernels;
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return e == NOMEM ? "out of memory" : e ? "error" : "no error"; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return OK; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return OK; }
int hipGetSymbolAddress(void **p, const void *s) { static double z[4096]; (void)s; *p = z; return OK; }
int hipSetDevice(int d) { (void)d; return OK; }
int hipDeviceSynchronize(void) { return OK; }
int hipEventCreate(void **e) { return (*e = malloc(8)) ? OK : NOMEM; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return (*e = malloc(8)) ? OK : NOMEM; }
int hipEventDestroy(void *e) { free(e); return OK; }
int hipEventElapsedTime(float *t, void *a, void *b) {
  (void)a; (void)b;
  *t = 1.0f + (float)labs(watched_grid - fastest_grid);
  return OK;
}
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return OK; }
int hipEventSynchronize(void *e) { (void)e; return OK; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; return (*s = malloc(8)) ? OK : NOMEM; }
int hipStreamDestroy(void *s) { free(s); return OK; }
int hipStreamIsCapturing(void *s, int *v) { (void)s; *v = 0; return OK; }
int hipStreamSynchronize(void *s) { (void)s; return OK; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return OK; }
