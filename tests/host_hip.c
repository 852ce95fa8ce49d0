/* A HIP runtime in host memory, for tests of the library's host side on a
 * machine without a GPU.  Loaded with RTLD_GLOBAL before libgsp.so, its
 * functions take the place of the runtime's: allocations are zeroed host
 * memory within a limit, copies are done at once, kernels are not run but
 * written to a log (name, grid, block, LDS bytes, the first bytes of the
 * first argument), a captured graph holds its launches and logs them at every
 * replay.  Events all have the same time. */
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct {
  char name[160];
  uint32_t grid[3], block[3];
  uint64_t lds;
  unsigned char arg[400];
  int32_t replayed, pad;
} launch_t;
typedef struct { launch_t *l; int n; } graph_t;
typedef struct { unsigned char *p; size_t n; } block_t;

enum { MAX_LOG = 1 << 18, MAX_FUN = 1 << 10, MAX_BLOCKS = 1 << 16 };
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static launch_t *log_;
static int n_log;
static struct { const void *f; const char *name; } *fun;
static int n_fun;
static block_t *blocks;
static int n_blocks;
static size_t used, limit = (size_t)1 << 36;
static graph_t *capture;
static __thread struct { dim3_t g, b; size_t sh; void *st; } call_;

/* ---- what the tests read and set ---- */
void hh_limit(uint64_t bytes) { limit = bytes; }
uint64_t hh_used(void) { return used; }
int hh_log_size(void) { return n_log; }
const launch_t *hh_log(int k) { return &log_[k]; }
void hh_log_clear(void) { n_log = 0; }
/* bytes from p to the end of its allocation, -1 if it is in none */
int64_t hh_room(uint64_t p) {
  pthread_mutex_lock(&mu);
  int64_t r = -1;
  for (int k = 0; k < n_blocks; ++k)
    if (p >= (uint64_t)blocks[k].p && p < (uint64_t)blocks[k].p + blocks[k].n) r = (int64_t)((uint64_t)blocks[k].p + blocks[k].n - p);
  pthread_mutex_unlock(&mu);
  return r;
}

/* ---- code objects ---- */
void **__hipRegisterFatBinary(const void *d) { (void)d; return calloc(1, 8); }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *var, char *h, char *d, int ext, size_t n, int c, int g) {
  (void)m, (void)var, (void)h, (void)d, (void)ext, (void)n, (void)c, (void)g;
}
void __hipRegisterFunction(void **m, const void *f, char *d, const char *name, unsigned t, void *a, void *b, void *c,
                           void *e, int *w) {
  (void)m, (void)d, (void)t, (void)a, (void)b, (void)c, (void)e, (void)w;
  if (!fun) fun = calloc(MAX_FUN, sizeof(*fun));
  if (strstr(name, "3gsp") && n_fun < MAX_FUN) fun[n_fun].f = f, fun[n_fun++].name = name;
}
int hipGetSymbolAddress(void **p, const void *sym) {
  (void)sym;
  static void *scratch;
  if (!scratch) scratch = calloc(1, 64 << 20);
  *p = scratch;
  return 0;
}

/* ---- launches ---- */
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void *st) {
  call_.g = g, call_.b = b, call_.sh = sh, call_.st = st;
  return 0;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *sh, void **st) {
  *g = call_.g, *b = call_.b, *sh = call_.sh, *st = call_.st;
  return 0;
}
static void append(const launch_t *l) {
  if (!log_) log_ = calloc(MAX_LOG, sizeof(*log_));
  if (n_log < MAX_LOG) log_[n_log++] = *l;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t sh, void *st) {
  (void)st;
  launch_t l;
  memset(&l, 0, sizeof(l));
  for (int k = 0; k < n_fun; ++k)
    if (fun[k].f == f) snprintf(l.name, sizeof(l.name), "%s", fun[k].name);
  l.grid[0] = g.x, l.grid[1] = g.y, l.grid[2] = g.z;
  l.block[0] = b.x, l.block[1] = b.y, l.block[2] = b.z;
  l.lds = sh;
  /* arguments by value in one struct are longer than others: copy what a test reads */
  size_t n = 8;
  if (strstr(l.name, "k_sum_parts")) n = 392;
  if (args && args[0]) memcpy(l.arg, args[0], n);
  pthread_mutex_lock(&mu);
  if (capture) {
    capture->l = realloc(capture->l, sizeof(launch_t) * (capture->n + 1));
    capture->l[capture->n++] = l;
  } else {
    append(&l);
  }
  pthread_mutex_unlock(&mu);
  return 0;
}
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f, (void)a, (void)v; return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { (void)e; return "host HIP error"; }

/* ---- graphs ---- */
int hipStreamBeginCapture(void *st, int mode) {
  (void)st, (void)mode;
  pthread_mutex_lock(&mu);
  capture = calloc(1, sizeof(graph_t));
  pthread_mutex_unlock(&mu);
  return 0;
}
int hipStreamEndCapture(void *st, void **g) {
  (void)st;
  pthread_mutex_lock(&mu);
  *g = capture;
  capture = NULL;
  pthread_mutex_unlock(&mu);
  return 0;
}
int hipGraphInstantiate(void **x, void *g, void **n, char *b, size_t s) {
  (void)n, (void)b, (void)s;
  graph_t *c = calloc(1, sizeof(graph_t)), *src = g;
  c->n = src->n;
  c->l = malloc(sizeof(launch_t) * (src->n + 1));
  memcpy(c->l, src->l, sizeof(launch_t) * src->n);
  *x = c;
  return 0;
}
int hipGraphLaunch(void *x, void *st) {
  (void)st;
  graph_t *g = x;
  pthread_mutex_lock(&mu);
  for (int k = 0; k < g->n; ++k) {
    g->l[k].replayed = 1;
    append(&g->l[k]);
  }
  pthread_mutex_unlock(&mu);
  return 0;
}
int hipGraphDestroy(void *g) { free(((graph_t *)g)->l); free(g); return 0; }
int hipGraphExecDestroy(void *g) { return hipGraphDestroy(g); }

/* ---- memory ---- */
int hipMalloc(void **p, size_t n) {
  pthread_mutex_lock(&mu);
  int rc = 2; /* out of memory */
  if (!blocks) blocks = calloc(MAX_BLOCKS, sizeof(*blocks));
  if (used + n <= limit && n_blocks < MAX_BLOCKS && (*p = aligned_alloc(256, (n + 255) / 256 * 256))) {
    memset(*p, 0, n < (64u << 20) ? n : (64u << 20));
    blocks[n_blocks].p = *p;
    blocks[n_blocks++].n = n;
    used += n;
    rc = 0;
  }
  pthread_mutex_unlock(&mu);
  return rc;
}
int hipFree(void *p) {
  pthread_mutex_lock(&mu);
  for (int k = 0; k < n_blocks; ++k)
    if (blocks[k].p == p) {
      used -= blocks[k].n;
      blocks[k] = blocks[--n_blocks];
      free(p);
      break;
    }
  pthread_mutex_unlock(&mu);
  return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; return (*p = malloc(n ? n : 1)) ? 0 : 2; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemGetInfo(size_t *f, size_t *t) { *f = limit - used; *t = limit; return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memmove(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)st; return hipMemcpy(d, s, n, k); }
int hipMemcpy2D(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, int k) {
  (void)k;
  for (size_t i = 0; i < h; ++i) memmove((char *)d + i * dp, (const char *)s + i * sp, w);
  return 0;
}

/* ---- devices, streams, events ---- */
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(1); return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipEventCreate(void **e) { *e = malloc(1); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *e, void *s) { (void)e, (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a, (void)b; *ms = 0.f; return 0; }
