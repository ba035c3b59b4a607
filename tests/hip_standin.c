/* A stand-in for the HIP host runtime, preloaded under libpr.so on a machine
 * without a GPU: device memory is host memory, copies and fills are done at
 * once, kernels do nothing but are logged.  It lets tests force what a device
 * does rarely: an allocation that fails, a launch whose workgroups lose each
 * other, a stream that may use few compute units.  Time is a count of launches
 * (si_cost microseconds each). */
#define _GNU_SOURCE
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef struct { void *slots; void *head; uint64_t *lost; } xbuf;
typedef struct { double v[2]; uint64_t tag, lost; int32_t flag; } result;

#define MAXF 4096
static struct { const void *f; char name[256]; double us; } fn[MAXF];
static int nfn;
static struct { const void *var; void *mem; size_t size; } var[64];
static int nvar;

/* controls */
static size_t fail_above;
static int cus = 256, nulls, copies;
static char lose[64];
static char logbuf[1 << 20];
static size_t loglen;
static double clock_us;
static int last_error;

void si_fail_above(size_t bytes) { fail_above = bytes; }
void si_cus(int n) { cus = n; }
void si_lose(const char *kernel) { snprintf(lose, sizeof lose, "%s", kernel); }
const char *si_log(void) { return logbuf; }
int si_nulls(void) { return nulls; }
int si_copies(void) { return copies; }
void si_clear(void) { loglen = 0; logbuf[0] = 0; copies = nulls = 0; }
void si_cost(const char *kernel, double us) {
  for (int i = 0; i < nfn; i++)
    if (strstr(fn[i].name, kernel)) fn[i].us = us;
}

/* launches */
typedef struct { int id; uint64_t *lost; result *res; } node;
typedef struct { node *v; int n; } graph;
static graph *capture;
static dim3 cfg_grid, cfg_block;
static size_t cfg_shm;
static void *cfg_stream;

static void run(node k) {
  static uint64_t tag;
  tag++;
  clock_us += fn[k.id].us;
  if (k.res) k.res->tag = tag, k.res->flag = 0;
  if (k.lost && lose[0] && strstr(fn[k.id].name, lose)) *k.lost = tag;
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t shm, void *s) {
  cfg_grid = g, cfg_block = b, cfg_shm = shm, cfg_stream = s;
  return 0;
}
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shm, void **s) {
  *g = cfg_grid, *b = cfg_block, *shm = cfg_shm, *s = cfg_stream;
  return 0;
}
void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **m, const void *f, char *d, const char *name, unsigned l, void *a, void *b, void *c,
                           void *e, int *w) {
  (void)m, (void)d, (void)l, (void)a, (void)b, (void)c, (void)e, (void)w;
  if (nfn == MAXF) abort();
  fn[nfn].f = f, fn[nfn].us = 1.0;
  snprintf(fn[nfn++].name, sizeof fn[0].name, "%s", name);
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int ext, size_t size, int c, int g) {
  (void)m, (void)h, (void)d, (void)ext, (void)c, (void)g;
  if (nvar == 64) abort();
  var[nvar].var = v, var[nvar++].size = size;
}
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t shm, void *s) {
  (void)b, (void)shm, (void)s;
  int id = 0;
  while (id < nfn && fn[id].f != f) id++;
  if (id == nfn) abort();
  const char *nm = fn[id].name;
  node k = {id, NULL, NULL};
  if (strstr(nm, "k_regularizer_x")) k.lost = ((xbuf *)args[9])->lost, k.res = *(result **)args[8];
  else if (strstr(nm, "k_prox_x")) k.lost = ((xbuf *)args[8])->lost, k.res = *(result **)args[7];
  else if (strstr(nm, "k_node_init_x") || strstr(nm, "k_node_step_x")) k.lost = ((xbuf *)args[5])->lost;
  if (strstr(nm, "k_feat_prep"))
    for (int i = 3; i < 6; i++) nulls += *(void **)args[i] == NULL;
  if (loglen + 320 < sizeof logbuf) loglen += (size_t)sprintf(logbuf + loglen, "%s %u %u\n", nm, g.x, g.y);
  if (capture) {
    capture->v = realloc(capture->v, sizeof(node) * (size_t)(capture->n + 1));
    capture->v[capture->n++] = k;
  } else {
    run(k);
  }
  return 0;
}
int hipStreamBeginCapture(void *s, int m) { (void)s, (void)m; capture = calloc(1, sizeof *capture); return 0; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = capture; capture = NULL; return 0; }
int hipGraphInstantiate(void **e, void *g, void *n, char *l, size_t z) {
  (void)n, (void)l, (void)z;
  graph *c = malloc(sizeof *c);
  *c = *(graph *)g;
  c->v = memcpy(malloc(sizeof(node) * (size_t)c->n + 1), c->v, sizeof(node) * (size_t)c->n);
  *e = c;
  return 0;
}
int hipGraphLaunch(void *e, void *s) {
  (void)s;
  for (int i = 0; i < ((graph *)e)->n; i++) run(((graph *)e)->v[i]);
  return 0;
}
int hipGraphDestroy(void *g) { free(((graph *)g)->v); free(g); return 0; }
int hipGraphExecDestroy(void *g) { return hipGraphDestroy(g); }

/* memory */
int hipMalloc(void **p, size_t n) {
  *p = NULL;
  if (fail_above && n > fail_above) return last_error = 2;
  return (*p = calloc(1, n ? n : 1)) ? 0 : 2;
}
int hipFree(void *p) { free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; return (*p = calloc(1, n ? n : 1)) ? 0 : 2; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memmove(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *q) {
  (void)q;
  copies += k == 1;
  memmove(d, s, n);
  return 0;
}
int hipMemsetAsync(void *d, int v, size_t n, void *q) { (void)q; memset(d, v, n); return 0; }
int hipGetSymbolAddress(void **p, const void *v) {
  for (int i = 0; i < nvar; i++)
    if (var[i].var == v) {
      if (!var[i].mem) var[i].mem = calloc(1, var[i].size);
      *p = var[i].mem;
      return 0;
    }
  return 1;
}

/* streams, events, device */
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) {
  const int e = last_error;
  last_error = 0;
  return e;
}
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(1); return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipEventCreate(void **e) { *e = calloc(1, sizeof(double)); return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *e, void *s) { (void)s; *(double *)e = clock_us; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { *ms = (float)((*(double *)b - *(double *)a) * 1e-3); return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a, (void)d; *v = cus; return 0; }
int hipExtStreamGetCUMask(void *s, uint32_t n, uint32_t *m) {
  if (s == (void *)1) abort(); /* hipStreamLegacy: the runtime takes it for a pointer */
  for (uint32_t i = 0; i < n; i++) {
    const int left = cus - 32 * (int)i;
    m[i] = left >= 32 ? 0xffffffffu : (left > 0 ? (1u << left) - 1u : 0u);
  }
  return 0;
}
