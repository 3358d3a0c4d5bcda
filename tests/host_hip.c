/* host_hip.c -- the HIP runtime calls of libbtdf without a GPU, preloaded by
 * test_host_cpu.py: device memory is host memory, kernels do nothing, and a
 * launch of the one-launch step is looked over where it would run (in a graph:
 * at every replay) and its findings kept for the test to read, as are the names
 * of the kernels that would run. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef struct { int t0, t1, m0, m1; } item;             /* StepItem */
typedef struct { const item *items; int count; } work;   /* StepWork */
typedef struct { int is_step; work w; uint32_t grid; const char *name; } launch;
typedef struct { launch *l; int n; } graph;

enum { kOk = 0, kOutOfMemory = 2, kMax = 1 << 16 };

/* per executed step launch: entries, workgroups, tiles stepped, tiles stepped twice */
static int found[kMax][4], n_found;
static work last_step;
static int pinned_calls, pinned_live, pinned_fails, sticky;
static graph *recording;
static const char *ran[kMax];
static int n_ran;

int host_hip_steps(const int **out) { *out = &found[0][0]; return n_found; }
int host_hip_last_step(const int **items) { *items = (const int *)last_step.items; return last_step.count; }
int host_hip_pinned_calls(void) { return pinned_calls; }
int host_hip_pinned_live(void) { return pinned_live; }
/* executed launches of kernels whose name holds part */
int host_hip_launched(const char *part) {
  int n = 0;
  for (int k = 0; k < n_ran; ++k) n += strstr(ran[k], part) != NULL;
  return n;
}
void host_hip_fail_pinned(int on) { pinned_fails = on; }

static void run(const launch *l) {
  if (n_ran < kMax) ran[n_ran++] = l->name;
  if (!l->is_step || n_found == kMax) return;
  last_step = l->w;
  static unsigned char seen[1 << 20];
  memset(seen, 0, sizeof seen);
  int *f = found[n_found++];
  f[0] = l->w.count;
  f[1] = (int)l->grid;
  f[2] = f[3] = 0;
  for (int k = 0; k < l->w.count; ++k)
    for (int half = 0; half < 2; ++half) {
      const item *it = &l->w.items[k];
      const int t = half ? it->t1 : it->t0;
      if (t < 0) continue;
      unsigned char *s = &seen[((t >> 16) & 1023) << 10 | (t & 1023)];
      f[*s ? 3 : 2]++;
      *s = 1;
    }
}

int hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t shared, void *stream) {
  (void)block, (void)shared, (void)stream;
  Dl_info d;
  launch l = {0};
  l.name = dladdr(fn, &d) && d.dli_sname ? d.dli_sname : "?";
  if (strstr(l.name, "step_kernel")) {
    l.is_step = 1;
    l.w = *(const work *)args[3];
    l.grid = grid.x;
  }
  if (recording) {
    recording->l = realloc(recording->l, (size_t)(recording->n + 1) * sizeof l);
    recording->l[recording->n++] = l;
  } else {
    run(&l);
  }
  return kOk;
}
static struct { dim3 g, b; size_t shared; void *stream; } config;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t shared, void *stream) {
  config.g = g, config.b = b, config.shared = shared, config.stream = stream;
  return kOk;
}
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shared, void **stream) {
  *g = config.g, *b = config.b, *shared = config.shared, *stream = config.stream;
  return kOk;
}

int hipMalloc(void **p, size_t n) { return posix_memalign(p, 256, n + 256) ? kOutOfMemory : kOk; }
int hipFree(void *p) { free(p); return kOk; }
int hipHostMalloc(void **p, size_t n, unsigned flags) {
  (void)flags;
  ++pinned_calls;
  *p = pinned_fails ? NULL : calloc(1, n);
  pinned_live += *p != NULL;
  return *p ? kOk : (sticky = kOutOfMemory);
}
int hipHostFree(void *p) { pinned_live -= p != NULL; free(p); return kOk; }
int hipGetLastError(void) { const int e = sticky; sticky = 0; return e; }
int hipGetDevice(int *d) { *d = 0; return kOk; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return kOk; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) { (void)kind, (void)st; memcpy(d, s, n); return kOk; }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)st; memset(d, v, n); return kOk; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(1); return kOk; }
int hipStreamDestroy(void *s) { free(s); return kOk; }
int hipStreamSynchronize(void *s) { (void)s; return kOk; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s, (void)e, (void)f; return kOk; }
int hipEventCreate(void **e) { *e = malloc(1); return kOk; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void *e) { free(e); return kOk; }
int hipEventRecord(void *e, void *s) { (void)e, (void)s; return kOk; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a, (void)b; *ms = 0.f; return kOk; }
int hipStreamBeginCapture(void *s, int mode) { (void)s, (void)mode; recording = calloc(1, sizeof(graph)); return kOk; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = recording; recording = NULL; return kOk; }
int hipGraphInstantiate(void **e, void *g, void *n, char *log, size_t len) {
  (void)n, (void)log, (void)len;
  graph *c = malloc(sizeof *c);
  c->n = ((graph *)g)->n;
  c->l = malloc((size_t)c->n * sizeof *c->l + 1);
  memcpy(c->l, ((graph *)g)->l, (size_t)c->n * sizeof *c->l);
  *e = c;
  return kOk;
}
int hipGraphLaunch(void *e, void *s) {
  (void)s;
  for (int k = 0; k < ((graph *)e)->n; ++k) run(&((graph *)e)->l[k]);
  return kOk;
}
int hipGraphDestroy(void *g) { free(((graph *)g)->l); free(g); return kOk; }
int hipGraphExecDestroy(void *g) { return hipGraphDestroy(g); }
