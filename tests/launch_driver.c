#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "tflbm.h"
/* Host side of the library without a GPU: the HIP runtime functions it calls
 * are defined here (exported, so that the library binds to these), launches are
 * recorded instead of run, and a chosen one of them fails.  Reads commands from
 * stdin (tests/launch_host.py), one a line, and prints for each its return code
 * and, per launch, the kernel's mangled name, its grid and the first two
 * pointers of its first argument (the state it reads and the one it writes). */
typedef struct { unsigned x, y, z; } dim3_t;
enum { kMaxKernels = 4096 };
static const void *fn_ptr[kMaxKernels];
static const char *fn_name[kMaxKernels];
static int n_fn, recording, fail_in = -1, last_error, per_cu = 8;

void **__hipRegisterFatBinary(const void *d) { (void)d; static void *h; return &h; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned tl, void *tid, void *bid,
                           void *bd, void *gd, int *ws) {
  (void)m; (void)dev; (void)tl; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
  if (n_fn < kMaxKernels) { fn_ptr[n_fn] = host; fn_name[n_fn++] = name; }
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
static dim3_t cfg_grid, cfg_block;
static size_t cfg_shared;
static void *cfg_stream;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void *st) {
  cfg_grid = g; cfg_block = b; cfg_shared = sh; cfg_stream = st;
  return 0;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *sh, void **st) {
  *g = cfg_grid; *b = cfg_block; *sh = cfg_shared; *st = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t sh, void *st) {
  (void)b; (void)sh; (void)st;
  if (fail_in >= 0 && fail_in-- == 0) return last_error = 719;
  if (!recording) return 0;
  const char *name = "?";
  for (int i = 0; i < n_fn; ++i)
    if (fn_ptr[i] == f) name = fn_name[i];
  uint64_t p[2];
  memcpy(p, args[0], sizeof(p));
  printf("launch %s %u %llx %llx\n", name, g.x, (unsigned long long)p[0], (unsigned long long)p[1]);
  return 0;
}
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return e ? "stub error" : "no error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t s) {
  (void)f; (void)b; (void)s; *n = per_cu; return 0;
}
int hipDeviceSynchronize(void) { return 0; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = (void *)0x1000; return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)d; (void)s; (void)n; (void)k; (void)st; return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)d; (void)v; (void)n; (void)st; return 0; }
int hipStreamSynchronize(void *st) { (void)st; return 0; }
int hipStreamIsCapturing(void *st, int *c) { (void)st; *c = 0; return 0; }
int hipStreamCreateWithFlags(void **st, unsigned f) { (void)f; *st = (void *)0x2000; return 0; }
int hipStreamDestroy(void *st) { (void)st; return 0; }
int hipStreamBeginCapture(void *st, int m) { (void)st; (void)m; return 0; }
int hipStreamEndCapture(void *st, void **g) { (void)st; *g = (void *)0x3000; return 0; }
int hipGraphDestroy(void *g) { (void)g; return 0; }
int hipGraphInstantiate(void **x, void *g, void *n, char *l, size_t s) { (void)g; (void)n; (void)l; (void)s; *x = (void *)0x4000; return 0; }
int hipGraphExecDestroy(void *x) { (void)x; return 0; }
int hipGraphLaunch(void *x, void *st) { (void)x; (void)st; return 0; }

int main(void) {
  /* addresses that nothing on the host reads */
  void *const ws = (void *)0x100000000000ull, *const cap = (void *)0x200000000000ull, *const adj = (void *)0x300000000000ull;
  double *const h0 = (double *)0x400000000000ull;
  char line[256], cmd[32];
  double mass, norms[8];
  tflbm_sim *s = NULL;
  while (fgets(line, sizeof line, stdin)) {
    int rc = 0, used = 0;
    if (sscanf(line, "%31s%n", cmd, &used) != 1) continue;
    const char *a = line + used;
    recording = 1;
    if (!strcmp(cmd, "sim")) { /* nx ny prec tau n m field(0 none, 1 theta, 2 gamma) g */
      tflbm_params p;
      tflbm_default_params(&p);
      int field = 0;
      sscanf(a, "%d %d %d %lf %d %d %d %lf", &p.nx, &p.ny, &p.prec, &p.tau, &p.n_exp, &p.m_exp, &field, &p.g);
      p.gamma_field = field == 2;
      tflbm_destroy(s);
      s = NULL;
      recording = 0;
      rc = tflbm_create(&p, &s);
      if (!rc) rc = tflbm_bind(s, ws, tflbm_workspace_bytes(s));
      if (!rc) rc = tflbm_init(s, h0, field == 1 ? h0 : NULL, NULL);
    } else if (!strcmp(cmd, "init")) {
      recording = 0;
      rc = tflbm_init(s, h0, NULL, NULL);
    } else if (!strcmp(cmd, "occupancy")) per_cu = atoi(a);
    else if (!strcmp(cmd, "fail")) fail_in = atoi(a);
    else if (!strcmp(cmd, "env")) {
      char name[64], value[64] = "";
      if (sscanf(a, "%63s %63s", name, value) == 2) setenv(name, value, 1);
      else unsetenv(name);
    } else if (!strcmp(cmd, "step")) rc = tflbm_step(s, atoll(a), NULL);
    else if (!strcmp(cmd, "capture")) rc = tflbm_step_capture(s, atoll(a), cap, NULL);
    else if (!strcmp(cmd, "read")) rc = tflbm_read(s, h0, NULL, NULL, NULL);
    else if (!strcmp(cmd, "mass")) rc = tflbm_mass(s, &mass, NULL);
    else if (!strcmp(cmd, "mass_noalloc")) rc = tflbm_mass_noalloc(s, h0, NULL);
    else if (!strcmp(cmd, "terms")) rc = tflbm_term_norms(s, norms, NULL);
    else if (!strcmp(cmd, "check")) rc = tflbm_check(s, NULL);
    else if (!strcmp(cmd, "save")) rc = tflbm_state_save(s, cap, NULL);
    else if (!strcmp(cmd, "load")) rc = tflbm_state_load(s, cap, 0, NULL);
    else if (!strcmp(cmd, "seed")) rc = tflbm_adj_seed(s, adj, h0, NULL);
    else if (!strcmp(cmd, "adj")) rc = tflbm_adj_steps(s, adj, cap, atoll(a), NULL);
    else if (!strcmp(cmd, "finish")) rc = tflbm_adj_finish(s, adj, h0, NULL, h0, h0, NULL);
    else if (!strcmp(cmd, "spp")) rc = tflbm_steps_per_pass(s);
    else if (!strcmp(cmd, "count")) rc = (int)tflbm_step_count(s);
    else rc = -99;
    printf("rc %d\n", rc);
    fflush(stdout);
  }
  tflbm_destroy(s);
  return 0;
}
