/* A HIP runtime without a device, for tests of the library's host code: memory of a given size that hands out host
 * addresses, streams that are or are not being captured, and a record of the launches. Loaded with global symbols
 * before the library, it takes the place of the runtime the library is linked to. No kernel runs. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
enum { MAXN = 4096 };

static size_t room = (size_t)1 << 40, used, peak;
static struct { void* p; size_t n; } block[MAXN];
static int blocks, mallocs, frees, last_error, capturing;
static struct { const void* host; const char* name; } fn[MAXN];
static int fns;
static char names[1 << 16];

/* what the tests set and read */
void stub_room(size_t bytes) { room = bytes; }
void stub_capturing(int on) { capturing = on; }
size_t stub_used(void) { return used; }
size_t stub_peak(void) { return peak; }
int stub_mallocs(void) { return mallocs; }
int stub_frees(void) { return frees; }
int stub_last_error(void) { return last_error; }
const char* stub_launches(void) { return names; }
void stub_reset(void);

int hipMalloc(void** out, size_t n) {
  mallocs++;
  if (capturing) { last_error = 900; return 900; }
  if (n > room - used || blocks == MAXN) { last_error = 2; return 2; }
  if (posix_memalign(out, 4096, n < (1u << 20) ? n : (1u << 20))) return 2;   /* the first part is enough: no kernel writes */
  memset(*out, 0, n < (1u << 20) ? n : (1u << 20));
  block[blocks].p = *out; block[blocks++].n = n;
  used += n;
  if (used > peak) peak = used;
  return 0;
}
int hipFree(void* p) {
  frees++;
  if (capturing) { last_error = 900; return 900; }
  for (int i = 0; i < blocks; i++)
    if (block[i].p == p) { used -= block[i].n; free(p); block[i] = block[--blocks]; return 0; }
  last_error = 1;
  return 1;
}
int hipMemGetInfo(size_t* f, size_t* t) { if (capturing) { last_error = 900; return 900; } *f = room - used; *t = room; return 0; }
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamIsCapturing(void* s, int* status) { (void)s; *status = capturing ? 1 : 0; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0; return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamBeginCapture(void* s, int mode) { (void)s; (void)mode; return 1; }
int hipStreamEndCapture(void* s, void** g) { (void)s; *g = 0; return 1; }
int hipMemcpy(void* d, const void* s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return 0; }

static struct { dim3_t g, b; size_t sh; void* s; } pushed;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void* s) { pushed.g = g; pushed.b = b; pushed.sh = sh; pushed.s = s; return 0; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* sh, void** s) { *g = pushed.g; *b = pushed.b; *sh = pushed.sh; *s = pushed.s; return 0; }
void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* hn, char* dn, int ext, size_t n, int c, int g) { (void)m; (void)v; (void)hn; (void)dn; (void)ext; (void)n; (void)c; (void)g; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned tl, void* a, void* b, void* c, void* d, int* w) {
  (void)m; (void)dev; (void)tl; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (fns < MAXN) { fn[fns].host = host; fn[fns++].name = name; }
}
static int misaligned;   /* launches of kernels whose loads take 16 bytes at a time that were given another address */
int stub_misaligned(void) { return misaligned; }
/* places (in words of 8 bytes of the first argument) of what such a kernel reads by these loads; those that are null or -1 it doesn't */
static const struct { const char* name; int at[4]; } wide[] = {
  {"mlp_hidden_kernel", {0, 1, 5, -1}}, {"mlp_output_kernel", {6, -1, -1, -1}}, {"mlp_dh_tiled_kernel", {0, 1, 4, 5}}, {"bilinear_project_kernel", {0, 1, -1, -1}},
  {"bilinear_end_kernel", {0, 1, 2, -1}}};
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t sh, void* s) {
  (void)s;
  const char* name = "?";
  for (int i = 0; i < fns; i++) if (fn[i].host == f) name = fn[i].name;
  for (int i = 0; i < (int)(sizeof wide / sizeof *wide); i++)
    if (strstr(name, wide[i].name))
      for (int k = 0; k < 4; k++)
        if (wide[i].at[k] >= 0 && ((const uint64_t*)args[0])[wide[i].at[k]] % 16) misaligned++;
  size_t at = strlen(names);
  snprintf(names + at, sizeof names - at, "%s %u %u %u %u %zu\n", name, g.x, g.y, g.z, b.x, sh);
  if (g.x == 0 || g.y == 0 || g.z == 0 || b.x == 0 || b.x > 1024 || sh > 163840) { last_error = 9; return 9; }
  return 0;
}
void stub_reset(void) { names[0] = 0; mallocs = frees = misaligned = 0; peak = used; }
