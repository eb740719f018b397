/* Stands in for the HIP runtime on a machine without a GPU: a process that loads this (globally) before liblookupffn.so
 * sees every kernel launch as a record instead of a launch.  Device memory is never touched, so a call may be of any size. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_;
enum { kMaxKernels = 4096, kArgBytes = 256, kLogBytes = 1 << 20 };
static struct { const void *host; const char *name; } kernels[kMaxKernels];
static int n_kernels;
static char text[kLogBytes];
static size_t used;
static int compute_units = 256;
static struct { dim3_ grid, block; size_t lds; void *stream; } pushed;

/* ---- what the test uses */
void recorder_set_compute_units(int n) { compute_units = n; }
/* the launches since the last call, a line each: name, grid, block, LDS bytes, the first bytes of the arguments in hex */
const char *recorder_take(void)
{
    static char out[kLogBytes];
    memcpy(out, text, used);
    out[used] = 0;
    used = 0;
    return out;
}

/* ---- what the library calls */
void **__hipRegisterFatBinary(const void *data) { (void)data; return malloc(8); }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void **m, const void *host, char *device, const char *name, unsigned limit, void *a, void *b, void *c,
                           void *d, int *e)
{
    (void)m; (void)device; (void)limit; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (n_kernels < kMaxKernels) {
        kernels[n_kernels].host = host;
        kernels[n_kernels++].name = name;
    }
}
int __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t lds, void *stream)
{
    pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_ *grid, dim3_ *block, size_t *lds, void **stream)
{
    *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void *host, dim3_ grid, dim3_ block, void **args, size_t lds, void *stream)
{
    const char *name = "?";
    (void)stream;
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == host) name = kernels[i].name;
    if (used + strlen(name) + 2 * kArgBytes + 256 > kLogBytes) return 2;
    used += (size_t)sprintf(text + used, "%s %u %u %u %u %zu ", name, grid.x, grid.y, grid.z, block.x, lds);
    /* one structure, or (the re-pack kernels) a list that starts with two pointers */
    if (strstr(name, "repack"))
        for (int i = 0; i < 16; ++i) used += (size_t)sprintf(text + used, "%02x", ((const unsigned char *)args[i / 8])[i % 8]);
    else
        for (int i = 0; i < kArgBytes; ++i) used += (size_t)sprintf(text + used, "%02x", ((const unsigned char *)args[0])[i]);
    used += (size_t)sprintf(text + used, "\n");
    return 0;
}
int hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = compute_units; return 0; }
int hipGetDevice(int *dev) { *dev = 0; return 0; }
int hipSetDevice(int dev) { (void)dev; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { (void)e; return ""; }
int hipFuncSetAttribute(const void *f, int attr, int v) { (void)f; (void)attr; (void)v; return 0; }
int hipFuncGetAttributes(void *attr, const void *f) { (void)attr; (void)f; return 0; }
int hipMalloc(void **p, size_t n) { (void)n; *p = (void *)(uintptr_t)(1ull << 30); return 0; }
int hipFree(void *p) { (void)p; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = (void *)(uintptr_t)(1ull << 30); return 0; }
int hipEventCreate(void **e) { *e = (void *)8; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0; return 0; }
