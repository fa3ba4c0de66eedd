/* The HIP runtime as libef's host code sees it, without a GPU: memory is the host's, kernels are not run but listed by name, and
 * the launch whose turn it is (fake_fail_at) fails.  Preloaded by tests/test_failed_launch.py.  Test infrastructure only. */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

enum { OK = 0, FAILED = 719 };
static struct { const void *host; const char *name; } kernels[512];
static int n_kernels, launches, fail_at = -1, last_error = OK;
static char listed[1 << 16];

void fake_begin(int launch) { launches = 0; fail_at = launch; listed[0] = 0; last_error = OK; }
const char *fake_launched(void) { return listed; }

void **__hipRegisterFatBinary(const void *data) { static void *one; (void)data; return &one; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void) {}
void __hipRegisterFunction(void **m, const void *host, char *device, const char *name, ...)
{
    (void)m; (void)device;
    if (n_kernels < 512) { kernels[n_kernels].host = host; kernels[n_kernels++].name = name; }
}
int __hipPushCallConfiguration(void) { return OK; }
int __hipPopCallConfiguration(void *grid, void *block, size_t *shared, void **stream)
{
    unsigned one[3] = {1, 1, 1};
    memcpy(grid, one, sizeof one); memcpy(block, one, sizeof one);
    *shared = 0; *stream = NULL;
    return OK;
}
int hipLaunchKernel(const void *host)
{
    const char *name = "?";
    int i;
    for (i = 0; i < n_kernels; ++i) if (kernels[i].host == host) name = kernels[i].name;
    if (launches++ == fail_at) return last_error = FAILED;
    if (strlen(listed) + strlen(name) + 2 < sizeof listed) { strcat(listed, name); strcat(listed, "\n"); }
    return OK;
}
int hipGetLastError(void) { int e = last_error; last_error = OK; return e; }
const char *hipGetErrorString(int e) { (void)e; return "made to fail"; }
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipDeviceGetAttribute(int *v) { *v = 256; return OK; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n) { *n = 7; return OK; }
int hipDeviceSynchronize(void) { return OK; }
int hipStreamSynchronize(void *s) { (void)s; return OK; }
int hipMalloc(void **p, size_t n) { *p = calloc(1, n + 256); return OK; }
int hipFree(void *p) { free(p); return OK; }
int hipMemcpy(void *d, const void *s, size_t n) { memcpy(d, s, n); return OK; }
int hipMemcpyAsync(void *d, const void *s, size_t n) { memcpy(d, s, n); return OK; }
int hipMemset(void *d, int v, size_t n) { memset(d, v, n); return OK; }
int hipMemsetAsync(void *d, int v, size_t n) { memset(d, v, n); return OK; }
int hipMemcpy2DAsync(void) { return OK; }
int hipGetSymbolAddress(void **p) { static double scratch[1 << 10]; *p = scratch; return OK; }
