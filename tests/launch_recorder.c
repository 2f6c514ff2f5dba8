/* Stands in for the HIP runtime in a process without a GPU (preloaded): device memory is address space only, every call
   succeeds, nothing runs; what was called is written down, one line each. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;

static char log_[1 << 20];
static size_t used;
static struct { const void *fn; char name[256]; } kernels[512];
static int n_kernels;
static struct { dim3 grid, block; size_t shared; void *stream; } call_;

#define NOTE(...) (used += (size_t)snprintf(log_ + used, sizeof log_ - used, __VA_ARGS__))

const char *recorder_take(void)          /* the lines since the last call */
{
    static char out[sizeof log_];
    memcpy(out, log_, used + 1);
    used = 0;
    log_[0] = 0;
    return out;
}

void __hipRegisterFunction(void **modules, const void *host, char *device_fn, const char *name, unsigned limit, void *tid,
                           void *bid, dim3 *block, dim3 *grid, int *wsize)
{
    (void)modules, (void)device_fn, (void)limit, (void)tid, (void)bid, (void)block, (void)grid, (void)wsize;
    if (strstr(name, "salus") && n_kernels < 512) {
        kernels[n_kernels].fn = host;
        snprintf(kernels[n_kernels++].name, 256, "%s", name);
    }
}

int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void *stream)
{
    call_.grid = grid;
    call_.block = block;
    call_.shared = shared;
    call_.stream = stream;
    return 0;
}

int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, void **stream)
{
    *grid = call_.grid;
    *block = call_.block;
    *shared = call_.shared;
    *stream = call_.stream;
    return 0;
}

int hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t shared, void *stream)
{
    (void)args;
    (void)shared;
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].fn == fn) NOTE("launch %s %u %u %p\n", kernels[i].name, grid.x, block.x, stream);
    return 0;
}

int hipMalloc(void **p, size_t n) { NOTE("hipMalloc %zu\n", n); *p = aligned_alloc(256, (n + 255) / 256 * 256); return 0; }
int hipFree(void *p) { NOTE("hipFree\n"); free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned flags)
{
    (void)flags;
    NOTE("hipHostMalloc %zu\n", n);
    *p = calloc(1, n);
    return 0;
}
int hipHostFree(void *p) { NOTE("hipHostFree\n"); free(p); return 0; }
int hipHostGetDevicePointer(void **d, void *h, unsigned flags) { (void)flags; *d = h; return 0; }
int hipMemset(void *p, int v, size_t n) { NOTE("hipMemset\n"); memset(p, v, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *stream)
{
    (void)d, (void)s, (void)n, (void)kind, (void)stream;
    NOTE("hipMemcpyAsync\n");
    return 0;
}
int hipStreamSynchronize(void *stream) { NOTE("hipStreamSynchronize %p\n", stream); return 0; }
int hipDeviceSynchronize(void) { NOTE("hipDeviceSynchronize\n"); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int attribute, int device) { (void)attribute, (void)device; *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int block, size_t shared)
{
    (void)f, (void)block, (void)shared;
    *n = 2;
    return 0;
}
int hipGetLastError(void) { return 0; }
