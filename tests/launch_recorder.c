/* Stands in for the HIP runtime's launch functions on a machine without a GPU: what the library's entry points
 * would launch is written down instead.  Loaded globally in front of libhalo.so (tests/launches.py), so that the
 * library's references find these definitions first.  Launches outside the documented grid limits fail, as they may
 * on a device: y and z up to 65535 workgroups, fewer than 2^32 threads along x; so do those with more than 64 KiB of dynamic
 * LDS that was not allowed on the current one of eight devices (recorder_device). */
#include <stddef.h>
#include <stdio.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;

static struct { const void *host; const char *name; int allowed[8]; } kernels[4096];
static int n_kernels, last_error, device;
static struct { dim3_t grid, block; size_t lds; void *stream; } pushed;
static char record[1 << 16];
static size_t used;

void **__hipRegisterFatBinary(const void *data) { (void)data; static void *module; return &module; }
void __hipUnregisterFatBinary(void **module) { (void)module; }
void __hipRegisterVar(void **module, void *var, char *host, char *name, int ext, size_t size, int constant, int global)
{
    (void)module; (void)var; (void)host; (void)name; (void)ext; (void)size; (void)constant; (void)global;
}
void __hipRegisterFunction(void **module, const void *host, char *name, const char *device_name, unsigned threads,
                           void *tid, void *bid, void *block, void *grid, int *warp)
{
    (void)module; (void)name; (void)threads; (void)tid; (void)bid; (void)block; (void)grid; (void)warp;
    if (n_kernels < 4096) {
        kernels[n_kernels].host = host;
        kernels[n_kernels++].name = device_name;
    }
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream)
{
    pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream)
{
    *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void *host, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream)
{
    const char *name = "?";
    size_t allowed = 65536;
    (void)args; (void)stream;
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == host) {
            name = kernels[i].name;
            if (kernels[i].allowed[device] > 65536) allowed = (size_t)kernels[i].allowed[device];
        }
    used += (size_t)snprintf(record + used, used < sizeof record - 512 ? 512 : 0, "%s %u %u %u %u\n", name, grid.x, grid.y,
                             grid.z, block.x);
    if (grid.y > 65535u || grid.z > 65535u || (unsigned long long)grid.x * block.x >= 1ull << 32) return last_error = 9;
    if (lds > allowed) return last_error = 1;
    return 0;
}
int hipFuncSetAttribute(const void *host, int attribute, int value)
{
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == host && attribute == 8) kernels[i].allowed[device] = value;   /* hipFuncAttributeMaxDynamicSharedMemorySize */
    return 0;
}
int hipGetDevice(int *dev) { *dev = device; return 0; }
void recorder_device(int dev) { device = dev; }
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }

/* the launches since the last call, a line each: mangled name, grid x y z, threads */
const char *recorder_take(void)
{
    static char out[sizeof record];
    memcpy(out, record, used);
    out[used] = 0;
    used = 0;
    return out;
}
