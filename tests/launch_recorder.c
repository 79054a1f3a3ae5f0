/* A stand-in for the HIP runtime: it records what the library launches and starts nothing.  Built and loaded ahead of
 * libmoe_wq.so by launches.py, in a process of its own. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;

enum { MAX_KERNELS = 4096 };
static struct { const void *host; char name[512]; } kernels[MAX_KERNELS];
static int n_kernels, device;
static char text[1 << 22];
static size_t used;
static struct { dim3_t grid, block; size_t shared; void *stream; } config;

static const char *name_of(const void *host)
{
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == host) return kernels[i].name;
    return "?";
}

void recorder_device(int d) { device = d; }
const char *recorder_take(void) { used = 0; return text; }
void recorder_clear(void) { used = 0; text[0] = 0; }

void **__hipRegisterFatBinary(const void *data) { static void *handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) { (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g; }
void __hipRegisterFunction(void **m, const void *host, char *device_fn, const char *device_name, unsigned limit, void *a, void *b, void *c, void *d, int *e)
{
    (void)m; (void)device_fn; (void)limit; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (n_kernels < MAX_KERNELS) {
        kernels[n_kernels].host = host;
        snprintf(kernels[n_kernels++].name, sizeof(kernels[0].name), "%s", device_name);
    }
}

int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shared, void *stream)
{
    config.grid = grid, config.block = block, config.shared = shared, config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *shared, void **stream)
{
    *grid = config.grid, *block = config.block, *shared = config.shared, *stream = config.stream;
    return 0;
}

int hipLaunchKernel(const void *host, dim3_t grid, dim3_t block, void **args, size_t shared, void *stream)
{
    (void)args; (void)stream;
    used += (size_t)snprintf(text + used, sizeof(text) - used, "launch %d %u %u %u %u %zu %s\n", device, grid.x, grid.y, grid.z, block.x, shared, name_of(host));
    return 0;
}
int hipFuncSetAttribute(const void *host, int attr, int value)
{
    (void)attr;
    used += (size_t)snprintf(text + used, sizeof(text) - used, "lds %d %d %s\n", device, value, name_of(host));
    return 0;
}
int hipGetDevice(int *d) { *d = device; return 0; }
int hipDeviceGetAttribute(int *v, int attr, int d) { (void)attr; (void)d; *v = 256; return 0; }     /* only asked for the compute units */
int hipGetDevicePropertiesR0600(void *p, int d) { (void)p; (void)d; return 1; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { (void)e; return "recorded"; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = (void *)0x100000; return 0; }
