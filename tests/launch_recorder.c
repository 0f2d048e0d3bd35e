/* Stands in for the HIP runtime under libq2d.so on a machine without a GPU: records
 * every kernel launch (name, grid, block, dynamic LDS) and runs nothing.  Loaded
 * with RTLD_GLOBAL before the library, in a process of its own. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef struct { const char *name; uint32_t grid, block; uint64_t lds; } launch;

enum { kMax = 4096 };
static struct { const void *fn; const char *name; } known[kMax];
static launch launches[kMax];
static int n_known, n_launches;
static struct { dim3 grid, block; size_t lds; void *stream; } config;

void **__hipRegisterFatBinary(const void *data) { static void *handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }

void __hipRegisterFunction(void **modules, const void *fn, char *device_fn, const char *name, unsigned limit, void *tid,
                           void *bid, void *block, void *grid, int *wsize)
{
    (void)modules; (void)device_fn; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)wsize;
    if (n_known < kMax) { known[n_known].fn = fn; known[n_known++].name = name; }
}

int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream)
{
    config.grid = grid; config.block = block; config.lds = lds; config.stream = stream;
    return 0;
}

int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream)
{
    *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream;
    return 0;
}

int hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, void *stream)
{
    (void)args; (void)stream;
    if (n_launches == kMax) return 1;
    launch *l = &launches[n_launches++];
    l->name = "?"; l->grid = grid.x; l->block = block.x; l->lds = lds;
    for (int i = 0; i < n_known; ++i)
        if (known[i].fn == fn) l->name = known[i].name;
    return 0;
}

int hipGetLastError(void) { return 0; }
int hipGetDevice(int *dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int *value, int attribute, int dev) { (void)attribute; (void)dev; *value = 256; return 0; }

int recorded(void) { return n_launches; }
const launch *recorded_launch(int i) { return &launches[i]; }
void record_clear(void) { n_launches = 0; }
