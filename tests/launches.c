/* Takes the place of the HIP runtime for a library that is loaded after it: kernels are named when the library registers them,
 * and a launch is written down instead of carried out.  No GPU is needed and no pointer is followed. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>

typedef struct { uint32_t x, y, z; } dim3;

static struct { const void *host; const char *name; } kernels[8192];
static int n_kernels;

void **__hipRegisterFatBinary(const void *data) { static void *handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void **handle) { (void)handle; }
void __hipRegisterVar(void **h, void *var, char *host, const char *device, int ext, size_t size, int constant, int global)
{
    (void)h; (void)var; (void)host; (void)device; (void)ext; (void)size; (void)constant; (void)global;
}
void __hipRegisterFunction(void **h, const void *host, char *device, const char *name, unsigned limit, void *tid, void *bid, void *block,
                           void *grid, int *size)
{
    (void)h; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)size;
    if (n_kernels < 8192) {
        kernels[n_kernels].host = host;
        kernels[n_kernels++].name = name;
    }
}
int hipLaunchKernel(const void *host, dim3 grid, dim3 block, void **args, size_t lds, void *stream)
{
    (void)args; (void)stream;
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == host) {
            printf("L %s %u %u %zu\n", kernels[i].name, grid.x, block.x, lds);
            fflush(stdout);
            /* the runtime refuses a launch of 2^32 threads or more, or of more than the largest workgroup */
            return (uint64_t)grid.x * block.x >= ((uint64_t)1 << 32) || block.x > 1024 || grid.x == 0 ? 9 : 0;
        }
    return 98;
}
