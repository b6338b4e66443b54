/* Stands in for the HIP runtime entry points that libstagefrontier calls, so
 * that a CPU test can see which kernels a call launches, and how wide.  Every
 * launch is recorded and reported as successful; nothing runs. */
#include <stdint.h>
#include <string.h>

struct dim3c { uint32_t x, y, z; };

#define MAX_KERNELS 4096
#define MAX_LAUNCHES 64
static struct { const void* fn; const char* name; } kernels[MAX_KERNELS];
static int n_kernels;
static struct { const void* fn; uint32_t grid, block; uint64_t lds; } launches[MAX_LAUNCHES];
static int n_launches;
static void* handle;

void** __hipRegisterFatBinary(const void* data) { (void)data; return &handle; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** h, const void* fn, char* device, const char* name, unsigned limit,
                           void* tid, void* bid, void* block, void* grid, int* wsize)
{
    (void)h; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)wsize;
    if (n_kernels < MAX_KERNELS) {
        kernels[n_kernels].fn = fn;
        kernels[n_kernels++].name = name;
    }
}
int __hipPopCallConfiguration(void* g, void* b, uint64_t* lds, void** s)
{
    (void)g; (void)b; (void)lds; (void)s;
    return 1;
}
int hipLaunchKernel(const void* fn, struct dim3c grid, struct dim3c block, void** args, uint64_t lds, void* stream)
{
    (void)args; (void)stream;
    if (n_launches < MAX_LAUNCHES) {
        launches[n_launches].fn = fn;
        launches[n_launches].grid = grid.x;
        launches[n_launches].block = block.x;
        launches[n_launches++].lds = lds;
    }
    return 0;
}
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipStreamGetDevice(void* stream, int* dev) { (void)stream; *dev = 0; return 0; }
int hipDeviceGetAttribute(int* value, int attr, int dev) { (void)attr; (void)dev; *value = 256; return 0; }

void rec_clear(void) { n_launches = 0; }
int rec_launches(void) { return n_launches; }
uint32_t rec_grid(int i) { return launches[i].grid; }
uint32_t rec_block(int i) { return launches[i].block; }
uint64_t rec_lds(int i) { return launches[i].lds; }
const char* rec_name(int i)
{
    for (int k = 0; k < n_kernels; ++k)
        if (kernels[k].fn == launches[i].fn) return kernels[k].name;
    return "?";
}
