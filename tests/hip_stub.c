/* The few HIP runtime functions that libfsdp_bucket.so calls, for a process
 * without a GPU: kernels are registered and launches recorded by name, nothing
 * is run.  Loaded before the library, with its symbols global. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { const void *host; char *name; } kernel_t;
typedef struct { const char *name; dim3_t grid, block; } launch_t;

enum { MAX_KERNELS = 512, MAX_LAUNCHES = 64, CUS = 256 };
static kernel_t kernels[MAX_KERNELS];
static int num_kernels;
static launch_t launches[MAX_LAUNCHES];
static int num_launches;
static void *fatbin;

void **__hipRegisterFatBinary(const void *data) { (void)data; return &fatbin; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned threads,
                           void *tid, void *bid, void *block, void *grid, int *wave) {
    (void)modules; (void)device; (void)threads; (void)tid; (void)bid; (void)block; (void)grid; (void)wave;
    if (num_kernels < MAX_KERNELS) {
        kernels[num_kernels].host = host;
        kernels[num_kernels++].name = strdup(name);
    }
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream) {
    (void)grid; (void)block; (void)lds; (void)stream;
    return 1;
}
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int *value, int attribute, int device) {
    (void)attribute; (void)device;
    *value = CUS;
    return 0;
}
const char *hipGetErrorString(int e) { (void)e; return "refused by the stub"; }
int hipLaunchKernel(const void *host, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream) {
    (void)args; (void)lds; (void)stream;
    for (int k = 0; k < num_kernels && num_launches < MAX_LAUNCHES; ++k)
        if (kernels[k].host == host) {
            launches[num_launches].name = kernels[k].name;
            launches[num_launches].grid = grid;
            launches[num_launches++].block = block;
            return 0;
        }
    return 1;
}

int stub_cus(void) { return CUS; }
int stub_kernels(void) { return num_kernels; }
const char *stub_kernel(int k) { return kernels[k].name; }
int stub_launches(void) { return num_launches; }
const char *stub_launch(int k) { return launches[k].name; }
void stub_reset(void) { num_launches = 0; }
