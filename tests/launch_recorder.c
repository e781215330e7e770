/* Stands in for the launch calls of the HIP runtime, so that a process without a GPU can ask libtwn.so which kernels a
 * call would launch.  Loaded with RTLD_GLOBAL before the library: its definitions come first.  Nothing runs and no
 * pointer argument is followed. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;

enum { MAX_KERNELS = 4096, MAX_LAUNCHES = 256 };
static struct { const void* stub; const char* name; } kernels[MAX_KERNELS];
static int kernel_count;
static struct { const char* name; dim3_t grid, block; } launches[MAX_LAUNCHES];
static int launch_count;
static struct { dim3_t grid, block; size_t shared; void* stream; } config;

void** __hipRegisterFatBinary(const void* data) { (void)data; static void* handle; return &handle; }
void __hipUnregisterFatBinary(void** modules) { (void)modules; }
void __hipRegisterFunction(void** modules, const void* stub, char* device_fn, const char* name, unsigned limit, void* a, void* b,
                           void* c, void* d, int* e) {
    (void)modules; (void)device_fn; (void)limit; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (kernel_count < MAX_KERNELS) {
        kernels[kernel_count].stub = stub;
        kernels[kernel_count++].name = name;
    }
}
void __hipRegisterVar(void** modules, void* var, char* host, const char* name, int ext, size_t size, int constant, int global) {
    (void)modules; (void)var; (void)host; (void)name; (void)ext; (void)size; (void)constant; (void)global;
}

int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shared, void* stream) {
    config.grid = grid; config.block = block; config.shared = shared; config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shared, void** stream) {
    *grid = config.grid; *block = config.block; *shared = config.shared; *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void* stub, dim3_t grid, dim3_t block, void** args, size_t shared, void* stream) {
    (void)args; (void)shared; (void)stream;
    if (launch_count < MAX_LAUNCHES) {
        launches[launch_count].name = "?";
        for (int i = 0; i < kernel_count; ++i)
            if (kernels[i].stub == stub) launches[launch_count].name = kernels[i].name;
        launches[launch_count].grid = grid;
        launches[launch_count++].block = block;
    }
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void* fn, int attribute, int value) { (void)fn; (void)attribute; (void)value; return 0; }
int hipGetDevice(int* device) { *device = 0; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* fn, int threads, size_t shared) {
    (void)fn; (void)threads; (void)shared;
    *n = 1;
    return 0;
}
int hipGetDevicePropertiesR0600(void* properties, int device) { (void)properties; (void)device; return 1; }

/* for the reader */
void recorder_clear(void) { launch_count = 0; }
int recorder_count(void) { return launch_count; }
const char* recorder_name(int i) { return launches[i].name; }
void recorder_grid(int i, uint32_t* out) {
    memcpy(out, &launches[i].grid, 12);
    memcpy(out + 3, &launches[i].block, 12);
}
