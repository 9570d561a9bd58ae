/* The HIP entry points that libmmvseg.so calls, for a process without a GPU: nothing runs, the kernels that would be launched
 * and the events that would be recorded are written down in their order.  Loaded with RTLD_GLOBAL ahead of the library, whose
 * references then resolve here. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
static struct { const void *host; const char *name; } g_kernels[1024];
static int g_num_kernels;
static dim3 g_grid, g_block;
static size_t g_shared;
static void *g_stream;
static char g_log[1 << 16];
static void *g_module;

void **__hipRegisterFatBinary(const void *data) { (void)data; return &g_module; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned limit, void *tid, void *bid,
                           dim3 *block, dim3 *grid, int *size) {
    (void)modules, (void)device, (void)limit, (void)tid, (void)bid, (void)block, (void)grid, (void)size;
    if (g_num_kernels < 1024) g_kernels[g_num_kernels].host = host, g_kernels[g_num_kernels++].name = name;
}
void __hipRegisterVar(void **modules, void *var, char *host, char *device, int ext, size_t size, int constant, int global) {
    (void)modules, (void)var, (void)host, (void)device, (void)ext, (void)size, (void)constant, (void)global;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void *stream) {
    g_grid = grid, g_block = block, g_shared = shared, g_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, void **stream) {
    *grid = g_grid, *block = g_block, *shared = g_shared, *stream = g_stream;
    return 0;
}
static void note(const char *line) {
    if (strlen(g_log) + strlen(line) + 2 < sizeof(g_log)) strcat(strcat(g_log, line), "\n");
}
int hipLaunchKernel(const void *host, dim3 grid, dim3 block, void **args, size_t shared, void *stream) {
    (void)args, (void)shared, (void)stream;
    char line[512];
    const char *name = "?";
    for (int i = 0; i < g_num_kernels; ++i)
        if (g_kernels[i].host == host) name = g_kernels[i].name;
    snprintf(line, sizeof(line), "launch %s %u %u", name, grid.x, block.x);
    note(line);
    return 0;
}
int hipEventRecord(void *event, void *stream) {
    (void)stream;
    char line[64];
    snprintf(line, sizeof(line), "event %llu", (unsigned long long)(uintptr_t)event);
    note(line);
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int *value, int attribute, int device) { (void)attribute, (void)device; *value = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *blocks, const void *kernel, int threads, size_t shared) {
    (void)kernel, (void)threads, (void)shared;
    *blocks = 2;
    return 0;
}
int hipGetSymbolAddress(void **address, const void *symbol) { (void)symbol; *address = (void *)(uintptr_t)0x7f0000000000; return 0; }

const char *recorder_log(void) { return g_log; }
void recorder_clear(void) { g_log[0] = 0; }
