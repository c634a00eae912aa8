/* A HIP runtime that does nothing and writes down what it is asked for, so that the host side of libppo.so (which
 * allocations a call makes, which kernels it launches and how) can be tested without a GPU.  Loaded with global symbol
 * scope before the library: its definitions are found before those of the real runtime.  Pointers it hands out are
 * never dereferenced. */
#include <stdio.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;

enum { kSuccess = 0, kOutOfMemory = 2, kInvalidConfiguration = 9 };

static size_t limit = ~(size_t)0;   /* requests for more fail */
static int is_capturing = 0;
static int last_error = kSuccess;
static char text[1 << 20];
static size_t used = 0;
static uintptr_t next_address = (uintptr_t)0x700000000000u;
static struct { dim3 grid, block; size_t lds; void *stream; } config;
static struct { const void *function; const char *name; } kernels[1024];
static int n_kernels = 0;
static void *module = &module;

static void note(const char *line) {
    const size_t n = strlen(line);
    if (used + n + 2 > sizeof text) return;
    memcpy(text + used, line, n);
    used += n;
    text[used++] = '\n';
    text[used] = 0;
}
static int fail(int e) { return last_error = e; }

void fake_reset(size_t most, int capturing) {
    limit = most;
    is_capturing = capturing;
    last_error = kSuccess;
    used = 0;
    text[0] = 0;
}
const char *fake_log(void) { return text; }

void **__hipRegisterFatBinary(const void *data) { (void)data; return &module; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterFunction(void **modules, const void *function, char *device_function, const char *name, unsigned limit_,
                           void *tid, void *bid, dim3 *block, dim3 *grid, int *warp) {
    (void)modules; (void)device_function; (void)limit_; (void)tid; (void)bid; (void)block; (void)grid; (void)warp;
    if (n_kernels < 1024) {
        kernels[n_kernels].function = function;
        kernels[n_kernels++].name = name;
    }
}
void __hipRegisterVar(void **modules, void *var, char *host, char *name, int ext, size_t size, int constant, int global) {
    (void)modules; (void)var; (void)host; (void)name; (void)ext; (void)size; (void)constant; (void)global;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
    config.grid = grid;
    config.block = block;
    config.lds = lds;
    config.stream = stream;
    return kSuccess;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *stream = config.stream;
    return kSuccess;
}
int hipLaunchKernel(const void *function, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
    char line[512];
    const char *name = "?";
    (void)args; (void)stream;
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].function == function) name = kernels[i].name;
    /* documented limits: fewer than 2^32 threads in each dimension, 65,535 blocks in y and z */
    if ((uint64_t)grid.x * block.x > 0xFFFFFFFFu || (uint64_t)grid.y * block.y > 0xFFFFFFFFu ||
        (uint64_t)grid.z * block.z > 0xFFFFFFFFu || grid.x == 0 || grid.y == 0 || grid.z == 0 || grid.y > 65535 || grid.z > 65535)
        return fail(kInvalidConfiguration);
    snprintf(line, sizeof line, "launch %.300s %u %u %u %u %zu", name, grid.x, grid.y, grid.z, block.x, lds);
    note(line);
    return kSuccess;
}
int hipMallocAsync(void **p, size_t size, void *stream) {
    char line[64];
    (void)stream;
    snprintf(line, sizeof line, "%s %zu", size > limit ? "refused" : "malloc", size);
    note(line);
    if (size > limit) return fail(kOutOfMemory);
    *p = (void *)next_address;
    next_address += (size + 4095) & ~(size_t)4095;
    return kSuccess;
}
int hipFreeAsync(void *p, void *stream) {
    (void)p; (void)stream;
    note("free");
    return kSuccess;
}
int hipFuncSetAttribute(const void *f, int attribute, int value) { (void)f; (void)attribute; (void)value; return kSuccess; }
int hipGetDevice(int *device) { *device = 0; return kSuccess; }
int hipGetLastError(void) { const int e = last_error; last_error = kSuccess; return e; }
const char *hipGetErrorString(int e) { (void)e; return "fake error"; }
int hipGetSymbolAddress(void **p, const void *symbol) { (void)symbol; *p = (void *)(uintptr_t)0x600000000000u; return kSuccess; }
int hipStreamIsCapturing(void *stream, int *status) { (void)stream; *status = is_capturing; return kSuccess; }
