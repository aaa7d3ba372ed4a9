// A HIP runtime without a GPU: the calls that libmlpmoe.so makes, recorded and answered on the host.  Loaded with
// RTLD_GLOBAL before the library, its symbols are found before the real runtime's.  No kernel runs: a launch is a line
// "launch NAME gx gy gz" of the record, and device memory is a number.
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <map>
#include <string>

namespace {
struct Dim3 {
    uint32_t x, y, z;
};
std::map<const void *, std::string> g_kernels;
std::string g_record;
size_t g_largest = ~(size_t)0;              // larger allocations fail
int g_capturing = 0, g_last_error = 0;
uintptr_t g_next = 1u << 20;
Dim3 g_grid, g_block;
size_t g_shared;
void *g_stream;
void note(const std::string &s) { g_record += s + "\n"; }
}  // namespace

extern "C" {
const char *fake_record(void) { return g_record.c_str(); }
void fake_clear(void) { g_record.clear(); }
void fake_largest_allocation(size_t n) { g_largest = n; }
void fake_capturing(int on) { g_capturing = on; }

void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    g_kernels[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream)
{
    g_grid = grid, g_block = block, g_shared = shared, g_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream)
{
    *grid = g_grid, *block = g_block, *shared = g_shared, *stream = g_stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3, void **, size_t, void *)
{
    note("launch " + g_kernels[f] + " " + std::to_string(grid.x) + " " + std::to_string(grid.y) + " " + std::to_string(grid.z));
    return 0;
}
int hipMalloc(void **p, size_t n)
{
    if (n > g_largest) {
        note("refuse " + std::to_string(n));
        return g_last_error = 2;            // out of memory
    }
    note("malloc " + std::to_string(n));
    *p = reinterpret_cast<void *>(g_next);
    g_next += (n + 4095) / 4096 * 4096 + 4096;
    return 0;
}
int hipFree(void *p)
{
    if (p) note("free");
    return 0;
}
int hipMemcpyAsync(void *dst, const void *, size_t n, int, void *)
{
    memset(dst, 0, n);                      // device to host only
    return 0;
}
int hipGetLastError(void)
{
    const int e = g_last_error;
    g_last_error = 0;
    return e;
}
int hipStreamIsCapturing(void *, int *status)
{
    *status = g_capturing;
    return 0;
}
const char *hipGetErrorString(int e) { return e == 1 ? "invalid argument" : e == 2 ? "out of memory" : "error"; }
int hipGetDevice(int *d)
{
    *d = 0;
    return 0;
}
int hipSetDevice(int) { return 0; }
int hipGetDevicePropertiesR0600(void *, int) { return 0; }      // the number of CUs stays what it was: only grids depend on it
int hipDeviceSynchronize(void) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
}
