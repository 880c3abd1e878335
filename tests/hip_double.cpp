// A stand-in for the HIP runtime, for tests of the library's host side without a GPU: loaded before liblords.so, its functions
// take the place of the runtime's.  Allocations are addresses that nobody reads, launches are written down by kernel name.
#include <cstddef>
#include <cstdint>
#include <map>
#include <string>

namespace {
std::map<const void *, std::string> kernels;
std::string launched;                   // names of the kernels launched so far, one a line
size_t largest = ~(size_t)0;            // an allocation above this many bytes is refused
int capturing = 0, asked = 0, refused = 0, last_error = 0;
uintptr_t next_address = (uintptr_t)1 << 40;
struct Dim3 { uint32_t x, y, z; };
struct Call { Dim3 grid, block; size_t shared; void *stream; } pushed;
}  // namespace

extern "C" {
void double_largest_allocation(size_t bytes) { largest = bytes; }
void double_capturing(int yes) { capturing = yes; }
int double_allocations_asked() { return asked; }
int double_allocations_refused() { return refused; }
const char *double_launched() { return launched.c_str(); }
void double_forget_launches() { launched.clear(); }

void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { kernels[host] = name; }
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream) { pushed = Call{grid, block, shared, stream}; return 0; }
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream)
{
    *grid = pushed.grid; *block = pushed.block; *shared = pushed.shared; *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void *host, Dim3, Dim3, void **, size_t, void *) { launched += kernels[host] + "\n"; return 0; }
int hipMalloc(void **out, size_t bytes)
{
    ++asked;
    if (bytes > largest) { ++refused; last_error = 2; return 2; }        // hipErrorOutOfMemory
    *out = (void *)next_address;
    next_address += (bytes + 255) & ~(size_t)255;
    return 0;
}
int hipFree(void *) { return 0; }
int hipMemset(void *, int, size_t) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
int hipGetSymbolAddress(void **out, const void *) { *out = (void *)((uintptr_t)1 << 30); return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipStreamIsCapturing(void *, int *status) { *status = capturing; return 0; }
}
