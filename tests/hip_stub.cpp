// CPU stand-in for the HIP runtime calls of the library, for tests of what it allocates: "device" memory comes out of a
// budget, kernels do nothing.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <unordered_map>

static std::unordered_map<void *, size_t> blocks;
static size_t used = 0, budget = SIZE_MAX;
static int capturing = 0, device_waits = 0, event_waits = 0;

extern "C" {
size_t stub_used() { return used; }
void stub_budget(size_t bytes) { budget = bytes; }
void stub_capturing(int on) { capturing = on; }
int stub_device_waits() { return device_waits; }
int stub_event_waits() { return event_waits; }

int hipMalloc(void **p, size_t n)
{
    if (n > budget || used > budget - n) {
        *p = nullptr;
        return 2;                                    // hipErrorOutOfMemory
    }
    *p = calloc(n ? n : 1, 1);
    blocks[*p] = n;
    used += n;
    return 0;
}
int hipFree(void *p)
{
    const auto it = blocks.find(p);
    if (it == blocks.end())
        return p ? 1 : 0;
    used -= it->second;
    blocks.erase(it);
    free(p);
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(n ? n : 1, 1); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpy(void *to, const void *from, size_t n, int) { memcpy(to, from, n); return 0; }
int hipMemcpyAsync(void *to, const void *from, size_t n, int, void *) { memcpy(to, from, n); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipDeviceSynchronize() { ++device_waits; return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamIsCapturing(void *, int *s) { *s = capturing; return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipEventCreate(void **e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { ++event_waits; return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "stub"; }
int hipFuncGetAttributes(void *a, const void *) { memset(a, 0, 56); return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipLaunchKernel(const void *, ...) { return 0; }
int __hipPushCallConfiguration(...) { return 0; }
int __hipPopCallConfiguration(...) { return 0; }
}
