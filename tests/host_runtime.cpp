// A HIP runtime without a device, for host tests of libscocg.so: memory is addresses that are counted but
// not backed, copies to the host give one repeated 32-bit word, launches are recorded and do nothing.
// Loaded before the library with its symbols global, so the library's calls come here.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

namespace {
struct Launch {
    std::string name;
    dim3 grid, block;
};
std::mutex mu;
std::map<const void *, std::string> names;
std::vector<Launch> launches;
std::map<uintptr_t, size_t> blocks;
uintptr_t next_address = 1ull << 44;
size_t live = 0, limit = ~(size_t)0;
int frees = 0, refused = 0;
uint32_t word = 0;
int new_fails_after_sync = 0;
thread_local bool new_fails = false;
// the runtime's own records
struct Recording {
    std::lock_guard<std::mutex> lock{mu};
    bool was = new_fails;
    Recording() { new_fails = false; }
    ~Recording() { new_fails = was; }
};
// one object stands for every stream, event and graph
char handle;
}  // namespace

extern "C" {

// ---- what a test sets and reads ----
void fake_set_word(uint32_t w) { word = w; }
void fake_set_limit(size_t bytes) { limit = bytes; }
void fake_new_fails_after_sync(int on) { new_fails_after_sync = on; new_fails = false; }
size_t fake_live(void) { return live; }
int fake_frees(void) { return frees; }
int fake_refused(void) { return refused; }
void fake_forget(void) { launches.clear(); }
int fake_launches(void) { return (int)launches.size(); }
const char *fake_name(int i) { return launches[i].name.c_str(); }
// threads of launch i along x
uint64_t fake_threads_x(int i) { return (uint64_t)launches[i].grid.x * launches[i].block.x; }

// ---- the runtime ----
hipError_t hipMalloc(void **ptr, size_t size)
{
    Recording rec;
    if (live + size > limit) {
        ++refused;
        return hipErrorOutOfMemory;
    }
    *ptr = (void *)next_address;
    blocks[next_address] = size;
    next_address += (size + 4095) / 4096 * 4096 + 4096;
    live += size;
    return hipSuccess;
}
hipError_t hipFree(void *ptr)
{
    Recording rec;
    auto b = blocks.find((uintptr_t)ptr);
    if (b == blocks.end()) abort();
    live -= b->second;
    ++frees;
    blocks.erase(b);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **ptr, size_t size, unsigned int)
{
    *ptr = calloc(1, size);
    return *ptr ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *ptr)
{
    free(ptr);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *, size_t size, hipMemcpyKind kind, hipStream_t)
{
    if (kind == hipMemcpyDeviceToHost)
        for (size_t i = 0; i + 4 <= size; i += 4) memcpy((char *)dst + i, &word, 4);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t)
{
    if (new_fails_after_sync) new_fails = true;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int) { return *s = (hipStream_t)&handle, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return *g = (hipGraph_t)&handle, hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    return *e = (hipGraphExec_t)&handle, hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t)&handle, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = (hipEvent_t)&handle, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 0.f, hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetSymbolAddress(void **p, const void *) { return *p = (void *)(1ull << 43), hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    memset(a, 0, sizeof(*a));
    a->type = hipMemoryTypeDevice;
    a->devicePointer = (void *)p;
    return hipSuccess;
}

void **__hipRegisterFatBinary(const void *) { return (void **)&handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned int, void *, void *, void *, void *,
                           int *)
{
    names[f] = name;
}
static thread_local struct {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
} call;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream)
{
    call = {grid, block, shared, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream)
{
    *grid = call.grid;
    *block = call.block;
    *shared = call.shared;
    *stream = call.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t, hipStream_t)
{
    Recording rec;
    launches.push_back({names[f], grid, block});
    return hipSuccess;
}
}

// operator new that can be made to fail (see fake_new_fails_after_sync)
void *operator new(size_t size)
{
    if (new_fails) throw std::bad_alloc();
    if (void *p = malloc(size ? size : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
