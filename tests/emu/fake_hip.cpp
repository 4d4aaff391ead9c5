// A HIP runtime for the CPU that launches nothing: memory calls work on host
// memory and every kernel launch is recorded, so that tests can check what the
// library's host code enqueues (kernels, grids, order) and how it takes a
// refused launch.  Loaded before libescg.so, whose HIP calls then end here.
#include <hip/hip_runtime_api.h>
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Launch {
    std::string name;
    uint32_t cooperative, grid, block, lds;
};
std::vector<Launch> launches;
std::map<const void *, std::string> kernels;
std::map<const void *, size_t> variables;
uint32_t refuse_from = ~0u; // cooperative launches from this one on fail
uint32_t cooperative = 0;
bool capturing = false;
size_t lds_bytes = 160 * 1024; // of a CU
// What a device-to-host copy of `row_words`-word count rows holds: every
// species alive, but in rows `stop_row` and after of the copy.
uint32_t row_words = 0, stop_row = ~0u;
uint64_t allocated = 0; // bytes of all stream-ordered allocations
dim3 call_grid, call_block;
size_t call_lds;
hipStream_t call_stream;

hipError_t record(const void *f, dim3 g, dim3 b, size_t lds, bool coop)
{
    launches.push_back({kernels[f], coop, g.x * g.y * g.z, b.x * b.y * b.z,
                        (uint32_t)lds});
    return hipSuccess;
}
} // namespace

extern "C" {
// ---- for the tests
void fake_lds(uint32_t bytes) { lds_bytes = bytes; } // before any other call
void fake_reset(uint32_t refuse, uint32_t capture, uint32_t words,
                uint32_t stop)
{
    launches.clear();
    allocated = 0;
    refuse_from = refuse;
    cooperative = 0;
    capturing = capture != 0;
    row_words = words;
    stop_row = stop;
}
uint64_t fake_allocated() { return allocated; }
uint32_t fake_launches() { return (uint32_t)launches.size(); }
const char *fake_launch(uint32_t i, uint32_t *out)
{
    const Launch &l = launches[i];
    out[0] = l.cooperative;
    out[1] = l.grid;
    out[2] = l.block;
    out[3] = l.lds;
    return l.name.c_str();
}

// ---- the runtime
void **__hipRegisterFatBinary(const void *)
{
    static void *module;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name,
                           unsigned, void *, void *, dim3 *, dim3 *, int *)
{
    kernels[host] = name;
}
void __hipRegisterVar(void **, void *var, char *, char *, int, size_t size,
                      int, int)
{
    variables[var] = size;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds,
                                      hipStream_t st)
{
    call_grid = g;
    call_block = b;
    call_lds = lds;
    call_stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds,
                                     hipStream_t *st)
{
    *g = call_grid;
    *b = call_block;
    *lds = call_lds;
    *st = call_stream;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int)
{
    std::memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = lds_bytes;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int)
{
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorName(hipError_t) { return "hipErrorFake"; }
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
// events: recorded among the launches, the event's number as their grid
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    static uintptr_t events = 0;
    *e = reinterpret_cast<hipEvent_t>(++events);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    launches.push_back({"event record", 0, (uint32_t)(uintptr_t)e, 0, 0});
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t e, unsigned)
{
    launches.push_back({"event wait", 0, (uint32_t)(uintptr_t)e, 0, 0});
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t)
{
    allocated += n;
    *p = std::calloc(1, n + 256);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFreeAsync(void *p, hipStream_t)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *var)
{
    static std::map<const void *, void *> at;
    if (!at[var])
        at[var] = std::calloc(1, variables[var]);
    *p = at[var];
    return hipSuccess;
}
hipError_t hipMemcpyFromSymbol(void *dst, const void *, size_t n, size_t,
                               hipMemcpyKind)
{
    std::memset(dst, 0, n);
    return hipSuccess;
}
hipError_t hipMemcpyToSymbol(const void *, const void *, size_t, size_t,
                             hipMemcpyKind)
{
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n,
                          hipMemcpyKind kind, hipStream_t)
{
    std::memcpy(dst, src, n);
    if (kind == hipMemcpyDeviceToHost && row_words && n > 8) {
        uint32_t *w = static_cast<uint32_t *>(dst);
        for (size_t i = 0; i < n / 4; ++i)
            w[i] = i / row_words < stop_row || i % row_words == 0 ? 5u : 0u;
    }
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *,
                                                        int block, size_t lds)
{
    // the kernels' registers: four waves a SIMD
    *n = (int)std::min<size_t>(1024 / block, lds_bytes / (lds + 2048));
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds,
                           hipStream_t)
{
    return record(f, g, b, lds, false);
}
hipError_t hipLaunchCooperativeKernel(const void *f, dim3 g, dim3 b, void **,
                                      unsigned lds, hipStream_t)
{
    if (cooperative++ >= refuse_from)
        return hipErrorCooperativeLaunchTooLarge;
    return record(f, g, b, lds, true);
}
} // extern "C"
