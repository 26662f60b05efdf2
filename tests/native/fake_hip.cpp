// A HIP runtime for host tests without a GPU: memory is host memory, copies
// are memcpy, kernels are logged and not run, and events complete at once.
// Loaded before libsllm.so with global symbols, it takes the place of the real
// runtime for that library.  The index-table kernel alone is carried out, from
// its arguments, since the host reads the tables back.  It keeps what the tests
// assert on: which blocks were allocated and freed, what was called on a
// capturing stream or on an event of a capture, and the error that stays pending
// until hipGetLastError.  Calls can be told to fail.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "device_layout.hpp"
#include "tables.hpp"

struct ihipStream_t {
    bool capturing = false;
};
struct ihipEvent_t {
    bool captured = false;  // recorded in a stream that was capturing
};

namespace {

std::map<uintptr_t, size_t> device_mem;
uint64_t n_malloc, n_free, n_launch, n_record_captured, n_bad_calls, n_wait, n_spread;
uint64_t device_limit = UINT64_MAX, device_used;
uint64_t corrupt = UINT64_MAX;  // 3 i + {0, 1, 2}: the table kernel writes a wrong o, d or s of tensor i
int64_t fail_launch = -1;  // the launch after this many more fails
std::string bad_calls;     // what was called on a capturing stream or a captured event
hipError_t pending = hipSuccess;
std::map<const void*, std::string> kernels;
std::string last_kernel;
struct {
    dim3 grid, block;
    size_t shmem;
    hipStream_t stream;
} call;

hipError_t err(hipError_t e) {
    if (e != hipSuccess) pending = e;
    return e;
}

bool capturing(hipStream_t s) { return s && s->capturing; }
int n_capturing;  // streams the test put in capture

hipError_t bad(const char* what, hipError_t e) {
    ++n_bad_calls;
    bad_calls += std::string(what) + ";";
    return err(e);
}

// the index-table kernel's work, one tensor after another
void run_tables(const sllm::TableArgs& a) {
    n_spread += a.spread;
    uint64_t o = a.o0, d = a.d0;
    for (uint32_t j = 0; j < a.m; ++j) {
        const uint64_t s = sllm::table_size(a, j), i = a.i0 + j;
        a.size[i] = s + (corrupt == 3 * i + 2);
        a.off[i] = o + (corrupt == 3 * i);
        a.dev[i] = d + (corrupt == 3 * i + 1);
        const uint64_t d_end = d + ((s + a.align_d - 1) & ~(a.align_d - 1));
        for (uint64_t p = (d + sllm::kPlanBytes - 1) / sllm::kPlanBytes; p * sllm::kPlanBytes < d_end; ++p)
            if (p >= a.p0 && p - a.p0 < a.n_plan)
                a.plan[p - a.p0] = (p + 1) * sllm::kPlanBytes <= d + s ? (int64_t)(o - d) : sllm::kMixedTile + (int64_t)i;
        o += (s + a.align_o - 1) & ~(a.align_o - 1);
        d = d_end;
    }
    if (a.last) {
        a.off[a.i0 + a.m] = o + (corrupt == 3 * (a.i0 + a.m));
        a.dev[a.i0 + a.m] = d + (corrupt == 3 * (a.i0 + a.m) + 1);
    }
}

hipError_t launched(const void* f, void** args) {
    ++n_launch;
    last_kernel = kernels[f];
    if (fail_launch == 0) {
        fail_launch = -1;
        return err(hipErrorLaunchFailure);
    }
    if (fail_launch > 0) --fail_launch;
    if (kernels[f].find("k3_tables") != std::string::npos) run_tables(*static_cast<const sllm::TableArgs*>(args[0]));
    return hipSuccess;
}

}  // namespace

extern "C" {

// ---- the tests' side --------------------------------------------------------
uint64_t fake_mallocs() { return n_malloc; }
uint64_t fake_frees() { return n_free; }
uint64_t fake_launches() { return n_launch; }
uint64_t fake_used() { return device_used; }
uint64_t fake_records_captured() { return n_record_captured; }
uint64_t fake_waits() { return n_wait; }
uint64_t fake_spread() { return n_spread; }  // table launches whose plan is spread over the grid
uint64_t fake_bad_calls() { return n_bad_calls; }
const char* fake_bad_list() { return bad_calls.c_str(); }
const char* fake_last_kernel() { return last_kernel.c_str(); }
int fake_pending() { return (int)pending; }
void fake_limit(uint64_t bytes) { device_limit = bytes; }
void fake_fail_launch(int64_t after) { fail_launch = after; }
void fake_corrupt(uint64_t what) { corrupt = what; }
void* fake_stream() { return new ihipStream_t; }
void fake_capture(void* s, int on) {
    bool& now = static_cast<ihipStream_t*>(s)->capturing;
    n_capturing += (on != 0) - now;
    now = on != 0;
}
void* fake_device_alloc(uint64_t n) {
    void* p = nullptr;
    return hipMalloc(&p, n) == hipSuccess ? p : nullptr;
}

// The n sizes packed and unpacked batch by batch; each batch's count and width.
uint64_t fake_pack(const uint64_t* s, uint64_t n, uint64_t* unpacked, uint64_t* counts, uint64_t* widths) {
    uint64_t batches = 0;
    sllm::TableArgs a{};
    for (uint64_t i = 0; i < n; i += a.m, ++batches) {
        std::memset(a.words, 0xA5, sizeof a.words);  // an earlier batch's
        a.m = sllm::pack_sizes(s + i, n - i, &a);
        counts[batches] = a.m;
        widths[batches] = a.width;
        for (uint32_t j = 0; j < a.m; ++j) unpacked[i + j] = sllm::table_size(a, j);
    }
    return batches;
}

// ---- memory -------------------------------------------------------------------
hipError_t hipMalloc(void** p, size_t n) {
    *p = nullptr;
    if (n_capturing) return bad("hipMalloc", hipErrorStreamCaptureUnsupported);
    if (n > device_limit || device_used > device_limit - n) return err(hipErrorOutOfMemory);
    *p = std::aligned_alloc(4096, (n + 4095) / 4096 * 4096);
    device_mem[(uintptr_t)*p] = n;
    device_used += n;
    ++n_malloc;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (n_capturing && p) return bad("hipFree", hipErrorStreamCaptureUnsupported);
    auto it = device_mem.find((uintptr_t)p);
    if (it == device_mem.end()) return p ? err(hipErrorInvalidValue) : hipSuccess;
    device_used -= it->second;
    device_mem.erase(it);
    std::free(p);
    ++n_free;
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::aligned_alloc(4096, (n + 4095) / 4096 * 4096);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
    *d = h;
    return hipSuccess;
}
static std::map<uintptr_t, size_t>::iterator holder(const void* p) {
    auto it = device_mem.upper_bound((uintptr_t)p);
    if (it == device_mem.begin()) return device_mem.end();
    --it;
    return (uintptr_t)p < it->first + it->second ? it : device_mem.end();
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    if (holder(p) == device_mem.end()) return err(hipErrorInvalidValue);
    std::memset(a, 0, sizeof *a);
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* n, hipDeviceptr_t p) {
    auto it = holder(p);
    if (it == device_mem.end()) return err(hipErrorInvalidValue);
    *base = (void*)it->first;
    *n = it->second;
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    if (n_capturing) return bad("hipMemcpy", hipErrorStreamCaptureImplicit);
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    if (!capturing(st)) std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyWithStream(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    if (capturing(st)) return bad("hipMemcpyWithStream", hipErrorStreamCaptureUnsupported);
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
    static void* scratch = std::aligned_alloc(4096, 16 << 20);
    *p = scratch;
    return hipSuccess;
}

// ---- device, errors -----------------------------------------------------------
hipError_t hipGetDeviceCount(int* n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() {
    const hipError_t e = pending;
    pending = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "an error"; }

// ---- streams, events ----------------------------------------------------------
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = new ihipStream_t;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    delete s;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    ++n_wait;
    return capturing(s) ? bad("hipStreamSynchronize", hipErrorStreamCaptureUnsupported) : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    *st = capturing(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    if (e->captured && s) s->capturing = true;  // the stream joins the capture
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = new ihipEvent_t;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    delete e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    e->captured = capturing(s);
    if (e->captured) ++n_record_captured;
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    return e->captured ? bad("hipEventQuery", hipErrorCapturedEvent) : hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    return e->captured ? bad("hipEventSynchronize", hipErrorCapturedEvent) : hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 0;
    return hipSuccess;
}

// ---- launches -----------------------------------------------------------------
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t s) {
    call = {grid, block, shmem, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* s) {
    *grid = call.grid;
    *block = call.block;
    *shmem = call.shmem;
    *s = call.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t) {
    return grid.x ? launched(f, args) : err(hipErrorInvalidConfiguration);
}
hipError_t hipExtLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t s, hipEvent_t, hipEvent_t end,
                              int) {
    if (end && capturing(s)) return bad("hipExtLaunchKernel with an event", hipErrorStreamCaptureUnsupported);
    if (end) end->captured = false;
    return launched(f, args);
}
void** __hipRegisterFatBinary(const void*) {
    static void* h;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    kernels[f] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
}
