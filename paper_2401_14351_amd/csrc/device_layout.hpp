// Device layouts with their own alignment A2: tensor i of the partition goes
// to d_i = sum_{j<i} align_up(s_j, A2) of the device buffer, zero padded (the
// closed form of Sec. 4.1's aligned packing, applied with A2).
//
// The device keeps the index as three u64 tables (file offsets o, sizes s and
// device offsets d, both offsets computed on the GPU by wave64 prefix sums) and
// a scatter kernel moves a window [x0, x1) of partition bytes to the device
// bytes that window owns: the data bytes whose source lies in the window plus
// the padding after every tensor whose last byte lies in it.  Windows that
// tile [0, T) therefore write every byte of [0, T2) exactly once.
#pragma once

#include <hip/hip_runtime_api.h>

#include <climits>
#include <cstdint>

#include "format.hpp"

namespace sllm {

// Device memory that outlives the handle that took it: a block given back stays
// idle, up to kMaxIdleBlockBytes and kMaxIdleBlocks a device, for the next
// handle, so opening and closing a handle per load costs no allocation and no
// hipFree (which waits for the whole device), unless its blocks do not fit
// (the staging of large copy-engine loads by four streams or more).  A block may
// be given back once no work uses it.  An allocation that fails frees the idle
// blocks and tries again.  Safe from several threads.
struct DeviceBlock {
    int device = 0;
    uint8_t* p = nullptr;
    uint64_t bytes = 0;  // capacity
};
constexpr uint64_t kMaxIdleBlockBytes = 256ull << 20;
constexpr size_t kMaxIdleBlocks = 32;
int32_t block_take(int device, uint64_t bytes, DeviceBlock* out);  // `device` is current
void block_give(DeviceBlock* b);                                   // b's device is current

struct DeviceLayout {
    uint64_t n = 0;                 // tensors
    uint64_t total = 0;             // T: bytes of the partition image
    uint64_t dev_total = 0;         // T2: bytes of the device image
    uint64_t align = 0;             // A
    uint64_t dev_align = 0;         // A2
    uint64_t* d_off = nullptr;      // device: o_i
    uint64_t* d_size = nullptr;     // device: s_i
    uint64_t* d_dev = nullptr;      // device: d_i for i < n, d_n = T2
    const TensorRec* tensors = nullptr;  // host: the index records, n of them
    const uint64_t* h_dev = nullptr;     // host: d_i
    int64_t* d_shift = nullptr;     // device: K2's plan, one entry per kPlanBytes of the device image
    uint64_t n_shift = 0;           // entries of d_shift: ceil(T2 / kPlanBytes)
    uint8_t* staging = nullptr;     // HBM staging chunks for copy-engine loads
    uint64_t staging_stride = 0;
    DeviceBlock tables, stage;      // device memory of the tables and plan, and of the staging chunks
};

// K2 from HBM moves the device image in tiles of kTileBytes (one 16-byte
// vector for each of kK2Lanes lanes) or twice that, one per workgroup.  Its plan
// holds, for each block of kPlanBytes, the shift o_m - d_m from a destination
// byte to its partition byte when the block lies inside the data bytes of one
// tensor m, or kMixedTile + m when it meets a boundary or padding and its first
// byte lies in the slot of tensor m (entries below kMixedEnd: a shift is at
// most the size of an image).
constexpr uint32_t kK2Lanes = 512;
constexpr uint64_t kTileBytes = (uint64_t)kK2Lanes * 16;
constexpr uint64_t kPlanBytes = 16384;
static_assert(kPlanBytes == 2 * kTileBytes, "a tile of either size lies in one plan block");
constexpr int64_t kMixedTile = INT64_MIN;
constexpr int64_t kMixedEnd = INT64_MIN / 2;

// Compute the tables and K2's plan on the device for the layout of `ix` at
// dev_align (host offsets dev_off, dev_total bytes; both arguments must outlive
// the layout), with `staging_chunks` HBM chunks of `chunk` bytes when asked.
// The tables are complete on return and were read back and compared with the
// host's.  The current device must be `device`.
int32_t device_layout_build(const IndexData& ix, int device, const uint64_t* dev_off, uint64_t dev_total,
                            uint64_t dev_align, uint64_t staging_chunks, uint64_t chunk, DeviceLayout* out);
// Give the layout's blocks back (park: no work may use them any more) or free
// them, which waits for the device.  Its device must be current.
void device_layout_free(DeviceLayout* l, bool park);

// Move partition window [x0, x1), held contiguously at `src` (device memory,
// or a device-visible mapping of pinned host memory), into the device image.
// With `end` (device memory sources only) that event completes with the last
// kernel, by the kernel's own completion signal: no packet of its own follows
// on the stream, and no system-scope fence.
int32_t launch_scatter_window(const DeviceLayout& l, uint8_t* dst, const uint8_t* src, uint64_t x0, uint64_t x1,
                              bool src_is_host, hipStream_t stream, hipEvent_t end = nullptr);

// Move the whole partition, held in pinned chunks listed by `table` (device
// array; chunk k holds partition bytes [kC, kC + C)), into the device image.
int32_t launch_scatter_table(const DeviceLayout& l, uint8_t* dst, const uint8_t* const* table, uint64_t chunk,
                             hipStream_t stream);

// Up to this many chunks, each from its own slot, in one scatter launch.
constexpr uint32_t kScatterBatch = 64;

// Move the run of m (<= kScatterBatch) consecutive chunks k0 .. k0 + m - 1,
// chunk k0 + j held at the device-visible host address srcs[j], into the
// device image (the window [k0 C, min((k0 + m) C, T))).
int32_t launch_scatter_run(const DeviceLayout& l, uint8_t* dst, const uint8_t* const* srcs, uint64_t k0, uint32_t m,
                           uint64_t chunk, hipStream_t stream);

// The allocation-free repack works in a fixed device area of
// kNoAllocScratchBytes per device: the sizes s_i, the file offsets o_i and the
// device offsets d_i (n + 1 entries each for the two scans) of at most
// kNoAllocMaxTensors tensors, then K2's plan for one window of the device
// image (kNoAllocPlanEntries blocks of kPlanBytes, 28 GiB).
constexpr uint64_t kNoAllocScratchBytes = SLLM_NOALLOC_SCRATCH_BYTES;
constexpr uint64_t kNoAllocMaxTensors = SLLM_NOALLOC_MAX_TENSORS;
constexpr uint64_t kNoAllocSizeOffset = 0;
constexpr uint64_t kNoAllocFileOffset = kNoAllocSizeOffset + 8 * kNoAllocMaxTensors;
constexpr uint64_t kNoAllocDevOffset = kNoAllocFileOffset + 8 * (kNoAllocMaxTensors + 1);
constexpr uint64_t kNoAllocPlanOffset = 2ull << 20;
constexpr uint64_t kNoAllocPlanEntries = (kNoAllocScratchBytes - kNoAllocPlanOffset) / sizeof(int64_t);
static_assert(kNoAllocDevOffset + 8 * (kNoAllocMaxTensors + 1) <= kNoAllocPlanOffset, "tables fit before the plan");

// Repack the file-layout image at src (T = ix.total bytes) into dst (T2 =
// dev_total bytes at alignment dev_align) with every device table in the
// scratch area: no allocation.  Calls that overlap on one device race for
// that area.  The current device must be `device`.
int32_t repack_noalloc(const IndexData& ix, int device, uint64_t dev_align, uint64_t dev_total, const uint8_t* src,
                       uint8_t* dst, hipStream_t stream);

}  // namespace sllm
