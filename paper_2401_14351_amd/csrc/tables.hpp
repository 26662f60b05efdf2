// The arguments of the index-table kernel: the sizes of a batch of consecutive
// tensors, packed by the host and unpacked on the device.
#pragma once

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdint>
#include <cstring>

namespace sllm {

// The index tables of a batch of consecutive tensors, sizes passed as kernel
// arguments, and the plan entries (device_layout.hpp) of the blocks whose first
// byte lies in the batch's slots.
constexpr uint32_t kTableBatch = 2048;  // tensors a batch holds at most
constexpr uint32_t kTableWords = 994;
struct TableArgs {
    uint64_t *size, *off, *dev;  // the layout's tables
    int64_t* plan;               // entry of block p at plan[p - p0], for p in [p0, p0 + n_plan)
    uint64_t p0, n_plan;
    uint64_t i0;                 // the batch's first tensor, at o0 in the file layout and d0 in the device layout
    uint64_t o0, d0;
    uint64_t align_o, align_d;
    uint64_t base;               // s = base + (v << shift), v the tensor's `width` bits of `words`
    uint32_t m, width, shift;
    uint32_t last;               // the batch ends the index: o_n and d_n too
    uint32_t spread;             // many plan blocks: they are spread over the grid
    uint32_t words[kTableWords];
};
static_assert(sizeof(TableArgs) <= 4096, "kernel arguments fit 4 KiB");
// bits of `words` in use: decoding reads up to two words past a value's first
constexpr uint64_t kTableBits = 32ull * (kTableWords - 2);

__host__ __device__ inline uint64_t table_size(const TableArgs& a, uint32_t j) {
    if (a.width == 0) return a.base;
    const uint64_t bit = (uint64_t)j * a.width;
    const uint32_t k = (uint32_t)(bit >> 5), sh = (uint32_t)(bit & 31);
    uint64_t v = (((uint64_t)a.words[k + 1] << 32) | a.words[k]) >> sh;
    if (sh) v |= (uint64_t)a.words[k + 2] << (64 - sh);
    if (a.width < 64) v &= (1ull << a.width) - 1;
    return a.base + (v << a.shift);
}

// Fill a.words with the first of the n sizes at s (at most kTableBatch of them)
// and return how many fit: the sizes less the smallest of them, without the low
// zero bits they share, in as many bits as the largest needs.
inline uint32_t pack_sizes(const uint64_t* s, uint64_t n, TableArgs* a) {
    uint64_t m = std::min<uint64_t>(kTableBatch, n);
    uint64_t lo = s[0], hi = s[0], diff = 0;
    for (uint64_t j = 1; j < m; ++j) {
        lo = std::min(lo, s[j]);
        hi = std::max(hi, s[j]);
        diff |= s[j] - s[0];
    }
    const uint32_t shift = diff ? (uint32_t)__builtin_ctzll(diff) : 0;
    const uint32_t width = hi == lo ? 0 : 64 - (uint32_t)__builtin_clzll((hi - lo) >> shift);
    a->base = lo;
    a->shift = shift;
    a->width = width;
    if (width == 0) return (uint32_t)m;
    m = std::min(m, kTableBits / width);
    uint64_t acc = 0;
    uint32_t fill = 0;
    uint32_t* w = a->words;
    for (uint64_t j = 0; j < m; ++j) {
        const uint64_t v = (s[j] - lo) >> shift;
        acc |= v << fill;
        if (fill + width >= 64) {
            std::memcpy(w, &acc, 8);
            w += 2;
            acc = fill ? v >> (64 - fill) : 0;
            fill = fill + width - 64;
        } else {
            fill += width;
        }
    }
    std::memcpy(w, &acc, 8);  // kTableBits leaves two words past the last value
    return (uint32_t)m;
}

}  // namespace sllm
