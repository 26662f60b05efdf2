// gfx950 kernels for device layouts with alignment A2.
//
// K3  index tables: o and d are the exclusive prefix sums of align_up(s_i, A)
//     and align_up(s_i, A2), scanned on the device from sizes that travel as
//     kernel arguments, about 2,000 tensors a launch, together with K2's plan.
// K2  index-driven scatter from HBM (the repack of a file-layout image, and
//     copy-engine loads staged in HBM): destination-driven, one 8 or 16 KiB
//     tile of the device image per workgroup of 512 lanes, in dispatch order.
//     The plan gives, per 16 KiB block of the device image, the shift from a
//     destination byte to its partition byte when the block lies inside one
//     tensor's data; such tiles copy after a single table load.  The waves of
//     the other tiles start from the tensor the plan names.
// K1-scatter (mapped pinned host source): each workgroup walks a span of
//     tiles, finds the tensors whose slots meet a tile (a forward search of
//     d), stages those index entries in LDS and keeps them for the following
//     tiles they still cover; every lane produces aligned 16-byte destination
//     vectors: a straight 16-byte load when source and destination agree mod
//     16, two aligned loads and a byte funnel shift when they do not, zeros for
//     padding.  Only vectors cut by the window's first or last destination byte
//     are written byte by byte.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <mutex>
#include <vector>

#include "common.hpp"
#include "device_layout.hpp"
#include "hip_util.hpp"
#include "tables.hpp"

namespace sllm {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kThreads = 256;
constexpr uint32_t kLdsEntries = 256;                          // index entries staged per tile

// ---------------------------------------------------------------------------
// K3
// ---------------------------------------------------------------------------

// x of another lane by a DPP move (0 in the lanes the control or the row mask leave out)
template <int Ctrl, int RowMask>
__device__ __forceinline__ uint64_t dpp64(uint64_t x) {
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, Ctrl, RowMask, 0xF, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), Ctrl, RowMask, 0xF, false);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t readlane64(uint64_t x, uint32_t lane) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// inclusive scan across the 64 lanes of a wave: shifts by 1, 2, 4 and 8 inside
// the rows of 16, then lane 15 of each row into the next and lane 31 into the
// upper half.  Register moves, where shuffles by lane address go through LDS.
__device__ __forceinline__ uint64_t wave_scan(uint64_t x) {
    x += dpp64<0x111, 0xF>(x);  // row_shr:1
    x += dpp64<0x112, 0xF>(x);  // row_shr:2
    x += dpp64<0x114, 0xF>(x);  // row_shr:4
    x += dpp64<0x118, 0xF>(x);  // row_shr:8
    x += dpp64<0x142, 0xA>(x);  // row_bcast:15 into rows 1 and 3
    x += dpp64<0x143, 0xC>(x);  // row_bcast:31 into rows 2 and 3
    return x;
}

// The plan entry of the block at destination byte y, whose first byte lies in
// the slot of tensor m.
__device__ __forceinline__ int64_t plan_entry(uint64_t y, uint64_t dm, uint64_t om, uint64_t sm, uint64_t m) {
    return y + kPlanBytes <= dm + sm ? (int64_t)(om - dm) : kMixedTile + (int64_t)m;
}

// Whether a batch of m tensors of sizes s and `blocks` plan blocks has its plan
// spread over a grid (k3_tables): beyond four blocks a tensor, and from one on
// where more than 4 % of the tensors hold more than kTableRun blocks ("runs",
// counted only there: a small batch's call is bound by the host).  Tensor by
// tensor such a run goes round its wave of 128 tensors alone, and the longest of
// the others holds up the lanes beside it; where all are short, or few are long,
// it saves the grid's bisection.  Allocation-free repacks, spread / tensor by
// tensor, sizes log-uniform from 256 B, 20,000 tensors: mean 0.7 blocks 123.1 /
// 118.6 us, 1.0 160.7 / 160.1, 1.3 (no runs) 199.3 / 203.5, 1.6 (4 % runs) 227.1
// / 240.7, 1.8 (6 %) 252.9 / 278.1, 2.3 (10 %) 303.0 / 350.3, 4.2 (20 %) 488.8 /
// 576.3; 150 to 1,000 tensors: 1.3 0.4-0.7 us longer, 1.8 0-1.2 and 2.3 0.9-2.9
// us shorter.  Sizes within 50 % of their mean, so no runs, 20,000 and 300
// tensors: 1.0 blocks 156.3 / 148.8, 3.0 374.5 / 379.5 and 9.5 / 8.7, 4.0 470.4 /
// 485.9 and 10.2 / 9.4.  2 % of 1 MiB among small ones, mean 1.4: 232.7 / 226.2.
constexpr uint64_t kTableRun = 8;
bool spread_plan(uint64_t blocks, const uint64_t* s, uint64_t m) {
    if (blocks <= m || blocks > 4 * m) return blocks > m;
    uint64_t runs = 0;
    for (uint64_t j = 0; j < m; ++j) runs += s[j] > kTableRun * kPlanBytes;
    return 25 * runs > m;
}

// One workgroup decodes the sizes, scans both layouts' padded sizes (two
// tensors a lane, a scan in each wave, the 16 wave totals through LDS) and
// writes the batch's tables.  Batches do not wait for each other's scan: the
// host passes where each starts.  The plan follows in one of two ways: tensor
// by tensor from the registers where the batch has few blocks (a.spread == 0,
// one workgroup; a run of more than kTableRun blocks goes round the wave), else every
// workgroup of a larger grid repeats the scan, leaves d, o and s in LDS and
// takes its share of the blocks, each by bisection of d.
//
// All of it is latency, so fewer launches and shorter chains count: 20,000
// tensors of 256 B to 64 KiB need 11 launches of these (16 bits a size), where
// 256 64-bit sizes a launch, a scan kernel per layout and a plan kernel took
// 82: the repack they prepare went from 336 to 139 us, and to 134 with the plan
// from registers and no second barrier.  Of a launch's 5.3 us by bisection, 2.0
// were the launch and its arguments, 0.6 the sizes, 1.3 the scans and 1.4 the
// plan.
__global__ __launch_bounds__(1024) void k3_tables(TableArgs a) {
    __shared__ uint64_t s_dev[kTableBatch], s_off[kTableBatch], s_size[kTableBatch];
    __shared__ uint64_t tot_o[16], tot_d[16];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t j0 = 2 * tid, j1 = j0 + 1;
    const uint64_t s0 = j0 < a.m ? table_size(a, j0) : 0, s1 = j1 < a.m ? table_size(a, j1) : 0;
    const uint64_t o_first = (s0 + a.align_o - 1) & ~(a.align_o - 1), d_first = (s0 + a.align_d - 1) & ~(a.align_d - 1);
    const uint64_t o_both = o_first + ((s1 + a.align_o - 1) & ~(a.align_o - 1));
    const uint64_t d_both = d_first + ((s1 + a.align_d - 1) & ~(a.align_d - 1));
    const uint64_t o_incl = wave_scan(o_both), d_incl = wave_scan(d_both);
    if (lane == 63) {
        tot_o[wave] = o_incl;
        tot_d[wave] = d_incl;
    }
    __syncthreads();
    // every wave scans the 16 totals for itself
    const uint64_t o_tot = wave_scan(lane < 16 ? tot_o[lane] : 0), d_tot = wave_scan(lane < 16 ? tot_d[lane] : 0);
    const uint32_t w = __builtin_amdgcn_readfirstlane(wave);
    const uint64_t o = a.o0 + (w ? readlane64(o_tot, w - 1) : 0) + o_incl - o_both;
    const uint64_t d = a.d0 + (w ? readlane64(d_tot, w - 1) : 0) + d_incl - d_both;
    const uint64_t o_end = a.o0 + readlane64(o_tot, 15), d_end = a.d0 + readlane64(d_tot, 15);
    if (blockIdx.x == 0) {
        if (j0 < a.m) {
            a.size[a.i0 + j0] = s0;
            a.off[a.i0 + j0] = o;
            a.dev[a.i0 + j0] = d;
        }
        if (j1 < a.m) {
            a.size[a.i0 + j1] = s1;
            a.off[a.i0 + j1] = o + o_first;
            a.dev[a.i0 + j1] = d + d_first;
        }
        if (a.last && tid == 0) {
            a.off[a.i0 + a.m] = o_end;
            a.dev[a.i0 + a.m] = d_end;
        }
    }
    // blocks p with d0 <= p * kPlanBytes < d_end, inside the plan's window
    const uint64_t w_begin = a.p0, w_end = a.p0 + a.n_plan;
    if (!a.spread) {
        auto fill = [&](uint64_t dm, uint64_t slot, uint64_t om, uint64_t sm, uint64_t m) {
            uint64_t p = (dm + kPlanBytes - 1) / kPlanBytes, p_end = (dm + slot + kPlanBytes - 1) / kPlanBytes;
            if (p < w_begin) p = w_begin;
            if (p_end > w_end) p_end = w_end;
            const bool run = p_end > p && p_end - p > kTableRun;
            if (!run)
                for (uint64_t b = p; b < p_end; ++b) a.plan[b - a.p0] = plan_entry(b * kPlanBytes, dm, om, sm, m);
            for (uint64_t left = __ballot(run); left; left &= left - 1) {
                const uint32_t k = __builtin_ctzll(left);
                const uint64_t dk = readlane64(dm, k), ok = readlane64(om, k), sk = readlane64(sm, k), mk = readlane64(m, k);
                const uint64_t pk = readlane64(p, k), ek = readlane64(p_end, k);
                for (uint64_t b = pk + lane; b < ek; b += 64) a.plan[b - a.p0] = plan_entry(b * kPlanBytes, dk, ok, sk, mk);
            }
        };
        fill(d, d_first, o, s0, a.i0 + j0);
        fill(d + d_first, d_both - d_first, o + o_first, s1, a.i0 + j1);
        return;
    }
    s_off[j0] = o;
    s_dev[j0] = d;
    s_size[j0] = s0;
    s_off[j1] = o + o_first;
    s_dev[j1] = d + d_first;
    s_size[j1] = s1;
    __syncthreads();
    uint64_t p = (a.d0 + kPlanBytes - 1) / kPlanBytes, p_end = (d_end + kPlanBytes - 1) / kPlanBytes;
    if (p < w_begin) p = w_begin;
    if (p_end > w_end) p_end = w_end;
    for (p += (uint64_t)blockIdx.x * 1024 + tid; p < p_end; p += (uint64_t)gridDim.x * 1024) {
        const uint64_t y = p * kPlanBytes;
        uint32_t l = 0, h = a.m - 1;  // d of the batch's first tensor <= y
        while (l < h) {
            const uint32_t mid = (l + h + 1) >> 1;
            if (s_dev[mid] <= y) l = mid;
            else h = mid - 1;
        }
        a.plan[p - a.p0] = plan_entry(y, s_dev[l], s_off[l], s_size[l], a.i0 + l);
    }
}

// ---------------------------------------------------------------------------
// K2 / K1-scatter
// ---------------------------------------------------------------------------

struct ScatterArgs {
    uint8_t* dst;
    const uint64_t* off;   // o_i
    const uint64_t* size;  // s_i
    const uint64_t* dev;   // d_i, d_n = T2
    uint64_t n;
    uint64_t y0, y1;       // destination bytes written by this launch
    uint64_t tile0, n_tiles;
    // source: a contiguous window ...
    const uint8_t* base;   // partition byte x at base[x - x0]
    uint64_t x0, x1;
    // ... or a table of chunks
    const uint8_t* const* table;  // partition byte x at table[x / chunk][x % chunk]
    uint64_t chunk;
    // ... or a run of chunks passed inline (run_n > 0): byte x of chunk
    // k = x / chunk at run_src[k - run_k0][x % chunk], for x in [x0, x1)
    uint32_t run_n;
    uint64_t run_k0;
    const uint8_t* run_src[kScatterBatch];
    uint64_t total;        // T
    uint32_t vec_ok;       // 16-byte aligned source vectors are addressable as such
};

// K2's arguments (an HBM source is one contiguous window, named as above).
struct K2Args {
    uint8_t* dst;
    const uint64_t* off;
    const uint64_t* size;
    const uint64_t* dev;
    uint64_t n;
    uint64_t y0, y1;
    uint64_t tile0;        // first tile of the launch
    const uint8_t* base;
    uint64_t x0, x1;
    const int64_t* shift;  // the plan: entry of destination block p at shift[p - plan0]
    uint64_t plan0;
    uint32_t vec_ok;
};

// Where a launch's source bytes are: one contiguous window, a device table
// of chunks, or a run of chunks passed inline.  A kernel instance serves one
// kind, so none of them pays for the others' addressing.
enum SrcKind : int { kWindow = 0, kTable = 1, kRun = 2 };

template <SrcKind K, class Args = ScatterArgs>
struct Src {
    const Args& a;
    __device__ __forceinline__ const uint8_t* at(uint64_t x) const {
        if constexpr (K == kRun) {
            const uint64_t k = x / a.chunk;
            return a.run_src[k - a.run_k0] + (x - k * a.chunk);
        } else if constexpr (K == kTable) {
            const uint64_t k = x / a.chunk;
            return a.table[k] + (x - k * a.chunk);
        } else {
            return a.base + (x - a.x0);
        }
    }
    // can the 16-byte aligned vectors covering [x, x + len) be loaded whole?
    __device__ __forceinline__ bool vectors_ok(uint64_t xa, uint64_t len) const {
        if (!a.vec_ok) return false;
        if constexpr (K == kTable) return xa + len <= a.total;
        return xa >= a.x0 && xa + len <= a.x1;
    }
};

__device__ __forceinline__ u32x4 ld16(const uint8_t* p) { return *reinterpret_cast<const u32x4*>(p); }

// bytes [s, s + 16) of the 32 bytes lo:hi, for s in [0, 16)
__device__ __forceinline__ u32x4 funnel(u32x4 lo, u32x4 hi, uint32_t s) {
    const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    const uint32_t b = s & 3;
    u32x4 r;
    switch (s >> 2) {
        case 0: r = u32x4{__builtin_amdgcn_alignbyte(w[1], w[0], b), __builtin_amdgcn_alignbyte(w[2], w[1], b),
                          __builtin_amdgcn_alignbyte(w[3], w[2], b), __builtin_amdgcn_alignbyte(w[4], w[3], b)}; break;
        case 1: r = u32x4{__builtin_amdgcn_alignbyte(w[2], w[1], b), __builtin_amdgcn_alignbyte(w[3], w[2], b),
                          __builtin_amdgcn_alignbyte(w[4], w[3], b), __builtin_amdgcn_alignbyte(w[5], w[4], b)}; break;
        case 2: r = u32x4{__builtin_amdgcn_alignbyte(w[3], w[2], b), __builtin_amdgcn_alignbyte(w[4], w[3], b),
                          __builtin_amdgcn_alignbyte(w[5], w[4], b), __builtin_amdgcn_alignbyte(w[6], w[5], b)}; break;
        default: r = u32x4{__builtin_amdgcn_alignbyte(w[4], w[3], b), __builtin_amdgcn_alignbyte(w[5], w[4], b),
                           __builtin_amdgcn_alignbyte(w[6], w[5], b), __builtin_amdgcn_alignbyte(w[7], w[6], b)}; break;
    }
    return r;
}

// the same for an s that differs between lanes: selects instead of branches
__device__ __forceinline__ u32x4 funnel_lanes(u32x4 lo, u32x4 hi, uint32_t s) {
    const uint32_t b = s & 3;
    const bool one = s & 4, two = s & 8;  // dwords to skip: one, then two more
    const uint32_t m0 = one ? lo.y : lo.x, m1 = one ? lo.z : lo.y, m2 = one ? lo.w : lo.z, m3 = one ? hi.x : lo.w,
                   m4 = one ? hi.y : hi.x, m5 = one ? hi.z : hi.y, m6 = one ? hi.w : hi.z;
    const uint32_t q0 = two ? m2 : m0, q1 = two ? m3 : m1, q2 = two ? m4 : m2, q3 = two ? m5 : m3, q4 = two ? m6 : m4;
    return u32x4{__builtin_amdgcn_alignbyte(q1, q0, b), __builtin_amdgcn_alignbyte(q2, q1, b),
                 __builtin_amdgcn_alignbyte(q3, q2, b), __builtin_amdgcn_alignbyte(q4, q3, b)};
}

// keep bytes [0, keep) of v, zero the rest
__device__ __forceinline__ u32x4 keep_bytes(u32x4 v, uint32_t keep) {
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t lo = 4 * j;
        if (keep <= lo) w[j] = 0;
        else if (keep < lo + 4) w[j] &= (1u << (8 * (keep - lo))) - 1u;
    }
    return u32x4{w[0], w[1], w[2], w[3]};
}

__device__ __forceinline__ uint32_t byte_of(u32x4 v, uint32_t b) {
    const uint32_t w = b < 4 ? v.x : b < 8 ? v.y : b < 12 ? v.z : v.w;
    return (w >> (8 * (b & 3))) & 0xFF;
}

// largest m in [lo, hi] with d[m] <= y (d[lo] <= y holds)
__device__ __forceinline__ uint64_t owner_global(const uint64_t* d, uint64_t lo, uint64_t hi, uint64_t y) {
    while (lo < hi) {
        const uint64_t mid = lo + (hi - lo + 1) / 2;
        if (d[mid] <= y) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// the same, searching forward from `from` (d[from] <= y): gallop 1, 2, 4 ...
// entries ahead, then bisect the last step; one load when y is still in the
// slot of tensor `from`, as it is for most tiles of a large tensor
__device__ __forceinline__ uint64_t owner_from(const uint64_t* d, uint64_t from, uint64_t last, uint64_t y) {
    uint64_t lo = from, step = 1;
    while (lo < last) {
        const uint64_t probe = last - lo < step ? last : lo + step;
        if (d[probe] > y) return owner_global(d, lo, probe - 1, y);
        lo = probe;
        step <<= 1;
    }
    return lo;
}

template <bool NT>
__device__ __forceinline__ void st16(uint8_t* p, u32x4 v) {
    if constexpr (NT) {
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
    } else {
        *reinterpret_cast<u32x4*>(p) = v;
    }
}

// The destination vector at y read byte by byte: its dn data bytes from
// partition byte x on where they lie in [lo, hi), zeros elsewhere.
template <class S>
__device__ __forceinline__ u32x4 bytes_vector(const S& src, uint64_t y, uint64_t lo, uint64_t hi, uint64_t x, uint32_t dn) {
    uint64_t w0 = 0, w1 = 0;
    for (uint32_t b = 0; b < dn; ++b) {
        if (y + b < lo || y + b >= hi) continue;
        const uint64_t v = (uint64_t)*src.at(x + b) << (8 * (b & 7));
        if (b < 8) w0 |= v;
        else w1 |= v;
    }
    return u32x4{(uint32_t)w0, (uint32_t)(w0 >> 32), (uint32_t)w1, (uint32_t)(w1 >> 32)};
}

// Store the vector at y: whole, or its bytes inside [lo, hi).
template <bool NT>
__device__ __forceinline__ void put_vector(uint8_t* dst, uint64_t y, uint64_t lo, uint64_t hi, bool whole, u32x4 v) {
    if (whole) {
        st16<NT>(dst + y, v);
        return;
    }
    for (uint32_t b = 0; b < 16; ++b)
        if (y + b >= lo && y + b < hi) dst[y + b] = (uint8_t)byte_of(v, b);
}

// Index entries of the tensors meeting a tile, staged in LDS.
struct Staging {
    uint64_t dev[kLdsEntries], off[kLdsEntries], size[kLdsEntries];
    uint64_t lo, hi, next;
};

// Tiles [t_begin, t_end) of the launch, in order (tile t covers destination
// bytes [(tile0 + t) S, (tile0 + t + 1) S), S = L lanes x 16 B x U).  For
// each tile every lane first produces its U destination vectors (all source
// loads in flight together), then stores them.  The index entries of the
// tensors meeting a tile are staged in LDS together with the start of the
// next tensor's slot; while the following tiles end before that start (the
// interior of a large tensor) they reuse the staged entries, with no search,
// no staging and no barrier.  Every lane of the workgroup must call this
// with the same span (it holds barriers).
template <uint32_t L, uint32_t U, bool NT, SrcKind K>
__device__ __forceinline__ void scatter_span(const ScatterArgs& a, Staging& stg, uint64_t t_begin, uint64_t t_end) {
    constexpr uint64_t kTileU = (uint64_t)L * 16 * U;
    uint64_t* const s_dev = stg.dev;
    uint64_t* const s_off = stg.off;
    uint64_t* const s_size = stg.size;
    const Src<K> src{a};
    uint64_t cursor = 0;   // thread 0: owner of the last searched tile's last byte
    bool staged = false;   // LDS holds entries i_lo .. i_lo + cnt - 1 (uniform)
    uint64_t i_lo = 0, cnt = 0, next = 0;  // next: d of the first tensor not staged
    for (uint64_t t = t_begin; t < t_end; ++t) {
        const uint64_t yt = (a.tile0 + t) * kTileU;
        const uint64_t lo = yt > a.y0 ? yt : a.y0;
        const uint64_t hi = yt + kTileU < a.y1 ? yt + kTileU : a.y1;
        if (!staged || hi > next) {
            __syncthreads();  // every wave is done with the entries staged before
            if (threadIdx.x == 0) {
                const uint64_t first =
                    t == t_begin ? owner_global(a.dev, 0, a.n - 1, lo) : owner_from(a.dev, cursor, a.n - 1, lo);
                cursor = owner_from(a.dev, first, a.n - 1, hi - 1);
                stg.lo = first;
                stg.hi = cursor;
            }
            __syncthreads();
            i_lo = stg.lo;
            cnt = stg.hi - stg.lo + 1;
            staged = cnt <= kLdsEntries;
            if (staged)
                for (uint32_t i = threadIdx.x; i < cnt; i += L) {
                    s_dev[i] = a.dev[i_lo + i];
                    s_off[i] = a.off[i_lo + i];
                    s_size[i] = a.size[i_lo + i];
                }
            if (threadIdx.x == 0) stg.next = a.dev[i_lo + cnt];  // d[n] = T2 ends the last slot
            __syncthreads();
            next = stg.next;
        }
        u32x4 v[U];
        uint32_t whole_mask = 0, in_mask = 0;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            v[u] = u32x4{0, 0, 0, 0};
            const uint64_t y = yt + ((uint64_t)u * L + threadIdx.x) * 16;
            if (y + 16 <= lo || y >= hi) continue;
            in_mask |= 1u << u;
            uint64_t dm, om, sm;
            if (cnt == 1) {
                dm = s_dev[0]; om = s_off[0]; sm = s_size[0];
            } else if (staged) {
                uint32_t l = 0, h = (uint32_t)cnt - 1;
                while (l < h) {
                    const uint32_t mid = (l + h + 1) >> 1;
                    if (s_dev[mid] <= y) l = mid;
                    else h = mid - 1;
                }
                dm = s_dev[l]; om = s_off[l]; sm = s_size[l];
            } else {
                const uint64_t m = owner_global(a.dev, i_lo, i_lo + cnt - 1, y);
                dm = a.dev[m]; om = a.off[m]; sm = a.size[m];
            }
            const bool whole = y >= lo && y + 16 <= hi;  // vector entirely ours to write
            if (whole) whole_mask |= 1u << u;
            const uint64_t r = y - dm;                   // byte of the slot
            const uint32_t dn = sm > r ? (sm - r < 16 ? (uint32_t)(sm - r) : 16u) : 0u;  // data bytes in vector
            const uint64_t x = om + r;                   // source of the vector's first byte
            if (!dn) continue;
            const uint64_t xa = x & ~15ull;
            const uint32_t sh = (uint32_t)(x & 15);
            const uint64_t need = sh + dn > 16 ? 32 : 16;  // aligned source bytes spanned
            if (whole && src.vectors_ok(xa, need)) {
                const u32x4 v0 = ld16(src.at(xa));
                u32x4 w = sh == 0 ? v0 : funnel(v0, need == 32 ? ld16(src.at(xa + 16)) : v0, sh);
                v[u] = dn < 16 ? keep_bytes(w, dn) : w;
            } else {
                v[u] = bytes_vector(src, y, lo, hi, x, dn);
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            if (!(in_mask >> u & 1)) continue;
            const uint64_t y = yt + ((uint64_t)u * L + threadIdx.x) * 16;
            put_vector<NT>(a.dst, y, lo, hi, whole_mask >> u & 1, v[u]);
        }
    }
}

// K1-scatter (host sources): each workgroup of a persistent grid walks a
// contiguous span of tiles, so the owner of the next tile is found by
// searching forward from the last one.
template <uint32_t U, bool NT, SrcKind K>
__global__ __launch_bounds__(kThreads) void k_scatter(ScatterArgs a) {
    __shared__ Staging stg;
    const uint64_t per_block = (a.n_tiles + gridDim.x - 1) / gridDim.x;
    const uint64_t t_begin = (uint64_t)blockIdx.x * per_block;
    const uint64_t t_end = t_begin + per_block < a.n_tiles ? t_begin + per_block : a.n_tiles;
    scatter_span<kThreads, U, NT, K>(a, stg, t_begin, t_end);
}

// The calling wave's N KiB of the device image at yw, from partition byte xs
// on: one tensor's data, so xs and the shift are the same for every lane.
// False if that reads past the window; nothing is written then.
template <bool NT, int N>
__device__ __forceinline__ bool k2_straight(const K2Args& a, uint64_t yw, uint64_t xs) {
    // aligned 16-byte source vectors spanning [xs, xs + N KiB)
    const uint64_t xa0 = xs & ~15ull, xa1 = (xs + N * 1024 + 15) & ~15ull;
    if (!a.vec_ok || xa0 < a.x0 || xa1 > a.x1) return false;
    const uint32_t at = (threadIdx.x & 63) * 16, r = (uint32_t)(xs & 15);
    // partition byte x sits at base + (x - x0); base and x0 are 16-byte aligned
    const uint8_t* p = a.base + (xs - a.x0) + at - r;
    uint8_t* q = a.dst + yw + at;
    u32x4 lo[N], hi[N];
#pragma unroll
    for (int k = 0; k < N; ++k) lo[k] = ld16(p + k * 1024);
    if (r) {
#pragma unroll
        for (int k = 0; k < N; ++k) hi[k] = ld16(p + k * 1024 + 16);
#pragma unroll
        for (int k = 0; k < N; ++k) lo[k] = funnel(lo[k], hi[k], r);
    }
#pragma unroll
    for (int k = 0; k < N; ++k) st16<NT>(q + k * 1024, lo[k]);
    return true;
}

// The calling wave's N KiB at yw where they meet a boundary, padding or a
// window edge, or their plan block does.  `w` is a tensor whose slot starts at
// or before yw.  The wave loads the index entries of 64 tensors from w on in
// one go, one per lane, and finds by ballot which of them own its bytes.
// Where that is one tensor and its data cover them all, the wave copies
// straight.  Else the owners, mostly two, go round the wave by scalar lane
// reads and every lane keeps, for each of its N vectors, the last that starts
// at or before it.  Only a wave that meets (or follows, within its plan block)
// more than 64 tensors loads another 64.  What bounds it is the chain of the
// plan entry, the index entries and the data, and the vector instructions, 4
// cycles each for a wave; hence the one load of entries, the scalar case and
// no LDS or barrier.
template <bool NT, int N>
__device__ __forceinline__ void k2_mixed(const K2Args& a, uint64_t yw, uint64_t w) {
    const Src<kWindow, K2Args> src{a};
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t lo = yw > a.y0 ? yw : a.y0;
    const uint64_t hi = yw + N * 1024 < a.y1 ? yw + N * 1024 : a.y1;
    if (lo >= hi) return;
    const uint64_t y = yw + lane * 16;  // the lane's first vector; the others 1 KiB apart
    uint64_t dm[N] = {}, om[N] = {}, sm[N] = {};
    for (;;) {
        const uint64_t i = w + lane;
        const bool in = i < a.n;
        const uint64_t d = in ? a.dev[i] : ~0ull, o = in ? a.off[i] : 0, s = in ? a.size[i] : 0;
        const uint64_t next = w + 64 < a.n ? a.dev[w + 64] : ~0ull;  // start of the first slot past these
        const uint32_t before = __popcll(__ballot(d <= lo)), last = __popcll(__ballot(d < hi));
        const uint32_t first = before ? before - 1 : 0;
        if (last == first + 1 && next >= hi && hi - lo == N * 1024) {
            const uint64_t dk = readlane64(d, first);
            if (dk <= lo && hi <= dk + readlane64(s, first) &&
                k2_straight<NT, N>(a, yw, readlane64(o, first) + (lo - dk)))
                return;
        }
        for (uint32_t k = first; k < last; ++k) {
            const uint64_t dk = readlane64(d, k), ok = readlane64(o, k), sk = readlane64(s, k);
#pragma unroll
            for (int j = 0; j < N; ++j) {
                if (y + j * 1024 >= dk) {
                    dm[j] = dk;
                    om[j] = ok;
                    sm[j] = sk;
                }
            }
        }
        if (next >= hi) break;
        w += 64;
    }
    struct Vec {
        uint64_t x;   // source of its first byte
        uint32_t dn;  // data bytes in it
        bool whole;   // entirely ours to write
        bool fast;    // its source vectors v0 and v1 could be loaded whole
        u32x4 v0, v1;
    } vec[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {  // every load in flight before the first is used
        const uint64_t yj = y + j * 1024, r = yj - dm[j];  // byte of the slot
        Vec& v = vec[j];
        v.dn = sm[j] > r ? (sm[j] - r < 16 ? (uint32_t)(sm[j] - r) : 16u) : 0u;
        v.x = om[j] + r;
        v.whole = yj >= lo && yj + 16 <= hi;
        const uint64_t xa = v.x & ~15ull;
        const bool two = (v.x & 15) + v.dn > 16;  // the data span two aligned source vectors
        v.fast = v.dn && v.whole && src.vectors_ok(xa, two ? 32 : 16);
        v.v0 = v.v1 = u32x4{0, 0, 0, 0};
        if (v.fast) {
            v.v0 = ld16(src.at(xa));
            if (two) v.v1 = ld16(src.at(xa + 16));
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const uint64_t yj = y + j * 1024;
        if (yj + 16 <= lo || yj >= hi) continue;
        const Vec& v = vec[j];
        u32x4 d = {0, 0, 0, 0};
        if (v.fast) d = keep_bytes(funnel_lanes(v.v0, v.v1, (uint32_t)(v.x & 15)), v.dn);
        else if (v.dn) d = bytes_vector(src, yj, lo, hi, v.x, v.dn);
        put_vector<NT>(a.dst, yj, lo, hi, v.whole, d);
    }
}

// K2 from HBM: one destination tile of 8 N KiB per workgroup of kK2Lanes
// lanes, N KiB a wave, tiles in dispatch order, so the workgroups in flight
// sweep a contiguous window of both images (HBM serves that order best).  A
// wave whose plan block lies inside one tensor's data, and whose source bytes
// all lie in the window, copies straight from source byte y + shift: one table
// load, then the data loads.  Every other wave goes from the tensor the plan
// entry names.
//
// Four workgroups fit a CU, and the copy needs all four.  With more than 80
// SGPRs a wave (the hardware takes them in steps of 16 and keeps 16 back) only
// seven waves fit a SIMD, so three workgroups a CU: a 2.1 GB repack of straight
// tiles took 680 us with 91 SGPRs and 646 us (6.5 TB/s) with 62 to 78.
//
// N = 2 halves the chains per byte and so is for layouts whose blocks mostly
// meet boundaries (k2_two_kib); copying straight it loses, 721 against 645 us
// on those 2.1 GB.  20,000 tensors of 256 B to 64 KiB, 239 MB packed densely,
// into A2 = 256: 184 us when one lane searched d and the workgroup staged the
// entries in LDS, 98 with N = 1 and 83 (5.8 TB/s) with N = 2; N = 4 takes 92,
// and two kilobytes in a workgroup whose neighbour then ends at once 120.
template <bool NT, int N>
__global__ __launch_bounds__(kK2Lanes) __attribute__((amdgpu_num_sgpr(80))) void k2_tiles(K2Args a) {
    constexpr uint64_t kTile = N * kTileBytes;
    const uint64_t yt = (a.tile0 + blockIdx.x) * kTile;
    const uint64_t yw = yt + N * 1024 * (uint64_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t sh = a.shift[yt / kPlanBytes - a.plan0];
    if (sh < kMixedEnd) {
        k2_mixed<NT, N>(a, yw, (uint64_t)(sh - kMixedTile));
    } else if (yw < a.y0 || yw + N * 1024 > a.y1 || !k2_straight<NT, N>(a, yw, yw + (uint64_t)sh)) {
        // a straight block cut by the window's edge names no tensor: search for it
        k2_mixed<NT, N>(a, yw, owner_global(a.dev, 0, a.n - 1, yw));
    }
}

// K2's plan for destination blocks p0 .. p0 + n_blocks - 1: shift[p - p0] =
// o_m - d_m when block p (kPlanBytes) lies inside the data bytes of tensor
// m, else kMixedTile + m, m being the tensor whose slot holds its first byte.
__global__ __launch_bounds__(256) void k3_tile_shift(const uint64_t* __restrict__ dev, const uint64_t* __restrict__ off,
                                                     const uint64_t* __restrict__ size, uint64_t n, uint64_t p0,
                                                     uint64_t n_blocks, int64_t* __restrict__ shift) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n_blocks; p += stride) {
        const uint64_t y = (p0 + p) * kPlanBytes;
        const uint64_t m = owner_global(dev, 0, n - 1, y);  // d_0 = 0 <= y
        shift[p] = plan_entry(y, dev[m], off[m], size[m], m);
    }
}

// A non-negative integer from the environment, or dflt when unset or malformed.
uint32_t env_uint(const char* name, uint32_t dflt) {
    const char* s = std::getenv(name);
    if (!s || !*s) return dflt;
    char* end = nullptr;
    const long v = std::strtol(s, &end, 10);
    return (end && *end == '\0' && v >= 0) ? (uint32_t)v : dflt;
}

// first device byte owned by partition byte x: the first tensor whose data
// ends after x starts owning there (padding belongs to a tensor's last byte)
uint64_t y_of(const DeviceLayout& l, uint64_t x) {
    const TensorRec* end = l.tensors + l.n;
    const TensorRec* t = std::upper_bound(l.tensors, end, x, [](uint64_t v, const TensorRec& r) { return v < r.offset + r.nbytes; });
    if (t == end) return l.dev_total;
    return l.h_dev[t - l.tensors] + (x > t->offset ? x - t->offset : 0);
}

// Whether K2 moves 2 KiB a wave (k2_tiles): where most plan blocks (16 KiB)
// meet a boundary, so by the mean slot.  Measured, 1 against 2 KiB a wave:
// every shift a multiple of 16, mean slots of 22 KiB 181 / 171 us, 39 KiB
// 303 / 317, 69 KiB 428 / 471; through the byte funnel, which the second
// vector in flight helps too, 21 KiB 191 / 170, 37 KiB 313 / 293, 68 KiB
// 441 / 443.
bool k2_two_kib(const DeviceLayout& l) {
    const uint64_t mean = l.align % 16 == 0 ? 24 << 10 : 48 << 10;
    return l.dev_total / mean <= l.n;
}

// Launch shape, read at every launch so that one process can compare shapes:
// SLLM_K2_NT (streaming stores) and SLLM_K2_MAX_GRID (workgroups a launch)
// for HBM sources; SLLM_K2_UNROLL (8 vectors per lane, any other value 4) and
// SLLM_K1_BLOCKS / SLLM_K1_STREAM_BLOCKS (grid of a launch that moves the
// whole image / part of it, as for K1) for host sources.
int32_t launch(const DeviceLayout& l, ScatterArgs a, bool src_is_host, hipStream_t stream, uint64_t plan0 = 0,
               hipEvent_t end = nullptr) {
    a.off = l.d_off;
    a.size = l.d_size;
    a.dev = l.d_dev;
    a.n = l.n;
    a.total = l.total;
    if (a.y0 >= a.y1 || l.n == 0) return SLLM_OK;
    if (a.y1 > l.dev_total) return fail(SLLM_E_INVAL, "scatter: destination range past the image");
    if (!src_is_host) {  // HBM source (K2): one tile per workgroup
        if (!l.d_shift) return fail(SLLM_E_INVAL, "scatter: the layout has no tile plan");
        const bool nt = env_uint("SLLM_K2_NT", 1) != 0;
        K2Args k{};
        k.dst = a.dst;
        k.off = a.off;
        k.size = a.size;
        k.dev = a.dev;
        k.n = a.n;
        k.y0 = a.y0;
        k.y1 = a.y1;
        k.base = a.base;
        k.x0 = a.x0;
        k.x1 = a.x1;
        k.shift = l.d_shift;
        k.plan0 = plan0;
        k.vec_ok = a.vec_ok;
        const bool two = k2_two_kib(l);
        const uint64_t tile = two ? 2 * kTileBytes : kTileBytes;
        const uint64_t t_end = ceil_div(a.y1, tile);
        // at most 2^31 lanes a launch (SLLM_K2_MAX_GRID lowers it, to exercise
        // the split on small images)
        constexpr uint64_t kMaxGrid = (1ull << 31) / kK2Lanes;
        const uint64_t max_grid = std::max<uint64_t>(1, std::min<uint64_t>(kMaxGrid, env_uint("SLLM_K2_MAX_GRID", kMaxGrid)));
        for (uint64_t t0 = a.y0 / tile; t0 < t_end; t0 += max_grid) {
            k.tile0 = t0;
            const dim3 grid((uint32_t)std::min(max_grid, t_end - t0)), block(kK2Lanes);
            const auto kernel = two ? (nt ? k2_tiles<true, 2> : k2_tiles<false, 2>) : (nt ? k2_tiles<true, 1> : k2_tiles<false, 1>);
            if (end && t_end - t0 <= max_grid) hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, nullptr, end, 0, k);
            else kernel<<<grid, block, 0, stream>>>(k);
            SLLM_HIP(hipGetLastError());
        }
        return SLLM_OK;
    }
    // host sources are PCIe-latency bound like K1: a persistent grid of spans
    // 32 KiB tiles, 8 vectors a lane; a small image ends before the link is
    // full, and there a workgroup's pass over its tile counts: 8 KiB tiles (U = 2)
    // take 11 us against 31 on 64 KB, 18.5 / 36.4 on 0.5 MB, 47.6 / 50.2 on 2.1
    // MB, and from 10 MB on no less (42 MB 772 / 758).
    constexpr uint32_t kUnset = UINT32_MAX;
    const uint32_t knob = env_uint("SLLM_K2_UNROLL", kUnset);
    const uint32_t unroll = knob == kUnset ? (a.table && a.y1 - a.y0 < (4u << 20) ? 2 : 8) : knob >= 8 ? 8 : 4;
    const uint64_t tile = (uint64_t)kThreads * 16 * unroll;
    a.tile0 = a.y0 / tile;
    a.n_tiles = ceil_div(a.y1, tile) - a.tile0;
    // a chunk table carries the whole image; runs and windows are parts of it
    const uint32_t want = std::max<uint32_t>(
        1, a.table ? env_uint("SLLM_K1_BLOCKS", 512) : env_uint("SLLM_K1_STREAM_BLOCKS", 64));
    const dim3 grid((uint32_t)std::min<uint64_t>(a.n_tiles, want)), block(kThreads);
    auto run = [&](auto kernel) { kernel<<<grid, block, 0, stream>>>(a); };
    const bool u8 = unroll == 8;
    if (a.run_n) run(u8 ? k_scatter<8, false, kRun> : k_scatter<4, false, kRun>);
    else if (a.table) run(u8 ? k_scatter<8, false, kTable> : unroll == 4 ? k_scatter<4, false, kTable> : k_scatter<2, false, kTable>);
    else run(u8 ? k_scatter<8, false, kWindow> : k_scatter<4, false, kWindow>);
    SLLM_HIP(hipGetLastError());
    return SLLM_OK;
}

}  // namespace

namespace {

// Compute the tables of the n tensors of sizes s (file layout at alignment
// `align`, device layout at `dev_align`) and the plan's first n_plan entries on
// `stream`.
int32_t launch_tables(const std::vector<uint64_t>& s, uint64_t align, uint64_t dev_align, uint64_t* size, uint64_t* off,
                      uint64_t* dev, int64_t* plan, uint64_t n_plan, hipStream_t stream) {
    TableArgs a{};
    a.size = size;
    a.off = off;
    a.dev = dev;
    a.plan = plan;
    a.p0 = 0;
    a.n_plan = n_plan;
    a.align_o = align;
    a.align_d = dev_align;
    for (a.i0 = 0; a.i0 < s.size(); a.i0 += a.m) {
        a.m = pack_sizes(s.data() + a.i0, s.size() - a.i0, &a);
        a.last = a.i0 + a.m == s.size();
        uint64_t o = a.o0, d = a.d0;
        for (uint32_t j = 0; j < a.m; ++j) {  // both totals were checked against 64 bits before
            o += (s[a.i0 + j] + align - 1) & ~(align - 1);
            d += (s[a.i0 + j] + dev_align - 1) & ~(dev_align - 1);
        }
        const uint64_t blocks = std::min(ceil_div(d, kPlanBytes), n_plan) - std::min(a.d0 / kPlanBytes, n_plan);
        a.spread = spread_plan(blocks, s.data() + a.i0, a.m);
        // spread: a workgroup for each 1024 blocks of the plan
        const uint32_t grid = a.spread ? (uint32_t)std::min<uint64_t>(512, ceil_div(blocks, 1024)) : 1;
        k3_tables<<<dim3(grid), dim3(1024), 0, stream>>>(a);
        SLLM_HIP(hipGetLastError());
        a.o0 = o;
        a.d0 = d;
    }
    return SLLM_OK;
}

constexpr int kMaxDevices = 64;

std::mutex g_blocks_mu;
std::vector<DeviceBlock> g_idle_blocks;  // oldest first

}  // namespace

int32_t block_take(int device, uint64_t bytes, DeviceBlock* out) {
    constexpr uint64_t kGrain = 64 << 10;
    *out = DeviceBlock{};
    out->device = device;
    if (bytes == 0) return SLLM_OK;
    if (bytes > UINT64_MAX - kGrain) return fail(SLLM_E_INVAL, "block size overflows");
    const uint64_t want = (bytes + kGrain - 1) / kGrain * kGrain;
    {
        // the smallest idle block that fits, unless it would waste most of itself
        std::lock_guard<std::mutex> g(g_blocks_mu);
        g_idle_blocks.reserve(kMaxIdleBlocks * kMaxDevices);  // giving a block back cannot fail
        size_t best = g_idle_blocks.size();
        for (size_t i = 0; i < g_idle_blocks.size(); ++i) {
            const DeviceBlock& b = g_idle_blocks[i];
            if (b.device != device || b.bytes < want || b.bytes / 4 > want) continue;
            if (best == g_idle_blocks.size() || b.bytes < g_idle_blocks[best].bytes) best = i;
        }
        if (best < g_idle_blocks.size()) {
            *out = g_idle_blocks[best];
            g_idle_blocks.erase(g_idle_blocks.begin() + (long)best);
            return SLLM_OK;
        }
    }
    void* p = nullptr;
    hipError_t e = hipMalloc(&p, want);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();  // leave no error behind for later launch checks
        std::vector<DeviceBlock> idle;
        {
            std::lock_guard<std::mutex> g(g_blocks_mu);
            for (size_t i = 0; i < g_idle_blocks.size();) {
                if (g_idle_blocks[i].device != device) {
                    ++i;
                    continue;
                }
                idle.push_back(g_idle_blocks[i]);
                g_idle_blocks.erase(g_idle_blocks.begin() + (long)i);
            }
        }
        for (const DeviceBlock& b : idle) (void)hipFree(b.p);
        (void)hipGetLastError();
        e = hipMalloc(&p, want);
    }
    if (e != hipSuccess) return fail(SLLM_E_HIP, "hipMalloc(%llu bytes) failed: %s", (unsigned long long)want, hip_message(e));
    out->p = static_cast<uint8_t*>(p);
    out->bytes = want;
    return SLLM_OK;
}

void block_give(DeviceBlock* b) {
    if (!b->p) return;
    DeviceBlock drop[kMaxIdleBlocks];
    size_t n_drop = 0;
    if (b->bytes > kMaxIdleBlockBytes) {
        drop[n_drop++] = *b;
    } else {
        // the device's oldest idle blocks make room, so that sizes no handle
        // takes any more do not fill the list for good
        std::lock_guard<std::mutex> g(g_blocks_mu);
        uint64_t held = b->bytes;
        size_t count = 1;
        for (const DeviceBlock& i : g_idle_blocks)
            if (i.device == b->device) {
                held += i.bytes;
                ++count;
            }
        for (size_t i = 0; count > kMaxIdleBlocks || held > kMaxIdleBlockBytes;) {
            if (g_idle_blocks[i].device != b->device) {
                ++i;
                continue;
            }
            held -= g_idle_blocks[i].bytes;
            --count;
            drop[n_drop++] = g_idle_blocks[i];
            g_idle_blocks.erase(g_idle_blocks.begin() + (long)i);
        }
        g_idle_blocks.push_back(*b);  // within the capacity block_take reserved
    }
    for (size_t i = 0; i < n_drop; ++i) (void)hipFree(drop[i].p);
    *b = DeviceBlock{};
}

int32_t device_layout_build(const IndexData& ix, int device, const uint64_t* dev_off, uint64_t dev_total,
                            uint64_t dev_align, uint64_t staging_chunks, uint64_t chunk, DeviceLayout* out) {
    DeviceLayout& l = *out;
    l.n = ix.tensors.size();
    l.total = ix.total;
    l.dev_total = dev_total;
    l.align = ix.alignment;
    l.dev_align = dev_align;
    l.tensors = ix.tensors.data();
    l.h_dev = dev_off;
    if (staging_chunks) {
        uint64_t bytes;
        if (!align_up(chunk, 256, &l.staging_stride) || !mul_ok(staging_chunks, l.staging_stride, &bytes))
            return fail(SLLM_E_INVAL, "chunk size overflows");
        SLLM_TRY(block_take(device, bytes, &l.stage));
        l.staging = l.stage.p;
    }
    if (l.n == 0) return SLLM_OK;
    // one block: o and d (n + 1 entries each), s, the plan
    l.n_shift = ceil_div(dev_total, kPlanBytes);
    SLLM_TRY(block_take(device, (3 * l.n + 2 + l.n_shift) * sizeof(uint64_t), &l.tables));
    l.d_off = reinterpret_cast<uint64_t*>(l.tables.p);
    l.d_dev = l.d_off + l.n + 1;
    l.d_size = l.d_dev + l.n + 1;
    l.d_shift = reinterpret_cast<int64_t*>(l.d_size + l.n);
    std::vector<uint64_t> got(3 * l.n + 2);
    const int32_t st = launch_tables(ix.sizes, ix.alignment, dev_align, l.d_size, l.d_off, l.d_dev, l.d_shift, l.n_shift, nullptr);
    // This form of the copy waits for the null stream too, but is not refused,
    // ending the capture, while another stream captures, as hipMemcpy is.  (Queued
    // and then waited for, it costs a load 5 us more.)  In any case the stream is
    // waited for: loads run on others, and after a failed launch the block may go
    // back.
    const hipError_t e =
        hipMemcpyWithStream(got.data(), l.tables.p, got.size() * sizeof(uint64_t), hipMemcpyDeviceToHost, nullptr);
    if (e != hipSuccess) (void)hipStreamSynchronize(nullptr);
    if (st != SLLM_OK) return st;
    SLLM_HIP(e);
    // the device's tables against the host's: a wrong entry would send bytes
    // past the image
    const uint64_t *off = got.data(), *dev = off + l.n + 1, *size = dev + l.n + 1;
    uint64_t o = 0;  // o_i, as the index was checked to hold them; its records lie further apart than the sizes
    for (uint64_t i = 0; i < l.n; ++i) {
        if (off[i] != o || dev[i] != dev_off[i] || size[i] != ix.sizes[i])
            return fail(SLLM_E_HIP, "device tables disagree at tensor %llu: offset %llu, device offset %llu, size %llu",
                        (unsigned long long)i, (unsigned long long)off[i], (unsigned long long)dev[i],
                        (unsigned long long)size[i]);
        o += (ix.sizes[i] + ix.alignment - 1) & ~(ix.alignment - 1);
    }
    if (off[l.n] != ix.total || dev[l.n] != dev_total) return fail(SLLM_E_HIP, "device tables disagree on the totals");
    return SLLM_OK;
}

void device_layout_free(DeviceLayout* l, bool park) {
    for (DeviceBlock* b : {&l->tables, &l->stage}) {
        if (park) block_give(b);
        else if (b->p) (void)hipFree(b->p);
    }
    *l = DeviceLayout{};
}

int32_t launch_scatter_window(const DeviceLayout& l, uint8_t* dst, const uint8_t* src, uint64_t x0, uint64_t x1,
                              bool src_is_host, hipStream_t stream, hipEvent_t end) {
    ScatterArgs a{};
    a.dst = dst;
    a.base = src;
    a.x0 = x0;
    a.x1 = x1;
    a.vec_ok = (reinterpret_cast<uintptr_t>(src) % 16 == 0) && (x0 % 16 == 0);
    a.y0 = y_of(l, x0);
    a.y1 = y_of(l, x1);
    return launch(l, a, src_is_host, stream, 0, end);
}

int32_t launch_scatter_run(const DeviceLayout& l, uint8_t* dst, const uint8_t* const* srcs, uint64_t k0, uint32_t m,
                           uint64_t chunk, hipStream_t stream) {
    if (m == 0) return SLLM_OK;
    if (m > kScatterBatch || chunk == 0) return fail(SLLM_E_INVAL, "scatter run: bad size");
    if (k0 >= ceil_div(l.total, chunk) || m > ceil_div(l.total, chunk) - k0)
        return fail(SLLM_E_INVAL, "scatter run: chunks past the end of the image");
    ScatterArgs a{};
    a.dst = dst;
    a.chunk = chunk;
    a.run_n = m;
    a.run_k0 = k0;
    bool aligned = chunk % 16 == 0;
    for (uint32_t j = 0; j < m; ++j) {
        a.run_src[j] = srcs[j];
        aligned = aligned && reinterpret_cast<uintptr_t>(srcs[j]) % 16 == 0;
    }
    a.vec_ok = aligned;
    a.x0 = k0 * chunk;
    a.x1 = std::min((k0 + m) * chunk, l.total);
    a.y0 = y_of(l, a.x0);
    a.y1 = y_of(l, a.x1);
    return launch(l, a, /*src_is_host=*/true, stream);
}

int32_t launch_scatter_table(const DeviceLayout& l, uint8_t* dst, const uint8_t* const* table, uint64_t chunk,
                             hipStream_t stream) {
    ScatterArgs a{};
    a.dst = dst;
    a.table = table;
    a.chunk = chunk;
    a.vec_ok = chunk % 16 == 0;
    a.y0 = 0;
    a.y1 = l.dev_total;
    return launch(l, a, /*src_is_host=*/true, stream);
}

}  // namespace sllm

// ---------------------------------------------------------------------------
// Allocation-free repack
// ---------------------------------------------------------------------------

// The device memory of the allocation-free repack: the size table, the two
// scanned offset tables and one window of K2's plan (layout in
// device_layout.hpp).  Every device holds its own copy from the library's
// first kernel launch on it until the process ends.  Host code reaches a
// device's copy only through the address hipGetSymbolAddress returns with
// that device current; the name itself is not a device address on the host.
static __device__ __align__(256) uint8_t scratch[sllm::kNoAllocScratchBytes];

namespace sllm {

namespace {

std::mutex g_scratch_mu;
uint8_t* g_scratch[kMaxDevices] = {};

// The scratch area's address on `device`, looked up once per device (the
// caller has made `device` current).
int32_t scratch_of(int device, uint8_t** out) {
    if (device < 0 || device >= kMaxDevices) return fail(SLLM_E_INVAL, "device %d is out of range", device);
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(SLLM_E_HIP, "hipGetSymbolAddress(scratch) on device %d failed: %s", device, hip_message(e));
        g_scratch[device] = static_cast<uint8_t*>(p);
    }
    *out = g_scratch[device];
    return SLLM_OK;
}

}  // namespace

int32_t repack_noalloc(const IndexData& ix, int device, uint64_t dev_align, uint64_t dev_total, const uint8_t* src,
                       uint8_t* dst, hipStream_t stream) {
    const uint64_t n = ix.tensors.size();
    if (n > kNoAllocMaxTensors)
        return fail(SLLM_E_RANGE, "%llu tensors exceed the %llu of the allocation-free repack", (unsigned long long)n,
                    (unsigned long long)kNoAllocMaxTensors);
    if (n == 0 || dev_total == 0) return SLLM_OK;
    uint8_t* base = nullptr;
    SLLM_TRY(scratch_of(device, &base));
    uint64_t* d_size = reinterpret_cast<uint64_t*>(base + kNoAllocSizeOffset);
    uint64_t* d_off = reinterpret_cast<uint64_t*>(base + kNoAllocFileOffset);
    uint64_t* d_dev = reinterpret_cast<uint64_t*>(base + kNoAllocDevOffset);
    int64_t* plan = reinterpret_cast<int64_t*>(base + kNoAllocPlanOffset);

    // windows of the device image, each planned into the plan area and then
    // moved by K2; one stream orders each window's plan after the previous
    // window's K2 (SLLM_NOALLOC_PLAN_BLOCKS lowers the window, to exercise
    // several on small images).  The first window's plan comes with the tables.
    DeviceLayout l;  // views of the scratch tables: owns nothing, never freed
    l.n = n;
    l.total = ix.total;
    l.dev_total = dev_total;
    l.align = ix.alignment;
    l.dev_align = dev_align;
    l.d_off = d_off;
    l.d_size = d_size;
    l.d_dev = d_dev;
    l.d_shift = plan;
    const uint64_t n_blocks = ceil_div(dev_total, kPlanBytes);
    const uint64_t window = std::max<uint64_t>(
        1, std::min<uint64_t>(kNoAllocPlanEntries, env_uint("SLLM_NOALLOC_PLAN_BLOCKS", (uint32_t)kNoAllocPlanEntries)));
    for (uint64_t p0 = 0; p0 < n_blocks; p0 += window) {
        const uint64_t nb = std::min(window, n_blocks - p0);
        if (p0 == 0) {
            SLLM_TRY(launch_tables(ix.sizes, ix.alignment, dev_align, d_size, d_off, d_dev, plan, nb, stream));
        } else {
            const uint64_t blocks = std::min<uint64_t>(ceil_div(nb, 256), 4096);
            k3_tile_shift<<<dim3((uint32_t)blocks), dim3(256), 0, stream>>>(d_dev, d_off, d_size, n, p0, nb, plan);
            SLLM_HIP(hipGetLastError());
        }
        ScatterArgs a{};
        a.dst = dst;
        a.base = src;
        a.x0 = 0;
        a.x1 = ix.total;
        a.vec_ok = reinterpret_cast<uintptr_t>(src) % 16 == 0;
        a.y0 = p0 * kPlanBytes;
        a.y1 = std::min((p0 + nb) * kPlanBytes, dev_total);
        SLLM_TRY(launch(l, a, /*src_is_host=*/false, stream, p0));
    }
    return SLLM_OK;
}

}  // namespace sllm
