// Types, constants and workgroup-wide helpers (scans) shared by the vote step's kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mvk {


typedef float    f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));

constexpr int      kWave           = 64;
constexpr int      kSeg            = 1024;   // coordinates per wavefront segment in the streaming pass: 4 KB of e
constexpr int      kStreamThreads  = 512;    // 8 segments per workgroup
constexpr int      kSegPerBlock    = kStreamThreads / kWave;
constexpr int      kXcds           = 8;      // consecutive workgroups run on as many dies, each with an L2 of its own
constexpr int      kGroupSegs      = kXcds * kSegPerBlock;   // segments that kXcds consecutive streaming workgroups share
constexpr int      kHistBits       = 13;     // sample histogram: exponent + 5 mantissa bits
constexpr int      kHistBins       = 1 << kHistBits;
constexpr int      kHistShift      = 31 - kHistBits;
constexpr int      kChunk          = 32;     // sampled chunk: 32 coordinates (one 128-byte line of fp32)
constexpr int      kRowThreads     = 1024;   // mv_row_select and the selects from lists
constexpr int      kVoteBlock      = 16384;  // coordinates per workgroup of mv_rs_keys and of msum's level counts
constexpr int      kVoteThreads    = 1024;   // mv_ad_emit and mv_rs_keys
constexpr uint32_t kAbsMask        = 0x7FFFFFFFu;
constexpr int      kFineBins       = 2048;   // mv_row_select: histogram of the candidates' magnitudes above tau
constexpr int      kFineShift      = 12;     // 2048 bins of 4096 bit patterns = one octave above tau

// ----------------------------------------------------------------------------
// small helpers
// ----------------------------------------------------------------------------

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & (kWave - 1); }

// Scans over the lanes of a wavefront by DPP moves (row shifts inside 16 lanes, then the two row
// broadcasts): adds that read a neighbour's register, where a shuffle goes through the LDS crossbar.
// The step's small kernels are chains of such scans: with shuffles, and a second barrier in the
// workgroup's scan, a step of 4 x 10,007 coordinates took 38.8 us and one of 4 x 2^20 62.2 us; so
// they take 35.2 and 58.5.  All lanes of the wavefront must be active.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
// inclusive sums inside every row of 16 lanes
__device__ __forceinline__ uint32_t row_incl_scan(uint32_t v)
{
    v += dpp_or_zero<0x111, 0xf>(v);              // row_shr:1, :2, :4, :8
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    return v;
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v = row_incl_scan(v);
    v += dpp_or_zero<0x142, 0xa>(v);              // row_bcast:15 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xc>(v);              // row_bcast:31 into rows 2 and 3
    return v;
}
// lane `l`'s value in every lane (l uniform)
__device__ __forceinline__ uint32_t from_lane(uint32_t v, uint32_t l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}

__device__ __forceinline__ uint64_t pack2(uint32_t hi, uint32_t lo) { return ((uint64_t)hi << 32) | lo; }

// a pair of 32-bit counts whose sums stay below 2^32: no carry between the halves
__device__ __forceinline__ uint64_t wave_incl_scan64(uint64_t v)
{
    return pack2(wave_incl_scan((uint32_t)(v >> 32)), wave_incl_scan((uint32_t)v));
}

// Exclusive scan of one value per thread over the whole workgroup (thread order),
// one barrier.  `lds` holds at least NT/64 entries.  Returns the exclusive prefix;
// `total` receives the workgroup sum.  The LDS scratch is free to reuse only after
// the caller's next __syncthreads().
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint64_t* lds, uint32_t& total)
{
    constexpr int NW = NT / kWave;
    static_assert(NW <= 16, "the wavefronts' sums are scanned in one row of lanes");
    const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t incl = wave_incl_scan(v);
    if (lane == kWave - 1) lds[wave] = incl;
    __syncthreads();
    const uint32_t w = row_incl_scan(lane < (uint32_t)NW ? (uint32_t)lds[lane] : 0u);
    total = from_lane(w, NW - 1);
    return (wave ? from_lane(w, wave - 1) : 0u) + incl - v;
}
// the same for a pair of 32-bit counts (pack2) whose sums stay below 2^32
template <int NT>
__device__ __forceinline__ uint64_t block_excl_scan64(uint64_t v, uint64_t* lds, uint64_t& total)
{
    constexpr int NW = NT / kWave;
    static_assert(NW <= 16, "the wavefronts' sums are scanned in one row of lanes");
    const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint64_t incl = wave_incl_scan64(v);
    if (lane == kWave - 1) lds[wave] = incl;
    __syncthreads();
    const uint64_t mine = lane < (uint32_t)NW ? lds[lane] : 0u;
    const uint32_t hi = row_incl_scan((uint32_t)(mine >> 32)), lo = row_incl_scan((uint32_t)mine);
    total = pack2(from_lane(hi, NW - 1), from_lane(lo, NW - 1));
    const uint64_t before = wave ? pack2(from_lane(hi, wave - 1), from_lane(lo, wave - 1)) : 0u;
    return before + incl - v;
}

// A row's segments begin at multiples of 4 KB of e's ADDRESS, so its first one may lack up to kMostShift coordinates:
// segment s of a row holds the coordinates [kSeg s - shift, kSeg (s + 1) - shift) that there are.
struct RowSegments {
    uint32_t first, step;                         // of e and of its row stride, in floats modulo kSeg
    uint32_t d;
    __device__ __forceinline__ uint32_t shift(uint32_t row) const { return (first + row * step) & (uint32_t)(kSeg - 1); }
    __device__ __forceinline__ uint32_t count(uint32_t row) const { return (d + shift(row) + kSeg - 1) / kSeg; }
};
constexpr int kMostShift = kSeg - 4;              // rows begin at multiples of 16 bytes
__device__ __forceinline__ uint32_t segment_of(uint32_t j, uint32_t shift) { return (j + shift) / kSeg; }
// A group's segments go round its workgroups, and what a workgroup notes of its segments' runs lies together: the place
// of segment s in the row's table of runs, and just so the segment whose run has place s.  A row of n segments
// may end with less than a group, whose workgroups take consecutive segments.
static_assert(kXcds == 8 && kSegPerBlock == 8, "the two halves of a segment's number in its group change places");
__device__ __forceinline__ uint32_t run_place(uint32_t s, uint32_t n)
{
    return s < (n & ~63u) ? (s & ~63u) | (s & 7u) << 3 | (s >> 3 & 7u) : s;
}

// The taken candidates per segment of a row, two counts to a word, counted where the sorted vote lists are wanted
// (else null).
struct SegmentTallies {
    uint32_t* taken;
    uint32_t  shift;
    __device__ __forceinline__ void add(uint32_t s, uint32_t n) const { atomicAdd(&taken[s >> 1], n << (s & 1u) * 16u); }
};
constexpr int kTallyUnit = 8;                     // segments whose tallies are read at once: 16 bytes
__device__ __forceinline__ uint32_t unit_sum(u32x4 w)
{
    const uint32_t s = w.x + w.y + w.z + w.w;     // two sums of four counts of at most kSeg
    return (s & 0xFFFFu) + (s >> 16);
}
// the first n counts of a unit, n < kTallyUnit
__device__ __forceinline__ uint32_t unit_sum_below(u32x4 w, uint32_t n)
{
    uint32_t s = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) s += n > 2 * k + 1 ? w[k] : n > 2 * k ? w[k] & 0xFFFFu : 0u;
    return (s & 0xFFFFu) + (s >> 16);
}

// bin of a candidate's magnitude key (>= tau) in the row's fine histogram; order preserving
__device__ __forceinline__ uint32_t fine_bin(uint32_t key, uint32_t tau)
{
    return min((key - tau) >> kFineShift, (uint32_t)(kFineBins - 1));
}

// widen four gradient elements to fp32
__device__ __forceinline__ f32x4 load4_grad(const float* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
}
__device__ __forceinline__ f32x4 load4_grad(const uint16_t* p)
{
    u16x4 h = __builtin_nontemporal_load(reinterpret_cast<const u16x4*>(p));
    f32x4 r;
    r.x = __uint_as_float((uint32_t)h.x << 16);
    r.y = __uint_as_float((uint32_t)h.y << 16);
    r.z = __uint_as_float((uint32_t)h.z << 16);
    r.w = __uint_as_float((uint32_t)h.w << 16);
    return r;
}
__device__ __forceinline__ float load1_grad(const float* p) { return *p; }
__device__ __forceinline__ float load1_grad(const uint16_t* p) { return __uint_as_float((uint32_t)(*p) << 16); }

// List length counters (the rows' candidate lists, the add-drop lists): many workgroups
// bump them with returning atomics, which complete one after the other per cache line,
// so every counter has a 128-byte line of its own.
constexpr uint32_t kCounterStride = 32;
__device__ __forceinline__ uint32_t ad_counter(uint32_t row, uint32_t which)
{
    return (2u * row + which) * kCounterStride;
}

}  // namespace mvk
