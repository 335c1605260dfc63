// Threshold estimate (sample histogram, pick) and the one streaming pass over g and e.
#pragma once

#include "mv_common.hpp"

namespace mvk {

// ----------------------------------------------------------------------------
// One kernel: threshold estimate (sample histogram, pick) and the streaming pass
// ----------------------------------------------------------------------------
// The grid is one-dimensional.  Its first N * spr workgroups sample the rows (spr
// per row); the last of a row's sampling workgroups to finish turns the row's
// histogram into the threshold estimate tau and publishes it.  All other workgroups
// stream: a wavefront owns a segment of 1024 coordinates, loads g and e, stores
// a = g + e, and only then needs tau to pick its candidates -- by which time the
// few sampling workgroups, which were started first, have long finished, except for
// the very first streaming workgroups, which wait a few microseconds.  The estimate
// therefore costs no launch of its own and overlaps the head of the streaming pass.
//
// The streaming pass overwrites e, which the sampling reads: a streaming wavefront
// holds back its stores until all of its row's sampling workgroups have their samples
// in registers (reads_done[row], a counter that only ever grows: spr per step).  That
// happens a few microseconds into the kernel, before the first streaming loads are
// back.  (Were a store to slip in early, the estimate would see a = g + e in place of e
// at that spot: a worse estimate, the same result.)
//
// The wait is bounded: a wavefront that has polled spin_limit times without seeing
// its row's tau marks the row (row_poison[row] = this step's number) and goes on
// without candidates; mv_row_select then reads the row's count as overflowed and
// selects the row exactly from memory, like any row whose estimate failed.  The
// result never depends on the estimate, only the time does.
//
// What crosses between workgroups inside the kernel travels through atomics only
// (the histogram, the counters, the published tau), which are performed in memory;
// ordinary stores of one workgroup are not visible to another before the kernel ends.
//
// Sampling: chunk c of a row is the coordinates [32c, 32c+32); chunk c is sampled
// when c % stride == 0.  bin = (bits(|g+e|)) >> kHistShift.  tau = lower edge of the
// highest bin such that at least m_target sampled coordinates lie in that bin or
// above (0 if fewer).  The picking workgroup also clears the row's histogram and
// resets the per-step counters.
//
// Streaming: one wavefront = one segment of 1024 consecutive coordinates of one row,
// read as 4 sub-blocks of 256 (lane l holds coordinates base + 256u + 4l .. +3).  Eight
// consecutive workgroups of 8 wavefronts share 64 consecutive segments, each taking every
// eighth: the dies, over which consecutive workgroups are spread, then work on neighbouring
// 4 KB of the same 32 KB, and whole, aligned ones (RowSegments).  Bare e = g + e on one box, with 8
// consecutive segments to a workgroup / so / so and aligned:
//   32 x 25.6 M fp32 1858 / 1630 / 1486 us, bf16 1565 / 1415 / 1268;
//   16 x 11.2 M fp32  399 /  356 /  335 us, bf16  337 /  313 /  290 (6.4 and 6.2 TB/s);
//   up to 4 x 2^20 no difference.
// Neighbouring pieces of 2 KB or 1 KB are slower where rows are not aligned to them and no faster
// where they are; segments that begin at 128-byte lines lose 1 to 3 % against 4 KB.
// Coordinates with
// (bits(a) & 0x7FFFFFFF) >= tau are appended to the row's candidate list as
// (magnitude bits, coordinate), in ascending coordinate order inside the segment's
// run; runs[row][run_place(s, number of segments)] = (start of segment s's run, its length).  Runs land in the list in any
// order; the table makes the order recoverable.  The workgroup reserves list space
// for its 8 runs with ONE atomic on the row's counter (returning atomics on one
// cache line complete only every few nanoseconds chip-wide, so one per wavefront
// would bound the whole pass when candidates are spread evenly).  Entries beyond
// `cap` are dropped, the counter keeps counting (the overflow is detected from it).
//
// A bin is 3 % of a magnitude wide.  Error buffers that a steady gradient has driven for long hold many magnitudes
// just below the K-th, and the edge of the bin lets them all into the list: one that overflows has its row
// selected from memory by one workgroup (1 x 16 M, after some thousand steps: 1.7 ms for 0.1).  So the samples are kept,
// and where more than `crowded` of them lie in the bin or above it, the picking workgroup goes through them once more and
// places tau inside the bin, at one of kSubBins edges.  One sampling workgroup keeps its samples in registers; several
// keep them in memory, past the caches, and only with few workers (see make_plan, which also has the line).
constexpr int      kSubBins = kStreamThreads;
constexpr int      kSubShift = kHistShift - 9;
static_assert(kSubBins == 512, "9 bits behind the bin's");
constexpr int      kSampleQuads = 4;              // quads of samples a sampling thread has in flight
constexpr uint32_t kSampleWgs = 16;               // at most so many workgroups sample a row
constexpr int      kAgainQuads = 8;               // ... that goes through them once more (1.6 M: four 761 us, eight 738)
constexpr uint32_t kRowPoison = 0x80000000u;      // set in a marked row's candidate counter by mv_row_select

struct StreamLds {
    __attribute__((aligned(16))) uint32_t h[kHistBins];   // sampling workgroups only
    uint64_t scan[kStreamThreads / kWave + 1];
    uint32_t found, is_last;
    uint32_t crowd[3];                                    // a crowded bin: its number, the samples above it, those in it
    uint32_t wave_total[kSegPerBlock];
    uint32_t block_base;
};

// 16 bytes past the caches, at byte offset `byte` of a buffer of `bytes` bytes (both uniform but for the offset)
constexpr int kRawBuffer = 0x00027000, kPastCaches = 17;       // plain 32-bit data; system scope
__device__ __forceinline__ void store_through(u32x4 v, void* buffer, uint32_t bytes, uint32_t byte)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, __builtin_amdgcn_make_buffer_rsrc(buffer, 0, bytes, kRawBuffer), byte, 0, kPastCaches);
}
__device__ __forceinline__ u32x4 load_through(void* buffer, uint32_t bytes, uint32_t byte)
{
    return __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(buffer, 0, bytes, kRawBuffer), byte, 0,
                                                 kPastCaches);
}

// The lower edge of the sub-bin of the crowded bin at which `want` of its samples are covered from above.  The samples are
// in memory or (null) the threads' kept ones.  The whole workgroup.
__device__ __forceinline__ uint32_t edge_inside_bin(StreamLds& lds, uint32_t* samples, uint32_t nquads,
                                                    const u32x4 (&kept)[kSampleQuads], uint32_t bin, uint32_t want)
{
    const uint32_t t = threadIdx.x;
    lds.h[t] = 0;
    __syncthreads();
    auto tally = [&](u32x4 k) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (k[c] >> kHistShift == bin) atomicAdd(&lds.h[k[c] >> kSubShift & (uint32_t)(kSubBins - 1)], 1u);
    };
    if (!samples) {
#pragma unroll
        for (int u = 0; u < kSampleQuads; ++u) tally(kept[u]);
    } else {
        for (uint32_t q0 = t; q0 < nquads; q0 += kAgainQuads * kStreamThreads) {
            u32x4 k[kAgainQuads];
#pragma unroll
            for (int u = 0; u < kAgainQuads; ++u) {
                const uint32_t q = q0 + (uint32_t)u * kStreamThreads;
                const u32x4 z = {0u, 0u, 0u, 0u};
                k[u] = q < nquads ? load_through(samples, nquads * 16u, q * 16u) : z;
            }
#pragma unroll
            for (int u = 0; u < kAgainQuads; ++u) tally(k[u]);
        }
    }
    __syncthreads();
    const uint32_t sub = (uint32_t)(kSubBins - 1) - t, n = lds.h[sub];           // from above
    uint32_t total;
    const uint32_t excl = block_excl_scan<kStreamThreads>(n, lds.scan, total);
    if (excl < want && want <= excl + n) lds.found = bin << kHistShift | sub << kSubShift;
    __syncthreads();
    return lds.found;
}

template <typename GT>
__device__ __forceinline__ void sample_and_pick(StreamLds& lds, const GT* __restrict__ g, int64_t ld_g,
                                                const float* __restrict__ e, int64_t ld_e, int64_t d,
                                                uint32_t row, uint32_t part, uint32_t spr, uint32_t stride,
                                                uint32_t n_sampled_chunks, uint32_t m_target, uint32_t crowded,
                                                uint32_t* __restrict__ hist, uint32_t* __restrict__ sample_done,
                                                uint32_t* __restrict__ reads_done,
                                                unsigned long long* __restrict__ tau_pub, uint32_t epoch,
                                                uint32_t* __restrict__ next_row_count, uint32_t* __restrict__ lvl_sets,
                                                uint32_t n_lvl_words, uint32_t n_rows,
                                                uint32_t* __restrict__ ad_count, uint32_t* __restrict__ all_samples)
{
    const uint32_t t = threadIdx.x;
    {
        const u32x4 z = {0u, 0u, 0u, 0u};
        u32x4* hz = reinterpret_cast<u32x4*>(lds.h);
        for (int b = t; b < kHistBins / 4; b += kStreamThreads) hz[b] = z;
    }
    __syncthreads();
    const GT*    grow = g + (int64_t)row * ld_g;
    const float* erow = e + (int64_t)row * ld_e;
    const uint32_t nquads = n_sampled_chunks * (kChunk / 4);       // at most 32,768, or about one coordinate in 512
    uint32_t* samples = all_samples ? all_samples + (size_t)row * nquads * 4 : nullptr;
    const uint32_t step = spr * kStreamThreads;
    auto start_of = [stride](uint32_t q) {
        return (int64_t)(q / (kChunk / 4)) * stride * kChunk + (int64_t)(q % (kChunk / 4)) * 4;
    };
    // The samples lie far apart in memory and every load pays the full latency: kSampleQuads
    // quads' loads are in flight per thread and the grid is sized for one round, or a few.  A round loads in every
    // lane (past the samples: the row's first quad) and assigns all of `kept`, which is therefore not alive in the
    // next round's loads.  The streaming workgroups have to do with the registers that this takes: 60, eight
    // waves to a SIMD.  Where a thread only assigned what it had loaded, 78 and six (7 x 1,000,003 bf16, K = 2000:
    // 49.5 -> 49.0 us, 1 x 80,003: 25.2 -> 24.8, 2 x 4,000,003: 70.9 -> 70.2).
    u32x4 kept[kSampleQuads];                     // the last round's: one sampling workgroup has no other
    uint32_t q0 = part * kStreamThreads + t;
    do {
        f32x4 gv[kSampleQuads], ev[kSampleQuads];
#pragma unroll
        for (int u = 0; u < kSampleQuads; ++u) {
            const uint32_t q = q0 + (uint32_t)u * step;
            const int64_t j = start_of(q), at = q < nquads && j + 4 <= d ? j : 0;
            gv[u] = load4_grad(grow + at);
            ev[u] = *reinterpret_cast<const f32x4*>(erow + at);
        }
#pragma unroll
        for (int u = 0; u < kSampleQuads; ++u) {
            const uint32_t q = q0 + (uint32_t)u * step;
            const int64_t j = start_of(q);
            u32x4 key = __builtin_bit_cast(u32x4, gv[u] + ev[u]) & kAbsMask;
            int n = q < nquads ? 4 : 0;
            if (q < nquads && j + 4 > d) {        // the row's last quad
                n = j < d ? (int)(d - j) : 0;
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (c < n) key[c] = __float_as_uint(load1_grad(grow + j + c) + erow[j + c]) & kAbsMask;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                key[c] = c < n ? key[c] : 0u;
                if (c < n) atomicAdd(&lds.h[key[c] >> kHistShift], 1u);
            }
            kept[u] = key;
            if (samples && q < nquads) store_through(key, samples, nquads * 16u, q * 16u);   // (samples: uniform)
        }
        q0 += kSampleQuads * step;
    } while (q0 < nquads);
    __syncthreads();
    // every sample of this workgroup has been used, so it has arrived: the row's streaming
    // wavefronts may overwrite e as far as this workgroup is concerned
    if (t == 0) atomicAdd(&reads_done[row * kCounterStride], 1u);
    uint32_t* hrow = hist + (size_t)row * kHistBins;
    constexpr int per = kHistBins / kStreamThreads;   // bins per thread, descending bin order
    uint32_t c[per];
    if (spr == 1u) {
        // Short rows: the row's only sampling workgroup has the whole histogram in LDS.
        const u32x4* hv = reinterpret_cast<const u32x4*>(lds.h);
#pragma unroll
        for (int q = 0; q < per; q += 4) {
            const u32x4 w = hv[(kHistBins - (int)t * per - q) / 4 - 1];
            c[q] = w.w;  c[q + 1] = w.z;  c[q + 2] = w.y;  c[q + 3] = w.x;
        }
    } else {
        for (int b = t; b < kHistBins; b += kStreamThreads) {
            const uint32_t n = lds.h[b];
            if (n) atomicAdd(&hrow[b], n);
        }
        // every atomic of this workgroup has been performed before it is counted as done
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (t == 0) lds.is_last = atomicAdd(&sample_done[row * kCounterStride], 1u) == spr - 1u;
        __syncthreads();
        if (!lds.is_last) return;                 // whole workgroup
        // the row's last sampling workgroup reads the sum from memory, where the others' atomics went
#pragma unroll
        for (int q = 0; q < per; ++q)
            c[q] = __hip_atomic_load(&hrow[kHistBins - 1 - ((int)t * per + q)], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
    }

    // ---- histogram -> tau
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < per; ++q) sum += c[q];
    if (t == 0) lds.found = 0;
    uint32_t total;
    const uint32_t excl = block_excl_scan<kStreamThreads>(sum, lds.scan, total);
    if (excl < m_target && m_target <= excl + sum) {
        uint32_t acc = excl;
#pragma unroll
        for (int q = 0; q < per; ++q) {
            if (acc < m_target && m_target <= acc + c[q]) {
                const uint32_t bin = (uint32_t)(kHistBins - 1 - ((int)t * per + q));
                lds.found = bin << kHistShift;
                lds.crowd[0] = bin;
                lds.crowd[1] = acc;
                lds.crowd[2] = c[q];
            }
            acc += c[q];
        }
    }
    __syncthreads();
    uint32_t tau = (total >= m_target) ? lds.found : 0u;
    const uint32_t bin = lds.crowd[0], above = lds.crowd[1], in_bin = lds.crowd[2];
    if (tau != 0u && above + in_bin > crowded) {                       // uniform
        __syncthreads();
        tau = edge_inside_bin(lds, samples, nquads, kept, bin, m_target - above);
    }
    if (t == 0) {
        __hip_atomic_store(&tau_pub[row * (kCounterStride / 2)], ((unsigned long long)epoch << 32) | tau,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // Behind the publication, what the NEXT step's kernel must find at zero (ordinary stores: they
    // are in memory when this kernel has ended): the histogram, the sampling counter, the row's
    // candidate counter of the other parity (this step's streaming workgroups bump row_count; the
    // next step's bump next_row_count), the add / drop list lengths, the vote-level counters.
    if (spr != 1u) {
#pragma unroll
        for (int q = 0; q < per; ++q) hrow[kHistBins - 1 - ((int)t * per + q)] = 0;
    }
    if (t == 0) {
        sample_done[row * kCounterStride] = 0;
        next_row_count[row * kCounterStride] = 0;
    }
    if (ad_count && t < 2) ad_count[ad_counter(row, t)] = 0;
    for (uint32_t i = row * kStreamThreads + t; i < n_lvl_words; i += n_rows * kStreamThreads) lvl_sets[i] = 0;
}

template <typename GT>
__global__ __launch_bounds__(kStreamThreads) void mv_stream_collect(
    const GT* __restrict__ g, int64_t ld_g, float* __restrict__ e, int64_t ld_e, int64_t d, uint32_t n_rows,
    uint32_t spr, uint32_t stride, uint32_t n_sampled_chunks, uint32_t m_target, uint32_t crowded,
    uint32_t* __restrict__ hist, uint32_t* __restrict__ sample_done, uint32_t* __restrict__ reads_done,
    unsigned long long* __restrict__ tau_pub, const uint32_t* __restrict__ step_no, uint32_t spin_limit, uint32_t* __restrict__ row_poison, uint32_t* __restrict__ lvl_sets,
    uint32_t n_lvl_words, uint32_t* __restrict__ ad_count, uint32_t* __restrict__ samples,
    u32x2* __restrict__ cand, uint32_t cap, uint32_t* __restrict__ row_count_sets, uint32_t row_count_set_words,
    u32x2* __restrict__ runs,
    uint32_t* __restrict__ run_taken, uint32_t n_runs, RowSegments segs, uint32_t head_wgs, int through,
    uint32_t* __restrict__ zero_votes32, int64_t votes_bytes)
{
    __shared__ StreamLds lds;
    // The step's number lives on the device (the step's last kernel counts it up), so that a
    // captured step can be replayed; the rows' candidate counters exist twice, and this step
    // counts into the set of its parity while it clears the other one for the next step.
    const uint32_t epoch = step_no[0] + 1u;
    uint32_t* row_count = row_count_sets + (epoch & 1u) * row_count_set_words;
    uint32_t* next_row_count = row_count_sets + ((epoch & 1u) ^ 1u) * row_count_set_words;
    if (blockIdx.x < n_rows * spr) {
        sample_and_pick<GT>(lds, g, ld_g, e, ld_e, d, blockIdx.x / spr, blockIdx.x % spr, spr, stride, n_sampled_chunks,
                            m_target, crowded, hist, sample_done, reads_done, tau_pub, epoch, next_row_count, lvl_sets, n_lvl_words,
                            n_rows, ad_count, samples);
        return;
    }
    const uint32_t sb = blockIdx.x - n_rows * spr;
    const uint32_t wgs_per_row = n_runs / kSegPerBlock;
    const uint32_t row = sb / wgs_per_row, bx = sb % wgs_per_row;
    const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t nseg = segs.count(row), place = bx * kSegPerBlock + wave, s = run_place(place, nseg);
    if (bx * kSegPerBlock >= nseg) return;       // whole workgroup (a shorter shift than the longest)
    const bool live = s < nseg;                  // whole wavefront; dead ones only keep the barriers company
    const int64_t base = (int64_t)s * kSeg - segs.shift(row);
    const GT* grow = g + (int64_t)row * ld_g;
    float*    erow = e + (int64_t)row * ld_e;
    const unsigned long long* tau_at = tau_pub + row * (kCounterStride / 2);
    // a first look at the row's tau together with the data loads: after the kernel's first
    // microseconds it is there, and the wavefront never waits
    unsigned long long tw = __hip_atomic_load(tau_at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t* rd_at = reads_done + row * kCounterStride;
    const uint32_t rd_target = spr * epoch;       // the counter grows by spr per step and wraps with this product
    uint32_t rd = __hip_atomic_load(rd_at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t spins = 0;
    // (all lanes of a wavefront load the same words, so the waits below are wave-uniform)
    auto samples_are_in = [&]() {
        while ((int32_t)(rd - rd_target) < 0 && spins < spin_limit) {
            __builtin_amdgcn_s_sleep(8);
            rd = __hip_atomic_load(rd_at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ++spins;
        }
    };

    // The kernel's first streaming workgroups would compete with the sampling for the memory
    // system and delay the estimate for everybody: they hold back even their loads (none where one
    // workgroup samples a row, see make_plan).
    if (sb < head_wgs) samples_are_in();

    uint32_t key[16];
    uint32_t inside = 0;                          // bit i: key[i] is a coordinate of the row
    if (live && base >= 0 && base + kSeg <= d) {
        f32x4 gv[4], ev[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = base + u * 256 + lane * 4;
            gv[u] = load4_grad(grow + j);
            ev[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(erow + j));
        }
        // (the counter's load was issued before the data loads, so looking at it waits for none of them;
        // each sub-block is stored as soon as its own loads are back: stores in one burst run slower)
        samples_are_in();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = base + u * 256 + lane * 4;
            const f32x4 a = gv[u] + ev[u];
            // (uniform: stored past the caches, nothing is left to be written back when the kernel ends; see make_plan)
            if (through) store_through(__builtin_bit_cast(u32x4, a), erow + base, kSeg * 4, (uint32_t)(j - base) * 4u);
            else         __builtin_nontemporal_store(a, reinterpret_cast<f32x4*>(erow + j));
            key[u * 4 + 0] = __float_as_uint(a.x) & kAbsMask;
            key[u * 4 + 1] = __float_as_uint(a.y) & kAbsMask;
            key[u * 4 + 2] = __float_as_uint(a.z) & kAbsMask;
            key[u * 4 + 3] = __float_as_uint(a.w) & kAbsMask;
        }
        inside = 0xFFFFu;
    } else if (live) {
        // first or last segment of the row: nothing outside it is read or written.  (base is a multiple of 4, so only
        // the row's last quad can be cut)
        f32x4 gv[4], ev[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = base + u * 256 + lane * 4;
            if (j >= 0 && j + 4 <= d) {
                gv[u] = load4_grad(grow + j);
                ev[u] = *reinterpret_cast<const f32x4*>(erow + j);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool there = j >= 0 && j + c < d;
                    gv[u][c] = there ? load1_grad(grow + j + c) : 0.0f;
                    ev[u][c] = there ? erow[j + c] : 0.0f;
                }
            }
        }
        samples_are_in();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = base + u * 256 + lane * 4;
            const f32x4 a = gv[u] + ev[u];
            if (j >= 0 && j + 4 <= d) *reinterpret_cast<f32x4*>(erow + j) = a;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const bool there = j >= 0 && j + c < d;
                if (there && j + 4 > d) erow[j + c] = a[c];
                key[u * 4 + c] = __float_as_uint(a[c]) & kAbsMask;
                inside |= (there ? 1u : 0u) << (u * 4 + c);
            }
        }
    }

    // tau: wait for it if need be (bounded), then the candidates' flags
    while (live && (uint32_t)(tw >> 32) != epoch && spins < spin_limit) {
        __builtin_amdgcn_s_sleep(16);
        tw = __hip_atomic_load(tau_at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ++spins;
    }
    uint32_t tau = (uint32_t)tw;
    if (live && (uint32_t)(tw >> 32) != epoch) {                       // not seen in time: the row goes the exact way
        tau = 0xFFFFFFFFu;                                             // above every key
        if (lane == 0) atomicMax(&row_poison[row], epoch);             // step numbers only grow: never reset
    }
    uint32_t flags = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) flags |= (key[i] >= tau ? 1u : 0u) << i;
    flags &= inside;

    // rank of each kept coordinate inside the wavefront's run
    uint32_t total = 0;
    uint32_t rank[4] = {0, 0, 0, 0};
    const bool any = __ballot(flags != 0) != 0ull;       // wave-uniform
    if (any) {
#pragma unroll
        for (int u = 0; u < 4; u += 2) {          // two sub-blocks' counts (at most 256 each) to a word
            const uint32_t c0 = __popc((flags >> (4 * u)) & 15u), c1 = __popc((flags >> (4 * u + 4)) & 15u);
            const uint32_t incl = wave_incl_scan(c0 | c1 << 16);
            const uint32_t sums = from_lane(incl, kWave - 1);
            rank[u] = total + (incl & 0xFFFFu) - c0;
            total += sums & 0xFFFFu;
            rank[u + 1] = total + (incl >> 16) - c1;
            total += sums >> 16;
        }
    }
    // one reservation for the workgroup's run
    if (lane == 0) lds.wave_total[wave] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t sum = 0;
#pragma unroll
        for (int w = 0; w < kSegPerBlock; ++w) {
            const uint32_t t = lds.wave_total[w];
            lds.wave_total[w] = sum;
            sum += t;
        }
        lds.block_base = sum ? atomicAdd(&row_count[row * kCounterStride], sum) : 0u;
    }
    __syncthreads();
    const uint32_t run_start = lds.block_base + lds.wave_total[wave];
    if (any) {
        u32x2* crow = cand + (size_t)row * cap;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (flags & (1u << (u * 4 + c))) {
                    const uint64_t pos = (uint64_t)run_start + rank[u]++;
                    if (pos < cap) {
                        u32x2 rec;
                        rec.x = key[u * 4 + c];
                        rec.y = (uint32_t)(base + u * 256 + lane * 4 + c);
                        crow[pos] = rec;
                    }
                }
    }
    // Row 0's wavefronts also clear the packed vote bytes (one per coordinate, 16 per lane), which the kernels
    // that follow fill and read.
    if (zero_votes32 && row == 0 && live) {
        const int64_t j = (int64_t)s * kSeg + (int64_t)lane * 16;
        const u32x4 z = {0u, 0u, 0u, 0u};
        if (j < votes_bytes) *reinterpret_cast<u32x4*>(zero_votes32 + (j >> 2)) = z;
    }
    // the runs' table, and the tallies that are counted when the votes are cast
    if (lane == 0) runs[(size_t)row * n_runs + place] = u32x2{run_start, total};
    constexpr uint32_t kWords = kSegPerBlock / 2;
    if (threadIdx.x < kWords) run_taken[((size_t)row * wgs_per_row + bx) * kWords + threadIdx.x] = 0;
}

}  // namespace mvk
