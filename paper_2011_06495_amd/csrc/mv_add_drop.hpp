// Majority voting with add-drop (Algorithm 2): candidate lists, K_ad-selects, update of the
// standing votes and of their sum, ordered compaction of the scratch bitmaps.
#pragma once

#include "mv_common.hpp"
#include "mv_select.hpp"
#include "mv_mask.hpp"

namespace mvk {

// ----------------------------------------------------------------------------
// 7. majority voting with add-drop (Algorithm 2)
// ----------------------------------------------------------------------------
// State, owned by the caller: vote_bits (row n = the bitmap of M~_n, the worker's
// standing vote) and msum (one byte per coordinate, M^sum = the sum of the
// standing votes).  After mv_row_select, membership of coordinate j in a row's
// plain top-K is a local test on (|a[n][j]|, j) against (kth, tie_cut), so
//   A = top-K and not in the standing vote   -> candidates for addition
//   D = in the standing vote and not top-K   -> candidates for removal
// are gathered into two lists per row; the K_ad largest of A and the K_ad
// smallest of D are selected exactly (ties to the lowest coordinate), applied to
// scratch bitmaps and to msum, and the scratch bitmaps are compacted in
// coordinate order into the sorted add / drop lists while the standing vote is
// updated.

// Threads of mv_ad_collect's workgroups: with 1024 a unit holds two, whose barriers leave it idle where rows and votes
// are many (128 x 400,003, K = 33,333, K_ad = 3333: 472 us, with 512 threads 375); a row whose bitmap is one workgroup's
// anyway is done sooner by more threads (255 x 33,001, K = 2750: 99 us, with 512 threads 105; 2 x 33,001: 47.6 and 49.5).
constexpr int kCollectThreads = 512, kCollectThreadsShort = 1024;

// One workgroup-wide reservation: every thread brings `n_mine` entries; returns the
// position of the thread's first entry in the row's list (the list counter is bumped
// once per workgroup).  All threads of the workgroup must call it.
template <int THREADS>
__device__ __forceinline__ uint32_t reserve_in_list(uint32_t n_mine, uint32_t* __restrict__ counter,
                                                    uint64_t* scan_lds, uint32_t* bcast)
{
    uint32_t total;
    const uint32_t ex = block_excl_scan<THREADS>(n_mine, scan_lds, total);
    if (threadIdx.x == 0) bcast[0] = total ? atomicAdd(counter, total) : 0u;
    __syncthreads();
    const uint32_t base = bcast[0];
    __syncthreads();
    return base + ex;
}

__device__ __forceinline__ bool vote_bit(const uint32_t* __restrict__ bits_row, uint32_t j)
{
    return (bits_row[j >> 5] >> (j & 31u)) & 1u;
}

constexpr int kAddUnroll = 4;                     // candidates per thread and reservation
__host__ __device__ constexpr int add_batch(int threads) { return threads * kAddUnroll; }
// A-lists.  Rows whose top-K came from the candidate list: a thread takes kAddUnroll candidates.
// Rows selected from memory (slow_flag == 1): the whole row is read.
template <int THREADS>
__device__ __forceinline__ void ad_collect_add_block(
    uint32_t bx, uint32_t nbx, uint64_t* scan_lds, uint32_t* bcast,
    const float* __restrict__ e, int64_t ld_e, int64_t d,
    const u32x2* __restrict__ cand, uint32_t cap, const uint32_t* __restrict__ row_count,
    const uint32_t* __restrict__ kth_in, const uint32_t* __restrict__ tie_cut_in,
    const uint32_t* __restrict__ slow_flag, const uint32_t* __restrict__ vote_bits, int64_t ld_bits,
    u32x2* __restrict__ a_list, uint32_t* __restrict__ ad_count)
{
    const uint32_t row = blockIdx.y, t = threadIdx.x;
    const uint32_t kth = kth_in[row], tie_cut = tie_cut_in[row];
    const uint32_t* bits = vote_bits + (int64_t)row * ld_bits;
    u32x2* arow = a_list + (size_t)row * cap;
    uint32_t* counter = ad_count + ad_counter(row, 0);
    if (slow_flag[row] == 1u) {
        const float* xrow = e + (int64_t)row * ld_e;
        for (int64_t j0 = (int64_t)bx * THREADS; j0 < d; j0 += (int64_t)nbx * THREADS) {
            const int64_t j = j0 + t;
            u32x2 c = {0u, 0u};
            bool in_a = false;
            if (j < d) {
                c.x = __float_as_uint(xrow[j]) & kAbsMask;
                c.y = (uint32_t)j;
                in_a = is_taken(c, kth, tie_cut) && !vote_bit(bits, c.y);
            }
            const uint32_t pos = reserve_in_list<THREADS>(in_a ? 1u : 0u, counter, scan_lds, bcast);
            if (in_a && pos < cap) arow[pos] = c;
        }
        return;
    }
    const uint32_t C = row_count[row];
    const u32x2* crow = cand + (size_t)row * cap;
    for (uint64_t i0 = (uint64_t)bx * add_batch(THREADS); i0 < C; i0 += (uint64_t)nbx * add_batch(THREADS)) {
        u32x2 c[kAddUnroll];
        uint32_t in_a = 0;
#pragma unroll
        for (int u = 0; u < kAddUnroll; ++u) {
            const uint64_t i = i0 + (uint32_t)u * THREADS + t;
            const u32x2 none = {0u, 0xFFFFFFFFu};
            c[u] = i < C ? crow[i] : none;
        }
#pragma unroll
        for (int u = 0; u < kAddUnroll; ++u)
            if (c[u].y != 0xFFFFFFFFu && is_taken(c[u], kth, tie_cut) && !vote_bit(bits, c[u].y)) in_a |= 1u << u;
        uint32_t pos = reserve_in_list<THREADS>((uint32_t)__popc(in_a), counter, scan_lds, bcast);
#pragma unroll
        for (int u = 0; u < kAddUnroll; ++u)
            if (in_a >> u & 1u) {
                if (pos < cap) arow[pos] = c[u];
                ++pos;
            }
    }
}

// Set bits of one workgroup's stretch staged in LDS per round, 16 (8) loads in flight per thread: rounds follow each
// other, and a stretch may be crowded (2 x 4 M, K = 400,000: 195 us with 4096, 181 so; 2 x 1 M, K = 33,333: 101 and 97).
constexpr int kDropStage = 8192;
// bitmap words per workgroup of mv_ad_collect and of mv_ad_emit, four to a thread (more measured no faster)
__host__ __device__ constexpr int collect_words(int threads) { return threads * 4; }
constexpr int kBitBlockWords = kVoteThreads * 4;
// D-lists: the standing vote's bitmap is scanned, 4 words per thread; a set
// coordinate that is not in the row's top-K goes to the list with the
// complemented magnitude, so that "largest first" selects the smallest magnitudes.
template <int THREADS>
__device__ __forceinline__ void ad_collect_drop_block(
    uint32_t bx, uint64_t* scan_lds, uint32_t* bcast, uint32_t* stage,
    const float* __restrict__ e, int64_t ld_e, int64_t d,
    const uint32_t* __restrict__ kth_in, const uint32_t* __restrict__ tie_cut_in,
    const uint32_t* __restrict__ vote_bits, int64_t ld_bits, uint32_t nwords,
    u32x2* __restrict__ d_list, uint32_t cap_d, uint32_t* __restrict__ ad_count)
{
    const uint32_t row = blockIdx.y, t = threadIdx.x;
    const uint32_t kth = kth_in[row], tie_cut = tie_cut_in[row];
    const float* xrow = e + (int64_t)row * ld_e;
    // the workgroup's stretch of the bitmap: four words per thread
    const uint32_t w0 = bx * collect_words(THREADS) + t * 4;
    uint32_t w[4] = {0, 0, 0, 0};
    if (w0 < nwords) {                            // rows are padded to a multiple of 4 words
        const u32x4 v = *reinterpret_cast<const u32x4*>(vote_bits + (int64_t)row * ld_bits + w0);
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        if ((uint64_t)w0 * 32 + 128 > (uint64_t)d) {             // bits at or beyond d do not exist
#pragma unroll
            for (int q = 0; q < 4; ++q)
                for (int b = 0; b < 32; ++b)
                    if ((int64_t)(w0 + q) * 32 + b >= d) w[q] &= ~(1u << b);
        }
    }
    const uint32_t n_bits = __popc(w[0]) + __popc(w[1]) + __popc(w[2]) + __popc(w[3]);
    uint32_t total;
    const uint32_t ex = block_excl_scan<THREADS>(n_bits, scan_lds, total);
    if (total == 0) return;                                  // whole workgroup
    u32x2* drow = d_list + (size_t)row * cap_d;
    // The members' coordinates are parked in LDS (kDropStage at a time; one round unless the
    // stretch is crowded with votes) and their values then fetched by all lanes together,
    // instead of one dependent load per set bit inside each thread's own loop.
    auto one_round = [&](const uint32_t c0) {
        uint32_t sp = ex;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            for (uint32_t m = w[q]; m != 0u; m &= m - 1) {
                const uint32_t b = __ffs((int)m) - 1;
                if (sp - c0 < (uint32_t)kDropStage) stage[sp - c0] = (w0 + q) * 32 + b;       // sp < c0 wraps: not staged
                ++sp;
            }
        __syncthreads();
        const uint32_t cnt = min((uint32_t)kDropStage, total - c0);
        constexpr int kRounds = kDropStage / THREADS;
        uint32_t x[kRounds];
        uint32_t n_keep = 0, keep = 0;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const uint32_t i = (uint32_t)r * THREADS + t;
            if (i < cnt) {
                const u32x2 c = {__float_as_uint(xrow[stage[i]]) & kAbsMask, stage[i]};
                x[r] = c.x;
                if (!is_taken(c, kth, tie_cut)) {            // left the top-K: a drop candidate
                    keep |= 1u << r;
                    ++n_keep;
                }
            }
        }
        uint32_t pos = reserve_in_list<THREADS>(n_keep, ad_count + ad_counter(row, 1), scan_lds, bcast);
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            if (keep & (1u << r)) {
                if (pos < cap_d) {
                    u32x2 o;
                    o.x = kAbsMask - x[r];
                    o.y = stage[(uint32_t)r * THREADS + t];   // (in LDS and not in a register: units hold more workgroups)
                    drow[pos] = o;
                }
                ++pos;
            }
        }
    };
    if (total <= (uint32_t)kDropStage) {                     // uniform; the usual case
        one_round(0u);
    } else {
        for (uint32_t c0 = 0; c0 < total; c0 += kDropStage) {
            if (c0) __syncthreads();                         // the stage is free again
            one_round(c0);
        }
    }
}

// One launch for both lists: the first add_blocks workgroups of a row walk its
// candidate list (A-list), the others its standing vote's bitmap (D-list).
// (the second bound: 64 registers, so that a unit holds 2048 threads)
template <int THREADS>
__global__ __launch_bounds__(THREADS, 8) void mv_ad_collect(
    const float* __restrict__ e, int64_t ld_e, int64_t d,
    const u32x2* __restrict__ cand, uint32_t cap, const uint32_t* __restrict__ row_count,
    const uint32_t* __restrict__ kth_in, const uint32_t* __restrict__ tie_cut_in,
    const uint32_t* __restrict__ slow_flag, const uint32_t* __restrict__ vote_bits, int64_t ld_bits,
    uint32_t nwords, u32x2* __restrict__ a_list, u32x2* __restrict__ d_list, uint32_t cap_d,
    uint32_t* __restrict__ ad_count, uint32_t add_blocks)
{
    __shared__ uint64_t scan_lds[THREADS / kWave];
    __shared__ uint32_t bcast[1];
    __shared__ uint32_t stage[kDropStage];
    if (blockIdx.x < add_blocks)
        ad_collect_add_block<THREADS>(blockIdx.x, add_blocks, scan_lds, bcast, e, ld_e, d, cand, cap, row_count, kth_in,
                                      tie_cut_in, slow_flag, vote_bits, ld_bits, a_list, ad_count);
    else
        ad_collect_drop_block<THREADS>(blockIdx.x - add_blocks, scan_lds, bcast, stage, e, ld_e, d, kth_in, tie_cut_in,
                                       vote_bits, ld_bits, nwords, d_list, cap_d, ad_count);
}

constexpr int kCollectChunk = 4096;               // coordinates
constexpr int kChunkWords = kCollectChunk / 32, kChunkSegs = kCollectChunk / kSeg;
constexpr int kCollectChunks = collect_words(kCollectThreads) / kChunkWords;     // per workgroup
constexpr int kRemovalStage = 4096;               // removals staged in LDS per round, 8 loads in flight per thread

struct ChunksLds {
    static constexpr int kRuns = kCollectChunks * (kChunkSegs + 1);
    __attribute__((aligned(16))) uint32_t vote[collect_words(kCollectThreads)];
    __attribute__((aligned(16))) uint32_t top[collect_words(kCollectThreads)];
    uint32_t first[kRuns];                        // entries in the runs before
    uint32_t start[kRuns];                        // where the run lies in the row's list
    uint32_t stage[kRemovalStage];
    uint64_t scan[kCollectThreads / kWave];
    uint32_t bcast[1];
};

// Both lists of a row whose list is long, in one pass over its candidates and its standing vote's bitmap.  A workgroup
// owns chunks of 4096 coordinates, gridDim.x apart (votes crowd where gradients are large; see mv_vote_count), finds
// their candidates through the segments' runs, marks the row's top K in a bitmap in LDS and has the standing vote's
// beside it: an addition is a marked candidate without a standing vote, a removal a standing vote without a mark, and
// only the removals' magnitudes have to be fetched from e (looked up candidate by candidate in memory, and all of the
// standing vote fetched, this took 31.5 us instead of 22.8 at 10 x 11.2 M, K = 111,740).  Removals go to the list with
// the complemented magnitude, so that "largest first" selects the smallest magnitudes.
// Rows selected from memory (slow_flag == 1) have no list: their chunks are read instead.
__global__ __launch_bounds__(kCollectThreads) void mv_ad_collect_chunks(
    const float* __restrict__ e, int64_t ld_e, int64_t d, const u32x2* __restrict__ cand, uint32_t cap,
    const u32x2* __restrict__ runs, uint32_t n_runs, RowSegments segs, const uint32_t* __restrict__ kth_in,
    const uint32_t* __restrict__ tie_cut_in, const uint32_t* __restrict__ slow_flag, const uint32_t* __restrict__ vote_bits,
    int64_t ld_bits, uint32_t nwords, u32x2* __restrict__ a_list, u32x2* __restrict__ d_list, uint32_t cap_d,
    uint32_t* __restrict__ ad_count)
{
    constexpr int THREADS = kCollectThreads;
    using Lds = ChunksLds;
    __shared__ Lds lds;
    const uint32_t row = blockIdx.y, t = threadIdx.x;
    const uint32_t kth = kth_in[row], tie_cut = tie_cut_in[row];
    const bool slow = slow_flag[row] == 1u;
    const float* xrow = e + (int64_t)row * ld_e;
    const u32x2* crow = cand + (size_t)row * cap;
    auto chunk_of = [&](uint32_t m) { return blockIdx.x + m * gridDim.x; };
    // the thread's four words of the bitmap
    const uint32_t own = t * 4, m_own = own / kChunkWords;
    const uint64_t w0 = (uint64_t)chunk_of(m_own) * kChunkWords + own % kChunkWords;
    u32x4 w = {0u, 0u, 0u, 0u};
    if (w0 < nwords)                              // (padded to a multiple of 4 words)
        w = *reinterpret_cast<const u32x4*>(vote_bits + (int64_t)row * ld_bits + w0);
    u32x2 run = {0u, 0u};
    if (t < (uint32_t)Lds::kRuns) {
        const uint32_t m = t / (kChunkSegs + 1), slot = t % (kChunkSegs + 1);
        const uint32_t shift = segs.shift(row), n_segs = segs.count(row);
        const uint64_t s = (uint64_t)chunk_of(m) * kChunkSegs + slot;
        // (a chunk's last segment is shared with the next one where the row is shifted)
        if (s < n_segs && (uint64_t)chunk_of(m) * kCollectChunk < (uint64_t)d &&
            (slot < (uint32_t)kChunkSegs || shift != 0u) && !slow)
            run = runs[(size_t)row * n_runs + s];           // (in order: see order_runs)
    }
    if (w0 < nwords && w0 * 32 + 128 > (uint64_t)d) {                // bits at or beyond d do not exist
#pragma unroll
        for (int q = 0; q < 4; ++q)
            for (int b = 0; b < 32; ++b)
                if ((int64_t)(w0 + q) * 32 + b >= d) w[q] &= ~(1u << b);
    }
    *reinterpret_cast<u32x4*>(&lds.vote[own]) = w;
    *reinterpret_cast<u32x4*>(&lds.top[own]) = u32x4{0u, 0u, 0u, 0u};
    uint32_t total;
    const uint32_t before = block_excl_scan<THREADS>(run.y, lds.scan, total);
    if (t < (uint32_t)Lds::kRuns) {
        lds.first[t] = before;
        lds.start[t] = run.x;
    }
    if (slow) total = collect_words(kCollectThreads) * 32;                   // uniform: every coordinate is an entry
    __syncthreads();
    u32x2* arow = a_list + (size_t)row * cap;
    for (uint32_t i0 = 0; i0 < total; i0 += THREADS * kAddUnroll) {
        u32x2 c[kAddUnroll];
        uint32_t at[kAddUnroll];                  // place in the workgroup's bitmaps, where it is the workgroup's
        uint32_t in_a = 0;
#pragma unroll
        for (int u = 0; u < kAddUnroll; ++u) {
            const uint32_t i = i0 + (uint32_t)u * THREADS + t;
            c[u] = u32x2{0u, 0xFFFFFFFFu};
            at[u] = 0xFFFFFFFFu;
            if (i >= total) continue;
            if (slow) {
                const uint64_t j = (uint64_t)chunk_of(i / kCollectChunk) * kCollectChunk + i % kCollectChunk;
                if (j < (uint64_t)d) c[u] = u32x2{__float_as_uint(xrow[j]) & kAbsMask, (uint32_t)j};
                at[u] = i;
            } else {
                uint32_t r = 0;                   // the last run that begins at or before entry i
#pragma unroll
                for (uint32_t step = 128; step != 0; step >>= 1)
                    if (r + step < (uint32_t)Lds::kRuns && lds.first[r + step] <= i) r += step;
                c[u] = crow[lds.start[r] + (i - lds.first[r])];
                at[u] = r / (kChunkSegs + 1);     // the chunk's number
            }
        }
#pragma unroll
        for (int u = 0; u < kAddUnroll; ++u) {
            if (!slow) {
                const uint32_t off = c[u].y - chunk_of(at[u]) * kCollectChunk;
                at[u] = c[u].y != 0xFFFFFFFFu && off < (uint32_t)kCollectChunk ? at[u] * kCollectChunk + off : 0xFFFFFFFFu;
            }
            if (c[u].y == 0xFFFFFFFFu || at[u] == 0xFFFFFFFFu || !is_taken(c[u], kth, tie_cut)) continue;
            const uint32_t bit = 1u << (at[u] & 31u);
            atomicOr(&lds.top[at[u] / 32], bit);
            if (!(lds.vote[at[u] / 32] & bit)) in_a |= 1u << u;
        }
        uint32_t pos = reserve_in_list<THREADS>((uint32_t)__popc(in_a), ad_count + ad_counter(row, 0), lds.scan, lds.bcast);
#pragma unroll
        for (int u = 0; u < kAddUnroll; ++u)
            if (in_a >> u & 1u) {
                if (pos < cap) arow[pos] = c[u];
                ++pos;
            }
    }
    __syncthreads();
    // the removals: their coordinates are parked in LDS (kRemovalStage at a time; one round unless the chunks are
    // crowded with them) and their values then fetched by all lanes together, instead of one dependent load per set
    // bit inside each thread's own loop
    uint32_t n_bits = 0;
    {
        const u32x4 top = *reinterpret_cast<const u32x4*>(&lds.top[own]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            w[q] &= ~top[q];
            n_bits += (uint32_t)__popc(w[q]);
        }
    }
    const uint32_t ex = block_excl_scan<THREADS>(n_bits, lds.scan, total);
    if (total == 0) return;                       // whole workgroup
    if (t == 0) lds.bcast[0] = atomicAdd(ad_count + ad_counter(row, 1), total);
    u32x2* drow = d_list + (size_t)row * cap_d;
    for (uint32_t c0 = 0; c0 < total; c0 += kRemovalStage) {
        if (c0) __syncthreads();                  // the stage is free again
        uint32_t sp = ex;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            for (uint32_t m = w[q]; m != 0u; m &= m - 1) {
                const uint32_t b = __ffs((int)m) - 1;
                if (sp - c0 < (uint32_t)kRemovalStage)           // (sp < c0 wraps: not staged)
                    lds.stage[sp - c0] = (uint32_t)(w0 + q) * 32 + b;
                ++sp;
            }
        __syncthreads();
        const uint32_t cnt = min((uint32_t)kRemovalStage, total - c0), to = lds.bcast[0] + c0;
        constexpr int kRounds = kRemovalStage / THREADS;
        uint32_t x[kRounds];
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const uint32_t i = (uint32_t)r * THREADS + t;
            x[r] = i < cnt ? __float_as_uint(xrow[lds.stage[i]]) & kAbsMask : 0u;
        }
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const uint32_t i = (uint32_t)r * THREADS + t;
            if (i < cnt && to + i < cap_d) drow[to + i] = u32x2{kAbsMask - x[r], lds.stage[i]};
        }
    }
}

// The K_ad first of row n's A-list under (magnitude desc, coordinate asc), and the same for the D-list, whose
// keys are the complemented magnitudes: list number 2n + which.  All of A is at or above the row's K-th
// magnitude and all of D at or below it, so the keys start there.  A crowds right above: 1024 bins to an octave
// for half an octave, then 32; D reaches far down: 128 bins to an octave for four octaves, then 32.
__device__ __forceinline__ ListView ad_list(uint32_t number, const u32x2* __restrict__ a_list, uint32_t cap_a,
                                            const u32x2* __restrict__ d_list, uint32_t cap_d,
                                            const uint32_t* __restrict__ ad_count, uint32_t k_ad,
                                            const uint32_t* __restrict__ kth_in, uint32_t* __restrict__ sample_hist)
{
    const uint32_t row = number / 2, which = number % 2;
    ListView v;
    v.list = which ? d_list + (size_t)row * cap_d : a_list + (size_t)row * cap_a;
    v.n = min(ad_count[ad_counter(row, which)], which ? cap_d : cap_a);
    v.want = k_ad;
    v.base = which ? kAbsMask - kth_in[row] : kth_in[row];
    v.fine = which ? 16 : 13;
    v.coarse = 18;
    lend_storage(v, sample_hist, row, which);
    return v;
}

// Long lists only (see list_split): the histograms
__global__ __launch_bounds__(kRowThreads) void mv_ad_hist(const u32x2* __restrict__ a_list, uint32_t cap_a,
                                                          const u32x2* __restrict__ d_list, uint32_t cap_d,
                                                          const uint32_t* __restrict__ ad_count, uint32_t k_ad,
                                                          const uint32_t* __restrict__ kth_in,
                                                          uint32_t* __restrict__ sample_hist)
{
    __shared__ uint32_t hist[kListBins];
    const ListView v = ad_list(blockIdx.y, a_list, cap_a, d_list, cap_d, ad_count, k_ad, kth_in, sample_hist);
    if (v.n <= k_ad) return;                      // whole workgroup: all of the list is taken
    list_hist(v, blockIdx.x, gridDim.x, hist);
}

// Selects and applies the additions and removals: marks them in the row's scratch bitmap (one bitmap for
// both: a marked coordinate that is in the standing vote is a removal, one that is not is an addition), counts
// them per block of the bitmap, and moves msum by +1 / -1 (bytes packed four to a word; a byte never carries
// because 0 <= msum <= N <= 255 holds before and after).  counts_out[2n + which] = how many are taken =
// min(K_ad, list length).  Grid (workgroups of a list, 2N); ALONE: one workgroup per list.
template <bool ALONE>
__global__ __launch_bounds__(kRowThreads) void mv_ad_pick(
    const u32x2* __restrict__ a_list, uint32_t cap_a, const u32x2* __restrict__ d_list, uint32_t cap_d,
    const uint32_t* __restrict__ ad_count, uint32_t k_ad, const uint32_t* __restrict__ kth_in,
    uint32_t* __restrict__ sample_hist, u32x2* __restrict__ list2, uint32_t* __restrict__ ad_bits,
    uint32_t nwords_pad, uint32_t nblk, u32x2* __restrict__ blk_cnt, uint32_t* __restrict__ msum32,
    uint32_t* __restrict__ counts_out)
{
    __shared__ SplitLds<kMembers> lds;
    const uint32_t row = blockIdx.y / 2, which = blockIdx.y % 2;
    ListView v = ad_list(blockIdx.y, a_list, cap_a, d_list, cap_d, ad_count, k_ad, kth_in, sample_hist);
    // the second lists share a row of storage (at most 2K and at most d entries together): one from each end
    v.list2 = list2 + (size_t)row * cap_a + (which ? cap_a - 1 : 0);
    v.step2 = which ? -1 : 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) counts_out[blockIdx.y] = min(v.n, k_ad);
    uint32_t* bits = ad_bits + (size_t)row * nwords_pad;
    const BlockTally tally = {lds.tally, reinterpret_cast<uint32_t*>(blk_cnt + (size_t)row * nblk) + which, 2, nblk};
    tally.clear();
    auto apply = [&](const u32x2 (&c)[kListUnroll], uint32_t taken) {
#pragma unroll
        for (int u = 0; u < kListUnroll; ++u) {
            const bool mine = taken >> u & 1u;
            if (mine) {
                atomicOr(&bits[c[u].y >> 5], 1u << (c[u].y & 31u));
                const uint32_t one = 1u << ((c[u].y & 3u) * 8u);
                if (which) atomicSub(&msum32[c[u].y >> 2], one);
                else       atomicAdd(&msum32[c[u].y >> 2], one);
            }
            tally.add(c[u].y / (32u * kBitBlockWords), mine);
        }
    };
    if (v.n <= k_ad) {                            // all of the list is taken
        __syncthreads();
        for (uint64_t i0 = (uint64_t)blockIdx.x * kListBatch; i0 < v.n; i0 += (uint64_t)gridDim.x * kListBatch) {
            u32x2 c[kListUnroll];
            uint32_t taken = 0;
#pragma unroll
            for (int u = 0; u < kListUnroll; ++u) {
                const uint64_t i = i0 + (uint32_t)u * kRowThreads + threadIdx.x;
                const u32x2 none = {0u, 0xFFFFFFFFu};
                c[u] = i < v.n ? v.list[i] : none;
                taken |= (i < v.n ? 1u : 0u) << u;
            }
            apply(c, taken);
        }
    } else {
        uint32_t kth, tie_cut;
        ListRest rest;
        (void)list_split<ALONE ? SplitEnd::Alone : SplitEnd::Last>(v, blockIdx.x, gridDim.x, lds, apply, kth, tie_cut, rest);
    }
    tally.merge();
}

// Histogram of the vote levels of msum (one byte per coordinate, values 0..N) over a
// block of kVoteBlock coordinates: lvl_sets[set][v] += coordinates with exactly v votes.
__device__ __forceinline__ void ad_levels_block(const uint32_t* __restrict__ msum32, int64_t d,
                                                uint32_t* __restrict__ lvl_sets, uint32_t bx, uint32_t* h /*256*/)
{
    static_assert(kVoteBlock == kVoteThreads * 16, "16 coordinates per thread");
    const int64_t j = (int64_t)bx * kVoteBlock + (int64_t)threadIdx.x * 16;
    const u32x4 z = {0u, 0u, 0u, 0u};
    const u32x4 w = j < d ? *reinterpret_cast<const u32x4*>(msum32 + (j >> 2)) : z;
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    if ((w.x | w.y | w.z | w.w) != 0u) {          // most coordinates have no vote
        const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const uint32_t v = (ww[q >> 2] >> (8 * (q & 3))) & 255u;
            if (v && j + q < d) atomicAdd(&h[v], 1u);
        }
    }
    __syncthreads();
    const uint32_t c = threadIdx.x < 256 ? h[threadIdx.x] : 0u;
    if (c && threadIdx.x) atomicAdd(&lvl_sets[(size_t)(bx % kLvlSets) * 256 + threadIdx.x], c);
}

// One launch behind mv_ad_pick.  The first n_emit_blocks workgroups (row = id / nblk): ordered compaction of the
// scratch bitmaps -- from the counts of the blocks before its own and a scan inside the block every thread writes
// its marked coordinates in ascending order to the add list or the drop list -- and the scratch words are cleared
// and folded into the standing vote.  The others take the histogram of msum's levels.
__global__ __launch_bounds__(kVoteThreads) void mv_ad_emit(uint32_t* __restrict__ ad_bits, uint32_t nwords_pad,
                                                           uint32_t nblk, const u32x2* __restrict__ blk_cnt,
                                                           uint32_t k_ad, uint32_t* __restrict__ add_idx,
                                                           uint32_t* __restrict__ drop_idx,
                                                           uint32_t* __restrict__ vote_bits, int64_t ld_bits,
                                                           uint32_t n_emit_blocks, const uint32_t* __restrict__ msum32,
                                                           int64_t d, uint32_t* __restrict__ lvl_sets)
{
    __shared__ uint64_t scan_lds[kVoteThreads / kWave];
    __shared__ uint32_t h[256];
    if (blockIdx.x >= n_emit_blocks) {
        ad_levels_block(msum32, d, lvl_sets, blockIdx.x - n_emit_blocks, h);
        return;
    }
    const uint32_t row = blockIdx.x / nblk, bx = blockIdx.x % nblk;
    uint32_t* vrow = vote_bits + (int64_t)row * ld_bits;
    // the thread's words first (cleared behind): their latency overlaps the prefix's loads
    const uint32_t w0 = bx * kBitBlockWords + threadIdx.x * 4;
    uint32_t w[4] = {0, 0, 0, 0}, in_vote[4] = {0, 0, 0, 0};
    if (w0 < nwords_pad) {
        u32x4* p = reinterpret_cast<u32x4*>(ad_bits + (size_t)row * nwords_pad + w0);
        const u32x4 v = *p;
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        if ((v.x | v.y | v.z | v.w) != 0u) {
            const u32x4 z = {0u, 0u, 0u, 0u};
            *p = z;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (w[q]) in_vote[q] = vrow[w0 + q];
        }
    }
    uint64_t mine = 0;
    for (uint32_t b = threadIdx.x; b < bx; b += kVoteThreads) {
        const u32x2 c = blk_cnt[(size_t)row * nblk + b];
        mine += pack2(c.x, c.y);
    }
    uint64_t before;
    (void)block_excl_scan64<kVoteThreads>(mine, scan_lds, before);
    __syncthreads();
    uint32_t* out_add = add_idx + (size_t)row * k_ad;
    uint32_t* out_drop = drop_idx + (size_t)row * k_ad;
    uint32_t n_add = 0, n_drop = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        n_add += __popc(w[q] & ~in_vote[q]);
        n_drop += __popc(w[q] & in_vote[q]);
    }
    uint64_t total;
    const uint64_t at = before + block_excl_scan64<kVoteThreads>(pack2(n_add, n_drop), scan_lds, total);
    uint32_t pos_add = (uint32_t)(at >> 32), pos_drop = (uint32_t)at;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (w[q]) atomicXor(&vrow[w0 + q], w[q]);   // additions enter the standing vote, removals leave it
        for (uint32_t m = w[q]; m != 0u; m &= m - 1) {
            const uint32_t b = __ffs((int)m) - 1, j = (w0 + q) * 32 + b;
            if ((in_vote[q] >> b) & 1u) {
                if (pos_drop < k_ad) out_drop[pos_drop] = j;
                ++pos_drop;
            } else {
                if (pos_add < k_ad) out_add[pos_add] = j;
                ++pos_add;
            }
        }
    }
}

}  // namespace mvk
