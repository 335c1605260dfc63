// The global mask (counting sort over the vote levels, ordered emission), the masked gather / mean / error update,
// and beside one of the two (in random selection beside mv_rs_pick) the sorted vote lists.
//
// These kernels are short (a few dependent memory round trips each), and the chip
// starts only a few hundred workgroups per microsecond: they use workgroups of 1024
// threads and grids of a few hundred workgroups.
#pragma once

#include "mv_common.hpp"
#include "mv_select.hpp"

namespace mvk {

constexpr int kMaskThreads = 1024;   // mv_mask_count / mv_gather_update
constexpr int kLookBack = 256;       // earlier blocks whose totals a block of mv_mask_count adds up itself

// ----------------------------------------------------------------------------
// 5. global mask = the K most voted coordinates, ties to the lowest coordinate
// ----------------------------------------------------------------------------
// Counting sort over the vote levels 0..N in two kernels.  The level counters (summed
// over their sets) say how many coordinates hold at least v votes (where the votes were
// cast from the lists) or exactly v votes (where mv_vote_count counted them, and in
// add-drop voting: a histogram of the vote sum).  The threshold v* is the level at which
// K coordinates are covered walking down from N: all coordinates above v* are taken, and
// the first K - (#above) coordinates, in coordinate order, with exactly v* votes.  A block is the 16384 Q
// coordinates of one workgroup (Q = 1 to 8 quads of 16 vote bytes per thread, chosen
// so that the grid stays at a few hundred workgroups).  mv_mask_count counts, per
// wavefront's stretch of the vote bytes, the coordinates above and at v*;
// mv_gather_update turns the counts of the earlier stretches into positions: each of
// its workgroups emits the part of the mask it gathers.

// All threads of the workgroup: vstar / take_eq from the level counters.  Thread v has level v: which
// level the K-th falls into is one comparison per thread, not a walk down the levels one by one.
__device__ __forceinline__ void vote_threshold(const uint32_t* __restrict__ lvl_sets, uint32_t N, uint32_t K,
                                               uint32_t* lvl /*LDS, 256*/, uint32_t* thr /*LDS, 2*/,
                                               uint64_t* scan_lds, uint32_t& vstar, uint32_t& take_eq,
                                               int exact_levels)
{
    const uint32_t t = threadIdx.x;
    // exact_levels: thread t has level N - t (t < N), so that the scan runs from the top down
    const uint32_t v = exact_levels ? (t < N ? N - t : 256u) : t;
    uint32_t sum = 0;
    if (t < 256) {                                // the level's sets are added up, all loads in flight together
        uint32_t c[kLvlSets];
#pragma unroll
        for (int q = 0; q < kLvlSets; ++q) c[q] = (v <= N) ? lvl_sets[(size_t)q * 256 + v] : 0u;
#pragma unroll
        for (int q = 0; q < kLvlSets; ++q) sum += c[q];
    }
    if (exact_levels) {
        // coordinates with EXACTLY v votes, v = N..1: the level at which K coordinates are covered from the
        // top; level 0 (every other coordinate) covers whatever is left
        uint32_t total;
        const uint32_t above = block_excl_scan<kMaskThreads>(sum, scan_lds, total);
        if (above < K && K <= above + sum) {
            thr[0] = v;
            thr[1] = K - above;
        }
        if (t == 0 && total < K) {
            thr[0] = 0;
            thr[1] = K - total;
        }
    } else {
        // coordinates with AT LEAST v votes, v = 1..N; at least K coordinates hold a vote
        if (t < 256) lvl[t] = sum;
        __syncthreads();
        if (t >= 1 && t <= N) {
            const uint32_t above = t < N ? lvl[t + 1] : 0u;
            if (above < K && (sum >= K || t == 1)) {
                thr[0] = t;
                thr[1] = K - above;
            }
        }
    }
    __syncthreads();
    vstar = thr[0];
    take_eq = thr[1];
}

// The bytes of x that are >= t (1 <= t <= 255), as the low bit of each byte: the low seven bits are
// compared by one subtraction that borrows from the eighth.
__device__ __forceinline__ uint32_t bytes_at_least(uint32_t x, uint32_t t)
{
    const uint32_t top = 0x80808080u;
    const uint32_t low = (x | top) - (t & 127u) * 0x01010101u;
    return ((t & 128u) ? x & low : x | low) >> 7 & 0x01010101u;
}
// A wavefront owns a stretch of 1024 Q coordinates, quad q of lane l being its 16 coordinates from
// kQuadStep q + 16 l on: 64 lanes read, and copy, a kilobyte in a row (with the Q quads of a thread in a row every
// instruction touched 64 separate pieces, and the copy of the votes alone took 14 of the mask kernel's 37 us at
// 32 x 25.6 M).
constexpr int kQuadStep = 16 * kWave;
// The thread's coordinates with more than / exactly vstar votes, its first quad lying at coordinate j0: bit b of
// marks[q] is set if coordinate j0 + kQuadStep q + b has more, bit 16 + b if it has exactly vstar.  Four bytes at a
// time (byte by byte, and once more for the emission, the mask kernel took 18.5 us instead of 14.9 at 10 x 11.2 M,
// K = 111,740, and 37 instead of 32 at 32 x 25.6 M).  Must be called by all lanes of a wavefront together: a quad that
// holds no vote in any lane is passed over by the whole wavefront (most quads, where votes are sparse); with
// vstar == 0 the coordinates without a vote count too and nothing is passed over.  A thread's only quad is not worth
// the question (7 x 272,475 bf16, steps 30.76 us : 30.65).
// before[q]: those of the stretch that lie before quad q of this lane, above | at << 16; returns the stretch's.
template <int Q>
__device__ __forceinline__ uint32_t count_above_and_at(const u32x4 (&w)[Q], int64_t j0, int64_t d, uint32_t vstar,
                                                       uint32_t (&marks)[Q], uint32_t (&before)[Q])
{
    static_assert(kQuadStep * 8 < 1 << 16, "a stretch's counts fit 16 bits");
    uint32_t sum = 0;                             // uniform: over the quads so far
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        marks[q] = 0;
        before[q] = sum;
        const uint32_t any = w[q].x | w[q].y | w[q].z | w[q].w;
        if (Q > 1 && vstar != 0u && __ballot(any != 0u) == 0ull) continue;     // wave-uniform
        uint32_t above[2] = {0, 0}, from[2] = {0, 0};                 // eight coordinates each
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t x = w[q][k], weights = k & 1 ? 0x80402010u : 0x08040201u;
            if (vstar < 255u) above[k / 2] = __builtin_amdgcn_udot4(bytes_at_least(x, vstar + 1u), weights, above[k / 2], false);
            if (vstar != 0u) from[k / 2] = __builtin_amdgcn_udot4(bytes_at_least(x, vstar), weights, from[k / 2], false);
        }
        const uint32_t up = above[0] | above[1] << 8;
        uint32_t all = from[0] | from[1] << 8;
        if (vstar == 0u) {                        // uniform: every coordinate there is
            const int64_t there = d - (j0 + kQuadStep * q);
            all = there >= 16 ? 0xFFFFu : there > 0 ? (1u << there) - 1u : 0u;
        }
        marks[q] = up | (all & ~up) << 16;
        if (Q > 1 && __ballot(marks[q] != 0u) == 0ull) continue;      // wave-uniform
        const uint32_t mine = (uint32_t)__popc(up) | (uint32_t)__popc(all & ~up) << 16;
        const uint32_t incl = wave_incl_scan(mine);
        before[q] = sum + incl - mine;
        sum += from_lane(incl, kWave - 1);
    }
    return sum;
}

// f(position, coordinate) for every mask coordinate among the thread's, g0 being the coordinates above the
// threshold before the wavefront's stretch and e0 those at it.
template <int Q, typename F>
__device__ __forceinline__ void each_mask_position(const uint32_t (&marks)[Q], const uint32_t (&before)[Q], int64_t j0,
                                                   uint32_t g0, uint32_t e0, uint32_t take_eq, F f)
{
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        uint32_t g = g0 + (before[q] & 0xFFFFu), e = e0 + (before[q] >> 16);
        const uint32_t up = marks[q] & 0xFFFFu, at = marks[q] >> 16;
        if (up == 0u && e >= take_eq) continue;
        for (uint32_t m = up | at; m != 0u; m &= m - 1u) {
            const uint32_t low = m & (0u - m);
            const bool is_up = (up & low) != 0u;
            if (is_up || e < take_eq) f(g + min(e, take_eq), (uint32_t)(j0 + kQuadStep * q) + (uint32_t)__ffs((int)low) - 1u);
            if (is_up) ++g;
            else ++e;
        }
    }
}

// ---- the sorted vote lists
constexpr int kMaskWaves = kMaskThreads / kWave;
constexpr int kEmitUnroll = 4;                    // list entries per thread in flight together
constexpr int kEmitBatch = kMaskThreads * kEmitUnroll;
constexpr int kListUnits = 4 * kMaskThreads;      // prefixes of a row's tallies in LDS, four to a thread
static_assert(kEmitUnroll * kMaskWaves == kWave, "a lane per wavefront's part of a batch");
struct EmitLds {
    uint32_t before[kListUnits];                  // taken entries in the units of segments before
    uint32_t wave_taken[kEmitUnroll * kMaskWaves];
    uint32_t wave_earlier[kMaskWaves];
    uint16_t number[kEmitBatch];                  // taken entries of the batch before each of its entries
};

// A row's vote list in ascending coordinate order, without a sort: a taken candidate's rank is (taken
// candidates in the segments before its own, from the tallies) + (before it in its own run; runs are ascending).
// A few workgroups per row (`part` of `parts`); each adds up the row's tallies for itself, eight segments to a
// prefix (1365 for 11.2 M coordinates), which arrive beside the entries, and an entry looks at its own eight segments'
// tallies again (32 x 25.6 M: mask kernel 36.6 us, 73 with a prefix for every two segments).  n_dealt: the segments
// whose runs lie as the streaming pass noted them (run_place), none once they are in order.
__device__ __forceinline__ void write_row_list(const u32x2* __restrict__ crow, uint32_t C,
                                               const u32x2* __restrict__ runs, const u32x4* __restrict__ units,
                                               uint32_t n_segs, uint32_t n_dealt, uint32_t shift, uint32_t K, uint32_t kth, uint32_t tie_cut,
                                               uint32_t part, uint32_t parts, uint32_t* __restrict__ out, EmitLds& lds,
                                               uint64_t* scan_lds)
{
    if ((uint64_t)part * kEmitBatch >= C) return;            // whole workgroup
    const uint32_t t = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave);
    u32x2 c[kEmitUnroll];
    uint32_t run0[kEmitUnroll], first_run = 0;    // where the entries' runs begin, and the first entry's of the batch
    uint32_t below[kEmitUnroll];                  // taken in the segments of the entry's unit before its own
    auto load = [&](uint64_t i0) {
#pragma unroll
        for (int u = 0; u < kEmitUnroll; ++u) {
            const uint64_t i = i0 + (uint64_t)u * kMaskThreads + t;
            const u32x2 none = {0u, 0xFFFFFFFFu};
            c[u] = (i < C) ? crow[i] : none;
        }
        first_run = segment_of(crow[i0].y, shift);       // uniform
    };
    auto load_runs = [&]() {
#pragma unroll
        for (int u = 0; u < kEmitUnroll; ++u) {
            run0[u] = 0;
            below[u] = 0;
            if (c[u].y != 0xFFFFFFFFu) {
                const uint32_t s = segment_of(c[u].y, shift);
                run0[u] = runs[run_place(s, n_dealt)].x;
                below[u] = unit_sum_below(units[s / kTallyUnit], s % kTallyUnit);
            }
        }
        first_run = runs[run_place(first_run, n_dealt)].x;
    };
    load((uint64_t)part * kEmitBatch);
    // `per` units to a prefix: one, in rows of up to 33.5 M coordinates
    const uint32_t n_units = (n_segs + kTallyUnit - 1) / kTallyUnit, per = (n_units + kListUnits - 1) / kListUnits;
    {
        uint32_t v[4];
        uint32_t sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t r0 = (4u * t + q) * per;
            v[q] = r0 < n_units ? unit_sum(units[r0]) : 0u;
            for (uint32_t r = r0 + 1; r < min(r0 + per, n_units); ++r) v[q] += unit_sum(units[r]);
        }
        load_runs();
#pragma unroll
        for (int q = 0; q < 4; ++q) sum += v[q];
        uint32_t total;
        uint32_t ex = block_excl_scan<kMaskThreads>(sum, scan_lds, total);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            lds.before[4u * t + q] = ex;
            ex += v[q];
        }
    }
    __syncthreads();
    // A workgroup takes kEmitBatch consecutive entries at a time and numbers the taken ones; an entry's rank
    // inside its run is the difference of two such numbers.  Only the first entry's run can have begun before
    // the batch: that part (fewer than kSeg entries) is counted by all threads together.
    for (uint64_t i0 = (uint64_t)part * kEmitBatch; i0 < C; i0 += (uint64_t)parts * kEmitBatch) {
        if (i0 != (uint64_t)part * kEmitBatch) {
            load(i0);
            load_runs();
        }
        uint32_t n_earlier = 0;
        {
            static_assert(kSeg <= kMaskThreads, "a thread per entry of a run");
            if (first_run < i0) {                                    // uniform
                const uint64_t j = min((uint64_t)first_run + t, i0 - 1);
                n_earlier = (uint32_t)__popcll(__ballot(first_run + t < i0 && is_taken(crow[j], kth, tie_cut)));
            }
        }
        uint32_t mine[kEmitUnroll];               // taken ones in the lanes below
        uint32_t taken = 0;
#pragma unroll
        for (int u = 0; u < kEmitUnroll; ++u) {
            const bool tk = c[u].y != 0xFFFFFFFFu && is_taken(c[u], kth, tie_cut);
            const uint64_t all = __ballot(tk);
            taken |= (tk ? 1u : 0u) << u;
            mine[u] = (uint32_t)__popcll(all & ((1ull << lane) - 1ull));
            if (lane == 0) lds.wave_taken[u * kMaskWaves + wave] = (uint32_t)__popcll(all);
        }
        if (lane == 0) lds.wave_earlier[wave] = n_earlier;
        __syncthreads();
        // the taken ones before each wavefront's part of the batch, in the order of the entries
        const uint32_t batch_part = lds.wave_taken[lane];
        const uint32_t before = wave_incl_scan(batch_part) - batch_part;
        const uint32_t carry_lanes = row_incl_scan(lane < (uint32_t)kMaskWaves ? lds.wave_earlier[lane] : 0u);
        const uint32_t carry = from_lane(carry_lanes, kMaskWaves - 1);
#pragma unroll
        for (int u = 0; u < kEmitUnroll; ++u) {
            mine[u] += from_lane(before, (uint32_t)u * kMaskWaves + wave);
            lds.number[u * kMaskThreads + t] = (uint16_t)mine[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kEmitUnroll; ++u)
            if (taken >> u & 1u) {
                const uint32_t r = segment_of(c[u].y, shift) / kTallyUnit, p = r / per;
                uint32_t pos = lds.before[p] + below[u] + (run0[u] >= i0 ? mine[u] - lds.number[run0[u] - i0] : mine[u] + carry);
                for (uint32_t q = p * per; q < r; ++q) pos += unit_sum(units[q]);
                if (pos < K) out[pos] = c[u].y;
            }
        __syncthreads();                          // the scratch is free for the next batch
    }
}

// The lists of all rows, by `per_row` workgroups to a row behind a kernel's own.  They run beside the mask kernel's
// blocks where those mostly wait for each other, in random selection beside mv_rs_pick, and beside the gather otherwise
// (mv_api.hip has the lines).
struct RowLists {
    uint32_t        per_row;
    const u32x2*    cand;
    uint32_t        cap;
    const uint32_t* row_count;
    const u32x2*    runs;
    int             in_order;                     // the runs are (see order_runs)
    const uint32_t* run_taken;
    uint32_t        n_runs;
    RowSegments     segs;
    const uint32_t *kth, *tie_cut, *slow_flag;
    uint32_t*       worker_idx;
};
__device__ __forceinline__ void write_row_lists(const RowLists& l, uint32_t block, uint32_t K, EmitLds& lds, uint64_t* scan_lds)
{
    const uint32_t row = block / l.per_row, part = block % l.per_row;
    if (l.slow_flag[row] == 1u) return;                        // its list is written already
    write_row_list(l.cand + (size_t)row * l.cap, l.row_count[row], l.runs + (size_t)row * l.n_runs,
                   reinterpret_cast<const u32x4*>(l.run_taken) + (size_t)row * (l.n_runs / kTallyUnit), l.segs.count(row),
                   l.in_order ? 0u : l.segs.count(row), l.segs.shift(row), K, l.kth[row], l.tie_cut[row], part, l.per_row,
                   l.worker_idx + (size_t)row * K, lds, scan_lds);
}

// Random selection: the winners are marked in a bitmap and counted per block already, so a block's
// mask follows from the counts of the blocks before it.  `halves`: the bitmap, 16 coordinates to a
// half-word; it is left at zero.
template <int Q>
__device__ __forceinline__ void write_winners(uint16_t* __restrict__ halves, const uint32_t* __restrict__ winners_per_block,
                                              int64_t d, uint32_t K, uint64_t* scan_lds, uint32_t* __restrict__ mask_idx)
{
    const int64_t h0 = ((int64_t)blockIdx.x * kMaskThreads + threadIdx.x) * Q;
    uint32_t m[Q];
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        m[q] = (h0 + q) * 16 < d ? halves[h0 + q] : 0u;
        mine += (uint32_t)__popc(m[q]);
    }
    uint32_t before = 0;
    for (uint32_t b = threadIdx.x; b < blockIdx.x; b += kMaskThreads) before += winners_per_block[b];
    uint64_t total;
    const uint64_t ex = block_excl_scan64<kMaskThreads>(pack2(before, mine), scan_lds, total);
    uint32_t pos = (uint32_t)(total >> 32) + (uint32_t)ex;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (m[q]) halves[h0 + q] = 0;
        for (uint32_t w = m[q]; w != 0u; w &= w - 1u, ++pos)
            if (pos < K) mask_idx[pos] = (uint32_t)((h0 + q) * 16) + (uint32_t)__ffs((int)w) - 1u;
    }
}

// Workgroups [0, n_vote_blocks): count the block's coordinates above and at the vote
// threshold (also per wavefront's stretch of 1024 Q coordinates), exchange the counts
// with the other blocks and write the block's part of the mask; optionally copy the vote
// bytes to the caller.  Workgroups beyond write the sorted vote lists, where they run
// beside this kernel.  RANDOM: the mask comes from the winners' bitmap.
template <int Q, bool RANDOM>
__global__ __launch_bounds__(kMaskThreads) void mv_mask_count(const uint32_t* __restrict__ votes32,
                                                              int64_t d, uint32_t N, uint32_t K,
                                                              const uint32_t* __restrict__ lvl_sets,
                                                              u32x2* __restrict__ sub_cnt,
                                                              u32x2* __restrict__ block_cnt,
                                                              uint32_t* __restrict__ vote_thr,
                                                              uint8_t* __restrict__ votes_out,
                                                              uint32_t n_vote_blocks, RowLists lists,
                                                              int exact_levels,
                                                              unsigned long long* __restrict__ lookback,
                                                              uint32_t* __restrict__ emit_fail, uint32_t spin_limit,
                                                              uint32_t* __restrict__ mask_idx,
                                                              uint16_t* __restrict__ winners,
                                                              const uint32_t* __restrict__ winners_per_block)
{
    __shared__ uint32_t lvl[256];
    __shared__ uint32_t thr[2];
    __shared__ uint64_t scan_lds[kMaskThreads / kWave + 1];
    __shared__ uint32_t mask_found;
    __shared__ uint64_t before_sh;
    if constexpr (!RANDOM) {
        if (blockIdx.x >= n_vote_blocks) {
            __shared__ EmitLds emit;
            write_row_lists(lists, blockIdx.x - n_vote_blocks, K, emit, scan_lds);
            return;
        }
    }
    // the block's vote words first: their latency overlaps the level counters' loads
    const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t j0 = ((int64_t)blockIdx.x * (kMaskThreads / kWave) + wave) * (kQuadStep * Q) + lane * 16;
    u32x4 w[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t j = j0 + q * kQuadStep;
        const u32x4 z = {0u, 0u, 0u, 0u};
        w[q] = (j < d) ? *reinterpret_cast<const u32x4*>(votes32 + (j >> 2)) : z;   // padded to 16 bytes with zeros
    }
    uint32_t vstar = 0, take_eq = 0;
    if constexpr (!RANDOM) vote_threshold(lvl_sets, N, K, lvl, thr, scan_lds, vstar, take_eq, exact_levels);
    if (votes_out) {
        // (past the caches: nothing of this step reads the copy.  Mask and gather 27.9 + 38.8 us -> 27.7 + 36.1 at 32 x
        // 25.6 M, 20.3 + 36.3 -> 19.7 + 34.5 at 10 x 11.2 M, K = 111,740; random selection's mask kernel 8.3 -> 7.4 at
        // 16 x 11.2 M)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int64_t j = j0 + q * kQuadStep;
            if (j + 16 <= d && ((reinterpret_cast<uintptr_t>(votes_out) & 15) == 0)) {
                __builtin_nontemporal_store(w[q], reinterpret_cast<u32x4*>(votes_out + j));
            } else {
                for (int b = 0; b < 16; ++b)
                    if (j + b < d) votes_out[j + b] = (uint8_t)((w[q][b >> 2] >> (8 * (b & 3))) & 255u);
            }
        }
    }
    if constexpr (RANDOM) {
        write_winners<Q>(winners, winners_per_block, d, K, scan_lds, mask_idx);
        return;
    }
    uint32_t marks[Q], in_stretch[Q];
    const uint32_t stretch = count_above_and_at<Q>(w, j0, d, vstar, marks, in_stretch);
    // (vote_threshold ended with a barrier, behind which nobody reads its scratch)
    if (lane == 0) scan_lds[wave] = pack2(stretch & 0xFFFFu, stretch >> 16);
    __syncthreads();
    uint64_t block_total, ex;                     // ex: before this wavefront's stretch, in the block
    {
        constexpr uint32_t kStretches = kMaskThreads / kWave;
        const uint64_t mine = lane < kStretches ? scan_lds[lane] : 0u;
        const uint32_t hi = row_incl_scan((uint32_t)(mine >> 32)), lo = row_incl_scan((uint32_t)mine);
        block_total = pack2(from_lane(hi, kStretches - 1), from_lane(lo, kStretches - 1));
        ex = wave ? pack2(from_lane(hi, wave - 1), from_lane(lo, wave - 1)) : 0u;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {    // the threshold, for the kernel that follows
        vote_thr[0] = vstar;
        vote_thr[1] = take_eq;
    }
    // The counts of the earlier blocks, without another kernel: every block publishes its own
    // totals at once (word 0 of its pair); its first wavefront then reads the totals of the
    // kLookBack blocks before it, all loads in flight together, and the sum over everything
    // up to the block before those (word 1 of that block's pair, published by that block once
    // it has summed up itself), polling until every word is there.  A word holds a "present"
    // bit and both counts (each below 2^31), so one 64-bit store publishes it whole.  Blocks
    // are dispatched in the order of their numbers and publish their totals before they wait,
    // so the wait ends; were a word still missing after spin_limit polls, the block gives up,
    // says so in emit_fail, and mv_gather_update finds the mask from the counts instead.
    constexpr unsigned long long kPresent = 1ull << 63, kCountMask = 0x7FFFFFFFull;
    constexpr int kPer = kLookBack / kWave;
    auto word_of = [&](uint64_t counts) { return kPresent | ((counts >> 32) << 31) | (counts & kCountMask); };
    auto counts_of = [&](unsigned long long w) {
        return pack2((uint32_t)((w >> 31) & kCountMask), (uint32_t)(w & kCountMask));
    };
    if (wave == 0) {
        const int64_t me = blockIdx.x;
        if (lane == 0)
            __hip_atomic_store(&lookback[2 * me], word_of(block_total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // lane l: the totals of blocks me - 1 - l - 64 r; lane 0 also the sum up to block me - kLookBack - 1
        const unsigned long long* src[kPer + 1];
        unsigned long long w[kPer + 1];
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int64_t b = me - 1 - (int64_t)lane - (int64_t)kWave * r;
            src[r] = b >= 0 ? &lookback[2 * b] : nullptr;
        }
        src[kPer] = (lane == 0 && me - kLookBack - 1 >= 0) ? &lookback[2 * (me - kLookBack - 1) + 1] : nullptr;
#pragma unroll
        for (int r = 0; r <= kPer; ++r) w[r] = src[r] ? 0ull : kPresent;
        bool found = true;
        for (uint32_t polls = 0;; ++polls) {
            bool all = true;
#pragma unroll
            for (int r = 0; r <= kPer; ++r)
                if (!(w[r] & kPresent)) w[r] = __hip_atomic_load(src[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int r = 0; r <= kPer; ++r) all = all && (w[r] & kPresent);
            if (__ballot(!all) == 0ull) break;
            if (polls >= spin_limit) {                                // uniform
                found = false;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        uint64_t before = 0;
#pragma unroll
        for (int r = 0; r <= kPer; ++r) before += counts_of(w[r]);
        before = wave_incl_scan64(before);
        before = pack2(from_lane((uint32_t)(before >> 32), kWave - 1), from_lane((uint32_t)before, kWave - 1));
        if (lane == 0) {
            if (found)
                __hip_atomic_store(&lookback[2 * me + 1], word_of(before + block_total), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            else
                __hip_atomic_store(emit_fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            before_sh = before;
            mask_found = found ? 1u : 0u;
        }
    }
    __syncthreads();
    // the counts per stretch and per block: what mv_gather_update scans when the mask could not be written here (behind
    // the exchange: the other blocks wait for what this one publishes, and nobody in this kernel for these)
    if (lane == 0) sub_cnt[(size_t)blockIdx.x * (kMaskThreads / kWave) + wave] = u32x2{stretch & 0xFFFFu, stretch >> 16};
    if (threadIdx.x == 0) block_cnt[blockIdx.x] = u32x2{(uint32_t)(block_total >> 32), (uint32_t)block_total};
    if (mask_found == 0u) return;                   // whole workgroup
    const uint64_t before = before_sh;
    if ((uint32_t)(before >> 32) + min((uint32_t)before, take_eq) >= K) return;   // the mask is full before this block
    each_mask_position<Q>(marks, in_stretch, j0, (uint32_t)((before + ex) >> 32), (uint32_t)(before + ex), take_eq,
                          [&](uint32_t pos, uint32_t j) {
                              if (pos < K) mask_idx[pos] = j;
                          });
}

// ----------------------------------------------------------------------------
// 6. masked gather, ordered sum over workers, mean, error update; the sorted vote lists that are not written
//    beside the mask kernel
// ----------------------------------------------------------------------------

// Positions [k0, k1) of the mask, whose coordinates are in slice[0 .. k1 - k0), at most `rounds` times
// kMaskThreads / N of them: thread (n, kl) reads a[n][j], stores +0.0 there, and parks the value in LDS;
// one thread per coordinate then adds the N values in worker order.  Neighbouring lanes have neighbouring
// positions of one row: masks crowd where gradients are large, so lanes share cache lines (10 x 11.2 M,
// K = 111,740: 48.6 -> 47.0 us).
constexpr int kGatherRounds = 4;                  // at most this many rounds of kb positions per workgroup

// The N values of a position lie together, positions an odd number of words apart: the threads that add them up,
// one per position, hit different banks.
constexpr uint32_t tile_pitch(uint32_t N) { return N | 1u; }
constexpr uint32_t kTileFloats = kMaskThreads + kMaskThreads / 2;     // two workers need the most
constexpr bool tile_holds_every_n()
{
    for (uint32_t N = 1; N <= 255; ++N)
        if ((kMaskThreads / N - 1) * tile_pitch(N) + N > kTileFloats) return false;
    return true;
}
static_assert(tile_holds_every_n(), "a round's values fit the tile for every number of workers");

__device__ __forceinline__ void gather_positions(float* tile /*LDS*/, const uint32_t* slice /*LDS*/,
                                                 float* __restrict__ e, int64_t ld_e, int64_t d, uint32_t N,
                                                 uint32_t k0, uint32_t k1, uint32_t rounds, float scale,
                                                 int apply_scale, float* __restrict__ agg)
{
    const uint32_t t = threadIdx.x, kb = kMaskThreads / N;
    const uint32_t n = t / kb, kl = t % kb;           // threads from N kb on have n >= N: idle
    const uint32_t pitch = tile_pitch(N);
    // a thread's loads of all rounds are in flight together
    float v[kGatherRounds];
#pragma unroll
    for (int r = 0; r < kGatherRounds; ++r) {
        const uint32_t k = k0 + (uint32_t)r * kb + kl;
        const uint32_t j = ((uint32_t)r < rounds && n < N && k < k1) ? slice[k - k0] : 0xFFFFFFFFu;
        v[r] = 0.0f;
        if ((int64_t)j < d) {                         // always true for a mask built above
            float* p = e + (int64_t)n * ld_e + j;
            v[r] = *p;
            *p = 0.0f;
        }
    }
#pragma unroll
    for (int r = 0; r < kGatherRounds; ++r) {
        if ((uint32_t)r >= rounds) break;             // uniform over the workgroup
        if (n < N) tile[kl * pitch + n] = v[r];
        __syncthreads();
        if (t < kb) {
            const uint32_t kk = k0 + (uint32_t)r * kb + t;
            if (kk < k1) {
                float s = tile[t * pitch];        // worker 0
                for (uint32_t m = 1; m < N; ++m) s = s + tile[t * pitch + m];
                agg[kk] = apply_scale ? s * scale : s;
            }
        }
        __syncthreads();
    }
}

// Workgroups [0, n_gather_blocks): each owns `rounds` times kb = 1024 / N consecutive positions of the mask.
// (a) Unless the mask is there (it is, but for a block that gave up waiting), the workgroup
//     first finds its own positions' coordinates: the counts per block of the vote bytes
//     and, inside the few blocks that matter, per wavefront stretch (from mv_mask_count)
//     are scanned, which says where in the mask each stretch's coordinates go; the few
//     stretches that reach into the workgroup's positions are read again, one wavefront each, and their coordinates above the
//     vote threshold, and the first take_eq at it, go to their positions -- in LDS for
//     the gather, and in mask_idx for the caller.  No kernel of its own emits the mask.
// (b) gather_positions reads a[n][mask[k]] (held in e), stores +0.0 there (the error
//     update: the residual of a transmitted coordinate is zero), adds the N values in
//     worker order 0..N-1 in fp32 and applies the 1/N of the mean once.
// Workgroups beyond write the sorted vote lists.
struct GatherLds {
    float    tile[kTileFloats];
    uint32_t slice[kGatherRounds * kMaskThreads];              // the workgroup's positions' coordinates
    uint32_t need[3 * (kMaskThreads + 2)];                     // stretches to read: (stretch, above before, at before)
    uint32_t blocks[3 * (kMaskThreads + 2)];                   // blocks whose stretches are looked at
    uint32_t n_need, n_blocks;
};

template <int Q>
__global__ __launch_bounds__(kMaskThreads) void mv_gather_update(float* __restrict__ e, int64_t ld_e,
                                                                 int64_t d, uint32_t N, uint32_t K,
                                                                 const uint32_t* __restrict__ votes32,
                                                                 const u32x2* __restrict__ sub_cnt,
                                                                 const u32x2* __restrict__ block_cnt, uint32_t n_blocks,
                                                                 const uint32_t* __restrict__ vote_thr,
                                                                 uint32_t* __restrict__ mask_idx, int mask_given,
                                                                 const uint32_t* __restrict__ emit_fail,
                                                                 float scale, int apply_scale,
                                                                 float* __restrict__ agg, uint32_t rounds,
                                                                 uint32_t n_gather_blocks, RowLists lists,
                                                                 uint32_t* __restrict__ step_no)
{
    __shared__ union { GatherLds gather; EmitLds emit; } shared;
    __shared__ uint64_t scan_lds[kMaskThreads / kWave];
    if (blockIdx.x >= n_gather_blocks) {
        write_row_lists(lists, blockIdx.x - n_gather_blocks, K, shared.emit, scan_lds);
        return;
    }
    GatherLds& lds = shared.gather;
    const uint32_t kb = kMaskThreads / N;             // N <= 255, so kb >= 4
    const uint32_t t = threadIdx.x, lane = lane_id(), wave = t / kWave;
    // This is the step's last kernel and nothing in it reads the step's number: the next step
    // gets the next number (kept on the device, so that a captured step can be replayed).
    if (blockIdx.x == 0 && t == 0) step_no[0] = step_no[0] + 1u;
    const uint32_t k0 = blockIdx.x * kb * rounds;     // the workgroup's positions: [k0, k1)
    const uint32_t k1 = min(K, k0 + kb * rounds);

    if (!mask_given && emit_fail[0] != 0u) {          // uniform over the grid; not expected
        const uint32_t vstar = vote_thr[0], take_eq = vote_thr[1];
        // one round of at most kb <= 1024 positions [q0, q1) at a time: that bounds the lists in LDS
        for (uint32_t r = 0; r < rounds; ++r) {
            const uint32_t q0 = k0 + r * kb, q1 = min(k1, q0 + kb);
            if (q0 >= q1) break;                          // uniform
            if (t == 0) {
                lds.n_need = 0;
                lds.n_blocks = 0;
            }
            // position of a stretch's (a block's) first mask coordinate = (coordinates above the threshold
            // before it) + min(coordinates at the threshold before it, take_eq)
            auto reaches_in = [&](uint32_t g, uint32_t q, u32x2 c) {
                const uint32_t q_taken = min(q, take_eq);                  // of the earlier ones at the threshold
                const uint32_t first = g + q_taken;
                const uint32_t n_in = c.x + min(c.y, take_eq - q_taken);
                return n_in != 0u && first < q1 && first + n_in > q0;
            };
            // first level: the blocks' totals
            uint32_t gt_before = 0, eq_before = 0;        // over the blocks of the earlier passes
            for (uint32_t b0 = 0; b0 < n_blocks; b0 += kMaskThreads) {
                const u32x2 none = {0u, 0u};
                const u32x2 c = b0 + t < n_blocks ? block_cnt[b0 + t] : none;
                uint64_t total;
                const uint64_t ex = block_excl_scan64<kMaskThreads>(pack2(c.x, c.y), scan_lds, total);
                const uint32_t g = gt_before + (uint32_t)(ex >> 32), q = eq_before + (uint32_t)ex;
                if (reaches_in(g, q, c)) {
                    const uint32_t at = atomicAdd(&lds.n_blocks, 1u);
                    lds.blocks[3 * at + 0] = b0 + t;
                    lds.blocks[3 * at + 1] = g;
                    lds.blocks[3 * at + 2] = q;
                }
                gt_before += (uint32_t)(total >> 32);
                eq_before += (uint32_t)total;
                __syncthreads();                          // the scan's scratch is reused by the next pass
                if (gt_before + min(eq_before, take_eq) >= q1) break;   // uniform: the rest lies behind these positions
            }
            __syncthreads();
            // second level: the stretches of those blocks (16 each), one wavefront per block
            constexpr uint32_t kSubs = kMaskThreads / kWave;
            const uint32_t n_blk = lds.n_blocks;
            for (uint32_t i = wave; i < n_blk; i += kSubs) {
                const uint32_t b = lds.blocks[3 * i];
                const u32x2 none = {0u, 0u};
                const u32x2 c = lane < kSubs ? sub_cnt[(size_t)b * kSubs + lane] : none;
                const uint64_t both = pack2(c.x, c.y);
                const uint64_t ex = wave_incl_scan64(both) - both;
                const uint32_t g = lds.blocks[3 * i + 1] + (uint32_t)(ex >> 32), q = lds.blocks[3 * i + 2] + (uint32_t)ex;
                if (lane < kSubs && reaches_in(g, q, c)) {
                    const uint32_t at = atomicAdd(&lds.n_need, 1u);
                    lds.need[3 * at + 0] = b * kSubs + lane;
                    lds.need[3 * at + 1] = g;
                    lds.need[3 * at + 2] = q;
                }
            }
            __syncthreads();
            // one wavefront per needed stretch
            const uint32_t n_need = lds.n_need;
            for (uint32_t i = wave; i < n_need; i += kSubs) {
                const uint32_t sidx = lds.need[3 * i];
                const int64_t j0 = (int64_t)sidx * (kQuadStep * Q) + lane * 16;
                u32x4 w[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int64_t j = j0 + q * kQuadStep;
                    const u32x4 z = {0u, 0u, 0u, 0u};
                    w[q] = (j < d) ? *reinterpret_cast<const u32x4*>(votes32 + (j >> 2)) : z;
                }
                uint32_t marks[Q], in_stretch[Q];
                (void)count_above_and_at<Q>(w, j0, d, vstar, marks, in_stretch);
                each_mask_position<Q>(marks, in_stretch, j0, lds.need[3 * i + 1], lds.need[3 * i + 2], take_eq,
                                      [&](uint32_t pos, uint32_t j) {
                                          if (pos >= q0 && pos < q1) {
                                              lds.slice[pos - k0] = j;
                                              mask_idx[pos] = j;
                                          }
                                      });
            }
            __syncthreads();                          // the lists are reused by the next round
        }
    } else {
        for (uint32_t k = k0 + t; k < k1; k += kMaskThreads) lds.slice[k - k0] = mask_idx[k];
    }
    __syncthreads();

    gather_positions(lds.tile, lds.slice, e, ld_e, d, N, k0, k1, rounds, scale, apply_scale, agg);
}

}  // namespace mvk
