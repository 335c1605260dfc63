// The votes of long lists (the rows' select went through mv_sel_hist, mv_sel_split and mv_sel_finish): counted in LDS
// by the workgroup that owns a coordinate, without an atomic in memory.
#pragma once

#include "mv_common.hpp"
#include "mv_select.hpp"

namespace mvk {

// A workgroup owns `per_wg` chunks of 2^chunk_shift coordinates, chunks gridDim.x apart: masks crowd in the few tensors
// with the largest gradients, and chunks dealt round give every workgroup its part of them.  (Handed stretches of
// coordinates in a row, one unit walked tens of thousands of entries while the others idled: 100 us and more.)  It
// finds its chunks' candidates of every row through the segments' runs, adds the votes of the taken ones up in LDS, and
// writes the vote bytes, the number of coordinates with exactly v votes for every v, and the segments' tallies for the
// sorted lists.  Rows are shifted against each other (RowSegments), so a chunk's last segment is usually shared with
// the next chunk: its entries are read by both, its tally is the next one's.
//
// Entries are dealt to threads by their number among all of the workgroup's, so that no thread has more than one more
// than another.  Which run an entry belongs to: the runs that are not empty are numbered, and a bit
// marks each entry that begins one, so the number is a count of bits, most of it a scalar's (found by bisection in the
// runs' summed lengths, with its place taken apart by divisions: 20.5 us instead of 15.2 at 10 x 11.2 M, K = 111,740).
// A batch of 4096 entries takes 3 us so, 2.3 of them finding the runs, and where the largest tensors' errors are zero
// the fullest workgroup has five.  So the runs of at least kLongRun entries go to a wavefront each, which has nothing
// to find: that workgroup is through with its entries in 7 us for 17.  10 x 11.2 M, K = 111,740, from a zero buffer
// 20.7 us for 25.7 (all of these between events around the kernel; runs from 64 entries on 20.6, but 15.8 for 13.4 at
// 16 x 6 M, K = 40,000; from 32 on 24.4), with carried errors 16.3 for 17.2.
// A chunk with kCrowdedEntries of them and more would hold the step up all the same.  order_runs lists such chunks, their
// owner leaves them out, and behind its own chunks every workgroup takes pieces of them, a segment's length each: all votes
// of 32 x 3 M, K = 30,000 in the same 30,000 coordinates 38 us for 77 (135 without long runs), steps 283 us for 319 (379;
// votes cast by atomics 259); all of 10 x 11.2 M, K = 111,740 in 111,740 305 for 311 (329; 306).  From 24,576 entries on 285
// and 309.  It costs the other steps 0.1 %, that from a zero buffer above 1.5 us.  Pieces as further units of the pass over
// the own chunks, or to workgroups of their own: 2 us more for everyone, who have to know the list before their first load.
//
// Of the kernel's time with carried errors 4.6 are the launch, 1.8 the runs, 6 the entries and 1.5 the bytes and their
// levels; at 32 x 25.6 M, 20.2 us by the trace, the runs are 7.  With workgroups of 1024 threads 26 there: four short
// ones to a unit fill each other's waits.
// With the votes as returning atomics in memory, cast by mv_sel_split and mv_sel_finish, these two took 37.5 and 45 us;
// with this kernel behind them the three take 28 and 39, and the vote bytes need not be cleared beforehand: steps
// 337.7 -> 322.5 us and 1413.7 -> 1406.4.  From a zero buffer, whose votes lie close together and share atomics,
// 307.3 -> 311.2.
constexpr int kVotesThreads = 512;
constexpr int kVotesWaves = kVotesThreads / kWave;
constexpr int kVotesRunsMost = 1024;              // runs of a workgroup: two to a thread
constexpr int kVotesBytesMost = 6 * 4096;         // coordinates of a workgroup
constexpr int kVotesUnroll = 8;                   // entries per thread in flight together
constexpr uint32_t kVotesBatch = kVotesThreads * kVotesUnroll;
static_assert(kVotesWaves * kVotesUnroll == kWave, "a lane per wavefront's part of a batch");
constexpr uint32_t kLongRun = 128;                // a run of so many entries is one wavefront's
constexpr int kLongUnroll = 4;                    // loads of it in flight together, twice
constexpr int kLvlCopies = 2;                     // copies of the level counters, one per lane % kLvlCopies

struct VotesLds {
    __attribute__((aligned(16))) uint32_t votes[kVotesBytesMost / 4];
    __attribute__((aligned(8))) uint32_t begins[kVotesBatch / 32];   // bit i: entry i of the batch begins a run
    uint32_t from[kVotesRunsMost];                // entry number i of the workgroup's, in run r: entry from[r] + i of the row's list
    uint16_t place[kVotesRunsMost];               // the run's row | the workgroup's chunk << 8
    uint32_t taken[kVotesRunsMost];               // (of a long run that is still to be walked: its length)
    uint32_t n_long;                              // long runs: they have the arrays' ends
    uint32_t lvl[kLvlCopies * 257];
    uint32_t kth[256], tie_cut[256];              // of the rows
    uint64_t scan[kVotesWaves];
    uint32_t any_slow;
    uint8_t  left_out[kVotesBytesMost >> 10];     // the workgroup's chunks that are crowded
};
static_assert(4 * sizeof(VotesLds) <= 160 * 1024, "four workgroups share a compute unit");
static_assert(2 * 255 <= kVotesThreads, "a thread for each of a piece's runs");
static_assert((kVotesBytesMost >> 10) <= 256, "a chunk's number fits a byte");

// x / divisor for x < 2048 and divisor <= 512 by m = ceil(2^20 / divisor): x m / 2^20 exceeds the quotient by less than
// 2048 / 2^20, which is at most 1 / divisor
struct SmallDivisor {
    uint32_t divisor, m;
    __device__ __forceinline__ explicit SmallDivisor(uint32_t by) : divisor(by), m(((1u << 20) + by - 1) / by) {}
    __device__ __forceinline__ uint32_t quotient(uint32_t x) const { return x * m >> 20; }
};

__global__ __launch_bounds__(kVotesThreads, 8) void mv_vote_count(
    const float* __restrict__ e, int64_t ld_e, int64_t d, uint32_t N, const u32x2* __restrict__ cand, uint32_t cap,
    const u32x2* __restrict__ runs, uint32_t n_runs, RowSegments segs, const uint32_t* __restrict__ kth_in,
    const uint32_t* __restrict__ tie_cut_in, const uint32_t* __restrict__ slow_flag, CrowdedChunks crowd,
    uint32_t per_wg, uint32_t* __restrict__ votes32, uint16_t* __restrict__ run_taken, uint32_t* __restrict__ lvl_sets)
{
    __shared__ VotesLds lds;
    const uint32_t t = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave);
    const uint32_t chunk_shift = crowd.chunk_shift, n_chunks = crowd.n_chunks, n_crowded = *crowd.n;
    const uint32_t chunk = 1u << chunk_shift, own = chunk / kSeg, slots = own + 1;      // segments of a chunk
    const uint32_t n = N * per_wg * slots;        // runs, row after row
    const SmallDivisor by_slots(slots), by_row(slots * per_wg);
    auto chunk_of = [&](uint32_t m) { return blockIdx.x + m * gridDim.x; };

    // the thread's two runs: of which row, which of the workgroup's chunks, which segment
    u32x2 run[2];
    uint32_t place[2], row_of[2], seg[2];
    bool tally[2];                                // written here: the chunk's own segments' and, behind the last chunk, one more's
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint32_t r = 2 * t + q, row = by_row.quotient(r), in_row = r - row * by_row.divisor, m = by_slots.quotient(in_row),
                       slot = in_row - m * by_slots.divisor, s = chunk_of(m) * own + slot;
        run[q] = u32x2{0u, 0u};
        row_of[q] = row;
        seg[q] = s;
        place[q] = row | m << 8;
        tally[q] = false;
        if (r < n && chunk_of(m) < n_chunks && s < segs.count(row) && (slot < own || segs.shift(row) != 0u)) {
            tally[q] = slot < own || chunk_of(m) == n_chunks - 1;
            run[q] = runs[(size_t)row * n_runs + s];                 // (in order: see order_runs)
            if (slow_flag[row] == 1u) run[q].y = 0;
            if (crowd.entries[chunk_of(m)] >= kCrowdedEntries) {     // not here, but in pieces
                run[q].y = 0;
                tally[q] = false;
            }
        }
    }
    if (t < per_wg) lds.left_out[t] = chunk_of(t) < n_chunks && crowd.entries[chunk_of(t)] >= kCrowdedEntries ? 1 : 0;
    uint32_t kth = 0, tie_cut = 0;
    bool slow = false;
    if (t < N) {
        kth = kth_in[t];
        tie_cut = tie_cut_in[t];
        slow = slow_flag[t] == 1u;
    }
    // cleared while those loads are under way
    if (t == 0) lds.any_slow = lds.n_long = 0;
    {
        const u32x4 z = {0u, 0u, 0u, 0u};
        u32x4* v = reinterpret_cast<u32x4*>(lds.votes);
        for (uint32_t i = t; i < (per_wg << chunk_shift) / 16; i += kVotesThreads) v[i] = z;
    }
    for (uint32_t i = t; i < kLvlCopies * 257; i += kVotesThreads) lds.lvl[i] = 0;
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();                              // (any_slow is cleared)
    if (t < N) {
        lds.kth[t] = kth;
        lds.tie_cut[t] = tie_cut;
        if (slow) lds.any_slow = 1u;
    }
    uint32_t number[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (run[q].y >= kLongRun) {
            number[q] = (uint32_t)kVotesRunsMost - 1u - atomicAdd(&lds.n_long, 1u);
            lds.from[number[q]] = run[q].x;
            lds.place[number[q]] = (uint16_t)place[q];
            lds.taken[number[q]] = run[q].y;
            run[q].y = kLongRun;
        }
    // the other runs' entries' numbers, and their own among those that are not empty
    uint32_t first[2], total;
    auto is_short = [&](int q) { return run[q].y - 1u < kLongRun - 1u; };
    {
        const uint32_t there[2] = {is_short(0) ? 1u : 0u, is_short(1) ? 1u : 0u}, there0 = is_short(0) ? run[0].y : 0u;
        uint64_t sums;
        const uint64_t ex = block_excl_scan64<kVotesThreads>(
            pack2(there0 + (is_short(1) ? run[1].y : 0u), there[0] + there[1]), lds.scan, sums);
        total = (uint32_t)(sums >> 32);
        first[0] = (uint32_t)(ex >> 32);
        first[1] = first[0] + there0;
        if (there[0]) number[0] = (uint32_t)ex;
        if (there[1]) number[1] = (uint32_t)ex + there[0];
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (is_short(q)) {
            lds.from[number[q]] = run[q].x - first[q];
            lds.place[number[q]] = (uint16_t)place[q];
            lds.taken[number[q]] = 0;
        }

    uint32_t runs_before = 0;                     // that begin before the batch
    for (uint32_t i0 = 0; i0 < total; i0 += kVotesBatch) {
        if (i0) __syncthreads();                  // the bits have been read
        if (t < kVotesBatch / 32) lds.begins[t] = 0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (is_short(q) && first[q] - i0 < kVotesBatch)
                atomicOr(&lds.begins[(first[q] - i0) / 32], 1u << ((first[q] - i0) & 31u));
        __syncthreads();
        const u32x2 bits = reinterpret_cast<const u32x2*>(lds.begins)[lane];       // lane l: of the batch's entries 64 l ..
        const uint32_t n_begin = (uint32_t)(__popc(bits.x) + __popc(bits.y)), incl = wave_incl_scan(n_begin);
        u32x2 c[kVotesUnroll];
        uint32_t r[kVotesUnroll], at[kVotesUnroll];
        uint64_t begins[kVotesUnroll];            // uniform
#pragma unroll
        for (int u = 0; u < kVotesUnroll; ++u) {
            c[u] = u32x2{0u, 0xFFFFFFFFu};
            const uint32_t b = (uint32_t)u * kVotesWaves + wave, i = i0 + b * kWave + lane;
            if (i0 + b * kWave >= total) continue;                   // uniform
            begins[u] = pack2(from_lane(bits.y, b), from_lane(bits.x, b));
            // the entry's run: the last that begins at or before it
            const uint32_t before = runs_before + from_lane(incl, b) - from_lane(n_begin, b) + ((uint32_t)begins[u] & 1u) - 1u;
            const uint64_t later = begins[u] >> 1;
            r[u] = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(later >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)later, 0u));
            at[u] = lds.place[r[u]];
            if (i < total) c[u] = cand[(size_t)(at[u] & 255u) * cap + (lds.from[r[u]] + i)];
        }
        runs_before += from_lane(incl, kWave - 1);
#pragma unroll
        for (int u = 0; u < kVotesUnroll; ++u) {
            if (i0 + ((uint32_t)u * kVotesWaves + wave) * kWave >= total) break;          // uniform
            const uint32_t row = at[u] & 255u, m = at[u] >> 8;
            const bool taken = c[u].y != 0xFFFFFFFFu && is_taken(c[u], lds.kth[row], lds.tie_cut[row]);
            const uint32_t j = c[u].y - (chunk_of(m) << chunk_shift);
            if (taken && j < chunk) atomicAdd(&lds.votes[((m << chunk_shift) + j) >> 2], 1u << (j & 3u) * 8u);
            if (run_taken) {
                // a run's taken ones among the wavefront's entries: those up to its last lane less those below its
                // first
                const uint64_t all = __ballot(taken);
                const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(all >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0u));
                const uint64_t begin = begins[u] | 1ull, end = begins[u] >> 1 | 1ull << 63;
                if (end >> lane & 1ull) atomicAdd(&lds.taken[r[u]], below + (taken ? 1u : 0u));
                if ((begin >> lane & 1ull) && below != 0u) atomicAdd(&lds.taken[r[u]], 0u - below);
            }
        }
    }
    // The long runs, a wavefront each; the next loads are under way while these are counted.
    auto walk_long_runs = [&](auto base_of, uint32_t length) {
        const uint32_t n_long = lds.n_long;
        if (wave >= n_long) return;               // uniform
        struct Run {
            const u32x2* entries;
            uint32_t n, place;
            u32x2 cut;                            // the row's K-th magnitude and tie cut
        };
        auto run_at = [&](uint32_t k) {
            const uint32_t at = (uint32_t)kVotesRunsMost - 1u - k;
            Run l;
            l.place = from_lane((uint32_t)lds.place[at], 0);
            l.n = from_lane(lds.taken[at], 0);
            l.entries = cand + ((size_t)(l.place & 255u) * cap + from_lane(lds.from[at], 0));
            l.cut = u32x2{lds.kth[l.place & 255u], lds.tie_cut[l.place & 255u]};
            return l;
        };
        auto load = [&](const Run& l, uint32_t i0, u32x2 (&c)[kLongUnroll]) {
#pragma unroll
            for (int u = 0; u < kLongUnroll; ++u) {
                const uint32_t i = i0 + (uint32_t)u * kWave + lane;
                c[u] = l.entries[min(i, l.n - 1u)];
            }
        };
        uint32_t k = wave, i0 = 0, n_taken = 0;
        Run l = run_at(k);
        u32x2 c[kLongUnroll];
        load(l, 0, c);
        while (true) {
            const bool ends = i0 + kLongUnroll * kWave >= l.n;       // uniform, as all that follows
            const uint32_t next_k = ends ? k + kVotesWaves : k, next_i0 = ends ? 0u : i0 + kLongUnroll * kWave;
            Run next = l;
            u32x2 ahead[kLongUnroll];
            if (next_k < n_long) {
                if (ends) next = run_at(next_k);
                load(next, next_i0, ahead);
            }
            const uint32_t m = l.place >> 8, base = base_of(m);
#pragma unroll
            for (int u = 0; u < kLongUnroll; ++u) {
                if (i0 + (uint32_t)u * kWave >= l.n) continue;
                const bool taken = i0 + (uint32_t)u * kWave + lane < l.n && is_taken(c[u], l.cut.x, l.cut.y);
                n_taken += (uint32_t)__popcll(__ballot(taken));
                const uint32_t j = c[u].y - base;
                if (taken && j < length) atomicAdd(&lds.votes[((m << chunk_shift) + j) >> 2], 1u << (j & 3u) * 8u);
            }
            if (ends) {
                if (lane == 0) lds.taken[(uint32_t)kVotesRunsMost - 1u - k] = n_taken;
                n_taken = 0;
            }
            if (next_k >= n_long) break;
            k = next_k;
            i0 = next_i0;
            l = next;
            for (int u = 0; u < kLongUnroll; ++u) c[u] = ahead[u];
        }
    };
    walk_long_runs([&](uint32_t m) { return chunk_of(m) << chunk_shift; }, chunk);    // (behind the scan's barrier)
    // the rows that were selected from memory are read again: `bytes` vote bytes, byte i's coordinate being at(i)
    auto read_slow_rows = [&](uint32_t bytes, auto at) {
        for (uint32_t row = 0; row < N; ++row) {
            if (slow_flag[row] != 1u) continue;
            for (uint32_t i = t; i < bytes; i += kVotesThreads) {
                const uint64_t j = at(i);
                if (j >= (uint64_t)d) continue;
                const u32x2 c = {__float_as_uint(e[(int64_t)row * ld_e + (int64_t)j]) & kAbsMask, (uint32_t)j};
                if (is_taken(c, lds.kth[row], lds.tie_cut[row])) atomicAdd(&lds.votes[i >> 2], 1u << (i & 3u) * 8u);
            }
        }
    };
    // the vote bytes, 16 at a time, and their levels
    auto write_votes = [&](uint32_t bytes, auto at, auto skip) {
        uint32_t* lvl = lds.lvl + (lane % kLvlCopies) * 257;
        const u32x4* v = reinterpret_cast<const u32x4*>(lds.votes);
        for (uint32_t i = t; i < bytes / 16; i += kVotesThreads) {
            const uint64_t j = at(i * 16);
            if (j >= (uint64_t)d || skip(i * 16)) continue;
            const u32x4 w = v[i];
            *reinterpret_cast<u32x4*>(votes32 + (j >> 2)) = w;       // zero from d on, up to a multiple of 16
            for (uint32_t x : {w.x, w.y, w.z, w.w})
                while (x != 0u) {
                    const uint32_t sh = (uint32_t)(__ffs((int)x) - 1) & 24u, b = x >> sh & 255u;
                    atomicAdd(&lvl[b], 1u);
                    x &= ~(255u << sh);
                }
        }
    };
    auto of_chunks = [&](uint32_t i) { return ((uint64_t)chunk_of(i >> chunk_shift) << chunk_shift) + (i & (chunk - 1)); };
    if (lds.any_slow) read_slow_rows(per_wg << chunk_shift, of_chunks);      // uniform
    __syncthreads();
    write_votes(per_wg << chunk_shift, of_chunks, [&](uint32_t i) { return lds.left_out[i >> chunk_shift] != 0; });
    if (run_taken)
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (tally[q]) run_taken[(size_t)row_of[q] * n_runs + seg[q]] = (uint16_t)(run[q].y != 0u ? lds.taken[number[q]] : 0u);
    // The crowded chunks' pieces, a segment's length each, are dealt round the grid; a thread has one of a piece's two
    // segments of a row, and all that are not empty are walked as long runs are.
    for (uint32_t p = blockIdx.x; p < n_crowded * own; p += gridDim.x) {     // uniform
        const uint32_t base = (crowd.list[p / own] << chunk_shift) + p % own * kSeg, row = t / 2, s = base / kSeg + t % 2;
        if (base >= (uint64_t)d) continue;
        u32x2 r = {0u, 0u};
        bool written_here = false;
        if (row < N && s < segs.count(row) && (t % 2 == 0 || segs.shift(row) != 0u)) {
            written_here = t % 2 == 0 || (uint64_t)base + kSeg >= (uint64_t)d;
            r = runs[(size_t)row * n_runs + s];
            if (slow_flag[row] == 1u) r.y = 0;
        }
        __syncthreads();                          // LDS is free again
        if (t == 0) lds.n_long = 0;
        if (t < kSeg / 16) reinterpret_cast<u32x4*>(lds.votes)[t] = u32x4{0u, 0u, 0u, 0u};
        __syncthreads();
        uint32_t at = 0;
        if (r.y != 0u) {
            at = (uint32_t)kVotesRunsMost - 1u - atomicAdd(&lds.n_long, 1u);
            lds.from[at] = r.x;
            lds.place[at] = (uint16_t)row;
            lds.taken[at] = r.y;
        }
        __syncthreads();
        walk_long_runs([&](uint32_t) { return base; }, (uint32_t)kSeg);
        auto of_piece = [&](uint32_t i) { return (uint64_t)base + i; };
        if (lds.any_slow) read_slow_rows(kSeg, of_piece);
        __syncthreads();
        write_votes(kSeg, of_piece, [](uint32_t) { return false; });
        if (run_taken && written_here)
            run_taken[(size_t)row * n_runs + s] = (uint16_t)(r.y != 0u ? lds.taken[at] : 0u);
    }
    __syncthreads();
    for (uint32_t b = t + 1; b < 256u; b += kVotesThreads) {
        uint32_t k = 0;
#pragma unroll
        for (int q = 0; q < kLvlCopies; ++q) k += lds.lvl[q * 257 + b];
        if (k) atomicAdd(&lvl_sets[(size_t)(blockIdx.x % kLvlSets) * 256 + b], k);
    }
}

}  // namespace mvk
