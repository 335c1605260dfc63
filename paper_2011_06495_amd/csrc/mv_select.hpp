// Exact selects: the K-th largest magnitude of a row's candidate list with its tie cut
// (one workgroup per row, or two kernels with many workgroups for long lists).
#pragma once

#include "mv_common.hpp"
#include "mv_stream.hpp"

namespace mvk {

// ----------------------------------------------------------------------------
// 3. per-row exact select
// ----------------------------------------------------------------------------

constexpr int kSelBins = 2048;   // radix-select digit: 11, 10, 10 bits of the 31-bit key
constexpr int kKeyBins = 4096;   // exact magnitudes inside one fine-histogram bin (1 << kFineShift)
constexpr int kRep     = 8;      // copies of the candidates' fine histogram, one per lane % kRep
constexpr int kTieCap  = 8192;   // ties with the K-th magnitude that fit the LDS list
constexpr int kRankCap = 256;    // at most this many entries are ranked by counting (quadratic work)
constexpr int kKeepMost = 32;    // list entries per thread of the largest instance of mv_row_select (8, 16, 32)

__device__ __forceinline__ int      sel_shift(int pass) { return pass == 0 ? 20 : pass == 1 ? 10 : 0; }
__device__ __forceinline__ uint32_t sel_dmask(int pass) { return pass == 0 ? 2047u : 1023u; }

// Adds one key's digit to the LDS histogram.  Must be called by all lanes of
// the wavefront together.  Gradient magnitudes share a few exponents, so most
// lanes hit the same digit in the first pass: one lane adds the whole group's
// count, the others add their own.
__device__ __forceinline__ void tally_digit(uint32_t* hist, bool active, uint32_t dg, uint32_t lane)
{
    const uint64_t am = __ballot(active);
    if (am != 0ull) {                                   // wave-uniform
        const int      leader = __ffsll((long long)am) - 1;
        const uint32_t ldg = __shfl(dg, leader, kWave);
        const uint64_t same = __ballot(active && dg == ldg);
        if (lane == (uint32_t)leader) atomicAdd(&hist[ldg], (uint32_t)__popcll(same));
        if (active && dg != ldg) atomicAdd(&hist[dg], 1u);
    }
}

// With a histogram of BINS bins complete (bins ordered like the keys): finds the
// bin that holds the `want`-th largest entry.  `bin` receives it, `want_in_bin`
// the rank inside the bin counted from its top (>= 1), `in_bin` the bin's count.
// Requires 1 <= want <= total count.  All kRowThreads threads must call it.
// With REP > 1 the histogram is kept in REP copies, each copy_pitch(BINS) words behind the one before.
constexpr int copy_pitch(int bins) { return bins + 8; }
template <int BINS, int REP = 1>
__device__ __forceinline__ void find_rank_bin(const uint32_t* hist, uint64_t* scan_lds, uint32_t* bcast,
                                              uint32_t want, uint32_t& bin, uint32_t& want_in_bin,
                                              uint32_t& in_bin)
{
    constexpr int per = BINS / kRowThreads;       // bins per thread, descending bin order over threads
    uint32_t h[per];
    uint32_t s = 0;
#pragma unroll
    for (int q = 0; q < per; ++q) {
        const int b = BINS - 1 - ((int)threadIdx.x * per + q);
        h[q] = 0;
#pragma unroll
        for (int r = 0; r < REP; ++r) h[q] += hist[r * copy_pitch(BINS) + b];
        s += h[q];
    }
    uint32_t total;
    const uint32_t ex = block_excl_scan<kRowThreads>(s, scan_lds, total);
    if (ex < want && want <= ex + s) {
        uint32_t acc = ex;
#pragma unroll
        for (int q = 0; q < per; ++q) {
            if (acc < want && want <= acc + h[q]) {
                bcast[0] = (uint32_t)(BINS - 1 - ((int)threadIdx.x * per + q));
                bcast[1] = want - acc;
                bcast[2] = h[q];
            }
            acc += h[q];
        }
    }
    __syncthreads();
    bin = bcast[0];
    want_in_bin = bcast[1];
    in_bin = bcast[2];
    __syncthreads();
}

// Keys of the selects below, re-read on every pass.  each(f) calls f(key, i, valid) the
// same number of times in every lane of the workgroup (so f may use wave-wide
// operations); i is the key's position, valid says whether it exists.
template <typename KeyAt>
struct KeysInMemory {
    KeyAt    key_at;
    uint64_t count;
    template <typename F>
    __device__ __forceinline__ void each(F f) const
    {
        for (uint64_t base = 0; base < count; base += (uint64_t)kRowThreads * 8) {
            uint32_t k[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint64_t i = base + (uint64_t)u * kRowThreads + threadIdx.x;
                k[u] = (i < count) ? key_at(i) : 0u;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint64_t i = base + (uint64_t)u * kRowThreads + threadIdx.x;
                f(k[u], i, i < count);
            }
        }
    }
};

// Exact K-th largest of the source's keys by an MSB-first radix select
// (11 + 10 + 10 bits) in one workgroup of kRowThreads threads.  Returns the K-th
// largest key; `take_eq` receives how many keys EQUAL to it belong to the top K
// (>= 1) and `n_eq` how many keys equal it in all.  Requires 1 <= K <= count.
template <typename Keys>
__device__ __forceinline__ uint32_t block_radix_select(const Keys& keys, uint32_t K, uint32_t* hist,
                                                       uint64_t* scan_lds, uint32_t* bcast,
                                                       uint32_t& take_eq, uint32_t& n_eq)
{
    const uint32_t lane = lane_id();
    uint32_t prefix = 0, known = 0, remaining = K, in_digit = 0;
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        for (int b = threadIdx.x; b < kSelBins; b += kRowThreads) hist[b] = 0;
        __syncthreads();
        keys.each([&](uint32_t k, uint64_t, bool valid) {
            tally_digit(hist, valid && ((k & known) == prefix), (k >> sel_shift(pass)) & sel_dmask(pass), lane);
        });
        __syncthreads();
        uint32_t digit;
        find_rank_bin<kSelBins>(hist, scan_lds, bcast, remaining, digit, remaining, in_digit);
        prefix |= digit << sel_shift(pass);
        known |= sel_dmask(pass) << sel_shift(pass);
    }
    take_eq = remaining;
    n_eq = in_digit;
    return prefix;
}

// Adds one vote for coordinate j.  Votes are bytes packed four to a word; N <= 255
// keeps a byte from carrying into its neighbour.  lvl[v] (LDS, 257 counters) counts
// coordinates that just reached v votes, so that, summed over all workgroups, lvl[v] =
// number of coordinates with at least v votes: the mask's vote threshold then follows
// from N + 1 numbers, and the passes over the vote bytes do work that does not depend
// on how the votes are spread.
__device__ __forceinline__ void cast_vote(uint32_t* __restrict__ votes32, uint32_t j, uint32_t* lvl)
{
    const uint32_t sh = (j & 3u) * 8u;
    const uint32_t old = atomicAdd(&votes32[j >> 2], 1u << sh);
    atomicAdd(&lvl[((old >> sh) & 255u) + 1u], 1u);
}

// The vote-level counters in memory: kLvlSets sets of 256 that the workgroups take turns
// over, so that their atomics do not queue up on one cache line.
constexpr int kLvlSets = 32;
__device__ __forceinline__ void merge_levels(const uint32_t* lvl, uint32_t* __restrict__ lvl_sets, uint32_t wg)
{
    for (uint32_t v = threadIdx.x; v < 256u; v += blockDim.x) {
        const uint32_t c = lvl[v];
        if (c) atomicAdd(&lvl_sets[(size_t)(wg % kLvlSets) * 256 + v], c);
    }
}

// One slot per lane with `want` set, consecutive within the wavefront: one LDS atomic
// per wavefront instead of one per entry.  All lanes of the wavefront must call it.
__device__ __forceinline__ uint32_t wave_slots(bool want, uint32_t* counter, uint32_t lane)
{
    const uint64_t m = __ballot(want);
    if (m == 0ull) return 0u;                              // wave-uniform
    const int leader = __ffsll((long long)m) - 1;
    uint32_t base = 0;
    if (lane == (uint32_t)leader) base = atomicAdd(counter, (uint32_t)__popcll(m));
    base = __shfl(base, leader, kWave);
    return base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
}

// f(key, count) by the first lane of every group of neighbouring lanes with equal keys, count being the
// group's lanes with `marked` set, if any.  All lanes of the wavefront must call it.
template <typename F>
__device__ __forceinline__ void tally_groups(uint32_t key, bool marked, F f)
{
    const uint32_t lane = lane_id();
    const uint32_t prev = __shfl_up(key, 1, kWave);
    const uint64_t heads = __ballot(lane == 0 || key != prev);
    const uint64_t tk = __ballot(marked);
    if (heads & (1ull << lane)) {
        const uint64_t above = (lane == kWave - 1) ? 0ull : (heads >> (lane + 1));
        const uint32_t len = above ? (uint32_t)__ffsll((long long)above) : (kWave - lane);
        const uint64_t span = (len >= 64 ? ~0ull : ((1ull << len) - 1)) << lane;
        const uint32_t n = (uint32_t)__popcll(tk & span);
        if (n) f(key, n);
    }
}

// A candidate (magnitude bits, coordinate) is in the row's top K iff its
// magnitude is above the K-th largest, or equals it and its coordinate is not
// beyond the last tie taken (ties go to the lowest coordinates).
__device__ __forceinline__ bool is_taken(u32x2 c, uint32_t kth, uint32_t tie_cut)
{
    return c.x > kth || (c.x == kth && c.y <= tie_cut);
}

// LDS of mv_row_select
struct SelectLds {
    __attribute__((aligned(16))) uint32_t hist[kKeyBins];   // histograms; then magnitudes of a bin's members
    __attribute__((aligned(16))) uint32_t ties[kTieCap];    // coordinates of a bin's members / of the ties
    __attribute__((aligned(16))) uint32_t rhist[copy_pitch(kFineBins) * kRep];   // the candidates' fine histogram, kRep copies
    uint32_t lvl[257];
    uint32_t bcast[3];
    uint32_t n_list;
    uint64_t scan[kRowThreads / kWave + 1];
};

__device__ __forceinline__ void clear_fine_histogram(SelectLds& lds)
{
    const u32x4 z = {0u, 0u, 0u, 0u};
    u32x4* rz = reinterpret_cast<u32x4*>(lds.rhist);
    for (int b = threadIdx.x; b < copy_pitch(kFineBins) * kRep / 4; b += kRowThreads) rz[b] = z;
}
// the lane's counter of a bin.  A bin's copies lie in different banks, eight words apart, and neighbouring bins of a
// copy in neighbouring words: the adds of a crowd do not queue up, nor the reads that sum the copies (with a bin's
// copies in neighbouring words every thread read 64 bytes in a row: 4 x 2^20, K = 10,486: 49.3 us, so 48.7).  The bins
// of a lattice lie far apart and meet in fewer banks so (16 x 11.2 M: 1.0 M conflict cycles for 0.5), in the same time.
__device__ __forceinline__ uint32_t* fine_counter(SelectLds& lds, uint32_t bin)
{
    return &lds.rhist[(lane_id() % kRep) * copy_pitch(kFineBins) + bin];
}

// The take-th SMALLEST of the n distinct coordinates in ties[0..n): ranked by
// counting when few; else narrowed by one histogram and then ranked by counting;
// a radix select on (0x7FFFFFFF - coordinate) if they crowd into one bin.
// (Lds: the scratch of the kernel at hand; ties has room for four more entries.)
template <typename Lds>
__device__ __forceinline__ uint32_t smallest_coordinate(Lds& lds, uint32_t* ties, uint32_t n, uint32_t take)
{
    if (n <= (uint32_t)kRankCap) {
        if (threadIdx.x < 4) ties[n + threadIdx.x] = 0xFFFFFFFFu;   // pad to a multiple of 4, ranked last
        __syncthreads();
        if (threadIdx.x < n) {
            const uint32_t mine = ties[threadIdx.x];
            const u32x4* tv = reinterpret_cast<const u32x4*>(ties);
            uint32_t below = 0;
#pragma unroll 4
            for (uint32_t j = 0; j < (n + 3) / 4; ++j) {
                const u32x4 o = tv[j];
                below += (o.x < mine) + (o.y < mine) + (o.z < mine) + (o.w < mine);
            }
            if (below == take - 1) lds.bcast[0] = mine;
        }
        __syncthreads();
        const uint32_t r = lds.bcast[0];
        __syncthreads();
        return r;
    }
    // Many ties: their coordinates are spread over the row, so one histogram of the
    // coordinate's leading bits (relative to the ties' own range) isolates a handful
    // around the wanted rank, which are then ranked by counting.
    const uint32_t t = threadIdx.x;
    if (t == 0) {
        lds.bcast[0] = 0u;
        lds.bcast[1] = 0xFFFFFFFFu;
    }
    for (int b = t; b < kSelBins; b += kRowThreads) lds.hist[b] = 0;
    __syncthreads();
    uint32_t mx = 0u, mn = 0xFFFFFFFFu;
    for (uint32_t i = t; i < n; i += kRowThreads) {
        const uint32_t c = ties[i];
        mx = max(mx, c);
        mn = min(mn, c);
    }
    for (int o = 1; o < kWave; o <<= 1) {
        mx = max(mx, (uint32_t)__shfl_xor(mx, o, kWave));
        mn = min(mn, (uint32_t)__shfl_xor(mn, o, kWave));
    }
    if (lane_id() == 0) {
        atomicMax(&lds.bcast[0], mx);
        atomicMin(&lds.bcast[1], mn);
    }
    __syncthreads();
    mx = lds.bcast[0];
    mn = lds.bcast[1];
    const uint32_t span = mx - mn;
    const uint32_t shift = span < (uint32_t)kSelBins ? 0u : (32u - (uint32_t)__clz(span)) - 11u;
    // bins ordered like the select's keys: the smallest coordinates in the highest bin
    for (uint32_t i = t; i < n; i += kRowThreads)
        atomicAdd(&lds.hist[(uint32_t)(kSelBins - 1) - ((ties[i] - mn) >> shift)], 1u);
    __syncthreads();                                  // also: everyone has read bcast
    uint32_t bin, want, in_bin;
    find_rank_bin<kSelBins>(lds.hist, lds.scan, lds.bcast, take, bin, want, in_bin);
    if (in_bin <= (uint32_t)kRowThreads) {            // uniform
        if (t == 0) lds.n_list = 0;
        __syncthreads();
        for (uint32_t i = t; i < n; i += kRowThreads) {
            const uint32_t c = ties[i];
            if ((uint32_t)(kSelBins - 1) - ((c - mn) >> shift) == bin) lds.hist[atomicAdd(&lds.n_list, 1u)] = c;
        }
        if (t < 4) lds.hist[in_bin + t] = 0xFFFFFFFFu;
        __syncthreads();
        if (t < in_bin) {
            const uint32_t mine = lds.hist[t];
            const u32x4* tv = reinterpret_cast<const u32x4*>(lds.hist);
            uint32_t below = 0;
#pragma unroll 4
            for (uint32_t j = 0; j < (in_bin + 3) / 4; ++j) {
                const u32x4 o = tv[j];
                below += (o.x < mine) + (o.y < mine) + (o.z < mine) + (o.w < mine);
            }
            if (below == want - 1) lds.bcast[0] = mine;
        }
        __syncthreads();
        const uint32_t r = lds.bcast[0];
        __syncthreads();
        return r;
    }
    uint32_t t_eq, n_eq;
    auto at = [ties](uint64_t i) { return kAbsMask - ties[i]; };
    const KeysInMemory<decltype(at)> src{at, n};
    return kAbsMask - block_radix_select(src, take, lds.hist, lds.scan, lds.bcast, t_eq, n_eq);
}

// Moves the members of fine-histogram bin `bin` into LDS: magnitude in lds.hist[p],
// coordinate in lds.ties[p], p = 0 .. in_bin-1 in no particular order.  The slots
// first receive the members' list positions; their coordinates are then fetched by
// all lanes together (one round trip, not one per member).  `in_bin` <= kKeyBins.
template <typename Keys>
__device__ __forceinline__ void collect_bin_members(const Keys& keys, const u32x2* __restrict__ crow, uint32_t tau,
                                                    uint32_t bin, uint32_t in_bin, SelectLds& lds)
{
    const uint32_t lane = lane_id(), t = threadIdx.x;
    keys.each([&](uint32_t k, uint64_t i, bool valid) {
        const bool mine = valid && fine_bin(k, tau) == bin;
        const uint32_t p = wave_slots(mine, &lds.n_list, lane);
        if (mine) {
            lds.hist[p] = k;
            lds.ties[p] = (uint32_t)i;
        }
    });
    __syncthreads();
    for (uint32_t p = t; p < in_bin; p += kRowThreads) lds.ties[p] = crow[lds.ties[p]].y;
    __syncthreads();
}

// K-th largest magnitude of a row's candidate list and the tie cut.  `keys`
// delivers the candidates' magnitudes (position i = position in the list crow).
// Returns through kth / tie_cut; `path` = 0 when the fine histogram sufficed,
// 2 when the radix select over all candidates had to run.
template <typename Keys>
__device__ __forceinline__ void select_among_candidates(const Keys& keys, const u32x2* __restrict__ crow,
                                                        uint32_t C, uint32_t K, uint32_t tau, SelectLds& lds,
                                                        uint32_t& kth, uint32_t& tie_cut, uint32_t& path)
{
    const uint32_t lane = lane_id(), t = threadIdx.x;
    uint32_t take_eq = 0, n_eq = 0;
    bool have_kth = false;
    path = 0;
    if (t == 0) lds.n_list = 0;                   // ordered by the first barrier below
    if (tau != 0) {
        // All candidates are >= tau and most lie within an octave of it: one
        // histogram of (key - tau) in 2048 bins finds the bin of the K-th largest.
        // Values on a lattice put thousands of candidates on a few dozen keys, and LDS
        // atomics of one instruction that meet on one address are served one after the
        // other: lane l adds to copy l % kRep of the histogram, which divides those queues.
        clear_fine_histogram(lds);
        __syncthreads();
        keys.each([&](uint32_t k, uint64_t, bool valid) {
            if (valid) atomicAdd(fine_counter(lds, fine_bin(k, tau)), 1u);
        });
        __syncthreads();
        uint32_t bin, want, in_bin;
        find_rank_bin<kFineBins, kRep>(lds.rhist, lds.scan, lds.bcast, K, bin, want, in_bin);
        if (in_bin <= (uint32_t)kRankCap) {       // uniform
            // few candidates in that bin: rank them by brute force under (magnitude desc,
            // coordinate asc); the one with exactly want-1 others ahead is the last of the top K
            collect_bin_members(keys, crow, tau, bin, in_bin, lds);
            if (t < 4) {                          // pad to a multiple of 4 with entries ranked last
                lds.hist[in_bin + t] = 0;
                lds.ties[in_bin + t] = 0xFFFFFFFFu;
            }
            __syncthreads();
            if (t < in_bin) {
                const uint32_t mk = lds.hist[t], mi = lds.ties[t];
                const u32x4* hk = reinterpret_cast<const u32x4*>(lds.hist);
                const u32x4* hi = reinterpret_cast<const u32x4*>(lds.ties);
                uint32_t ahead = 0;
#pragma unroll 4
                for (uint32_t j = 0; j < (in_bin + 3) / 4; ++j) {
                    const u32x4 ok = hk[j], oi = hi[j];
                    ahead += (ok.x > mk) || (ok.x == mk && oi.x < mi);
                    ahead += (ok.y > mk) || (ok.y == mk && oi.y < mi);
                    ahead += (ok.z > mk) || (ok.z == mk && oi.z < mi);
                    ahead += (ok.w > mk) || (ok.w == mk && oi.w < mi);
                }
                if (ahead == want - 1) {
                    lds.bcast[0] = mk;
                    lds.bcast[1] = mi;
                }
            }
            __syncthreads();
            kth = lds.bcast[0];
            tie_cut = lds.bcast[1];
            return;
        }
        if (bin < (uint32_t)(kFineBins - 1)) {
            // a crowded bin (many equal magnitudes): it spans exactly 4096 key values,
            // so a second histogram over the exact keys inside it finds the K-th largest
            const uint32_t bin_lo = tau + (bin << kFineShift);
            for (int b = t; b < kKeyBins; b += kRowThreads) lds.hist[b] = 0;
            __syncthreads();
            keys.each([&](uint32_t k, uint64_t, bool valid) {
                tally_digit(lds.hist, valid && fine_bin(k, tau) == bin, (k - bin_lo) & (uint32_t)(kKeyBins - 1), lane);
            });
            __syncthreads();
            uint32_t sub;
            find_rank_bin<kKeyBins>(lds.hist, lds.scan, lds.bcast, want, sub, take_eq, n_eq);
            kth = bin_lo + sub;
            have_kth = true;
        }
    }
    if (!have_kth) {
        path = 2;
        kth = block_radix_select(keys, K, lds.hist, lds.scan, lds.bcast, take_eq, n_eq);
    }
    // ties with the K-th magnitude: all taken, or only the take_eq lowest coordinates
    tie_cut = 0xFFFFFFFFu;
    if (take_eq < n_eq) {                         // uniform
        if (n_eq <= (uint32_t)kTieCap) {
            keys.each([&](uint32_t k, uint64_t i, bool valid) {
                const bool mine = valid && k == kth;
                const uint32_t p = wave_slots(mine, &lds.n_list, lane);
                if (mine) lds.ties[p] = (uint32_t)i;
            });
            __syncthreads();
            for (uint32_t p = t; p < n_eq; p += kRowThreads) lds.ties[p] = crow[lds.ties[p]].y;
            __syncthreads();
            tie_cut = smallest_coordinate(lds, lds.ties, n_eq, take_eq);
        } else {
            // more ties than the LDS list holds: select over the whole candidate list in
            // memory, entries that are not ties mapped below every tie
            uint32_t t_eq, t_n;
            auto at = [crow, kth](uint64_t i) {
                const u32x2 c = crow[i];
                return c.x == kth ? kAbsMask - c.y : 0u;
            };
            const KeysInMemory<decltype(at)> src{at, C};
            tie_cut = kAbsMask - block_radix_select(src, take_eq, lds.hist, lds.scan, lds.bcast, t_eq, t_n);
        }
    }
}

// Casts votes for the marked ones of a batch of list entries, U per thread (bit u of `taken`: c[u]): each
// adds one to its coordinate's vote byte and, when the sorted vote lists are wanted, is
// tallied in its segment (the tallies were zeroed by the streaming pass).  Lanes of a wavefront
// mostly hold consecutive list entries, which share a segment: the first lane of each
// group of equal segments adds the group's count.  All threads of the workgroup must call it.
template <int U, bool MERGE>
__device__ __forceinline__ void cast_votes(const u32x2 (&c)[U], uint32_t taken_mask, uint32_t* __restrict__ votes32,
                                           uint32_t* lvl, SegmentTallies tallies)
{
    const uint32_t lane = lane_id();
    // MERGE (long lists, where the atomics' rate at the memory side is what the step waits for): lanes
    // hold consecutive list entries, ascending inside a run, and a row votes at most once per
    // coordinate, so neighbouring taken lanes whose coordinates share a vote word (four bytes) cast
    // their votes with ONE atomic, the sum of their byte increments, issued by the first of them;
    // the returned word holds every byte's count before this row's vote.  Where the mask is dense
    // that is up to four votes per atomic (measured at K = d/100: 27 -> 19 us).  Short lists
    // wait for latency, not rate: there every taken lane issues its own.
    uint32_t old[U];
    uint32_t ahead[U];                            // lanes between this lane and the first of its group
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool taken = (taken_mask >> u) & 1u;
        const uint32_t inc = taken ? 1u << ((c[u].y & 3u) * 8u) : 0u;
        uint32_t before = 0;                      // lanes of the same group just below this one
        uint32_t sum = inc;
        if (MERGE) {
            const uint32_t key = taken ? (c[u].y >> 2) : (0xFFFFFF00u | lane);   // never equal to a neighbour's
            bool run = true;
#pragma unroll
            for (int k = 1; k < 4; ++k) {
                const uint32_t below = __shfl_up(key, k, kWave);
                run = run && lane >= (uint32_t)k && below == key;
                before += run ? 1u : 0u;
            }
            run = true;
#pragma unroll
            for (int k = 1; k < 4; ++k) {
                const uint32_t above_key = __shfl_down(key, k, kWave);
                const uint32_t above_inc = __shfl_down(inc, k, kWave);
                run = run && lane + (uint32_t)k < (uint32_t)kWave && above_key == key;
                sum += run ? above_inc : 0u;
            }
        }
        ahead[u] = before;
        old[u] = 0;
        if (taken && before == 0u) old[u] = atomicAdd(&votes32[c[u].y >> 2], sum);
    }
    if (MERGE) {
#pragma unroll
        for (int u = 0; u < U; ++u) old[u] = __shfl(old[u], lane - ahead[u], kWave);   // the group's returned word
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool taken = (taken_mask >> u) & 1u;
        if (taken) atomicAdd(&lvl[((old[u] >> ((c[u].y & 3u) * 8u)) & 255u) + 1u], 1u);
        if (tallies.taken)
            tally_groups(segment_of(c[u].y, tallies.shift), taken, [&](uint32_t s, uint32_t n) { tallies.add(s, n); });
    }
}

// The votes of the list entries i with (i / kRowThreads) % parts == part, those that are taken.
__device__ __forceinline__ void cast_votes_of_share(const u32x2* __restrict__ crow, uint32_t C, uint32_t kth,
                                                    uint32_t tie_cut, uint32_t part, uint32_t parts,
                                                    uint32_t* __restrict__ votes32, uint32_t* lvl,
                                                    SegmentTallies tallies)
{
    // all the loads, then all the vote atomics, then what depends on their results: a thread's
    // entries wait for memory together, not one after the other
    constexpr int kU = 8;                         // list entries per thread in flight together
    for (uint64_t q0 = part; q0 * kRowThreads < C; q0 += (uint64_t)parts * kU) {
        u32x2 c[kU];
        uint32_t taken = 0;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t i = (q0 + (uint64_t)u * parts) * kRowThreads + threadIdx.x;
            const u32x2 none = {0u, 0xFFFFFFFFu};
            c[u] = (i < C) ? crow[i] : none;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
            taken |= (c[u].y != 0xFFFFFFFFu && is_taken(c[u], kth, tie_cut) ? 1u : 0u) << u;
        cast_votes<kU, false>(c, taken, votes32, lvl, tallies);
    }
}

// ---- the rows' select from registers ------------------------------------------
// A thread keeps its list entries from the first load to the votes; entry number q of
// thread t is at q * kRowThreads + t of the list.  That is two round trips less than
// reading the members of the K-th's bin and the entries to vote for again -- while the
// unrolled code stays short: every launch fetches it anew.  So there are instances for 8
// and 16 entries, the votes from registers only in the first (7 x 272,475, K = 2725:
// 38.0 us with one instance for 32, 34.5 so), and beyond 16 a thread keeps only the
// number of each entry's bin (16 bits, two to a register; 0xFFFF: no entry), which is
// all the histogram pass and the search for the bin's members need (with whole entries
// 4 x 2^20, K = 10,486 took 50.7 us instead of 48.8; left to mv_sel_split, 50.1).
template <int KEEP>
struct KeptEntries {
    static constexpr bool kWhole = true;
    u32x2 entry[KEEP];
    // f(bin, q) for every entry slot below `count`, the same number of times in every lane of the workgroup;
    // bin = 0xFFFF: no entry
    template <typename F>
    __device__ __forceinline__ void each(uint32_t count, uint32_t tau, F f) const
    {
#pragma unroll
        for (int q = 0; q < KEEP; ++q)
            if ((uint32_t)q * kRowThreads < count)                   // uniform over the workgroup
                f((uint32_t)q * kRowThreads + threadIdx.x < count ? fine_bin(entry[q].x, tau) : 0xFFFFu, q);
    }
};
template <int KEEP>
struct KeptBins {
    static constexpr bool kWhole = false;
    uint32_t b[KEEP / 2];
    __device__ __forceinline__ void set(int q, uint32_t bin)
    {
        if (q & 1) b[q / 2] = (b[q / 2] & 0x0000FFFFu) | (bin << 16);
        else       b[q / 2] = bin;
    }
    template <typename F>
    __device__ __forceinline__ void each(uint32_t count, uint32_t, F f) const
    {
#pragma unroll
        for (int q = 0; q < KEEP; ++q)
            if ((uint32_t)q * kRowThreads < count)                   // uniform over the workgroup
                f((q & 1) ? (b[q / 2] >> 16) : (b[q / 2] & 0xFFFFu), q);
    }
};

// Exact K-th largest magnitude and tie cut of a candidate list that is kept in registers.  Returns false
// when the bin of the K-th largest holds more members than the LDS lists take (the caller then runs the generic
// select).
// LDS use: rhist holds the histogram, then (words [0, 4096)) the members' magnitudes,
// ([4096, 8192)) their coordinates, ([8192, 12288)) the histogram of their exact keys.
template <typename Kept>
__device__ __forceinline__ bool select_from_registers(const Kept& kept, const u32x2* __restrict__ crow, uint32_t C,
                                                      uint32_t K, uint32_t tau, SelectLds& lds, uint32_t& kth,
                                                      uint32_t& tie_cut)
{
    static_assert(kFineBins * kRep >= 3 * kKeyBins, "the members' lists reuse the histogram's storage");
    const uint32_t lane = lane_id(), t = threadIdx.x;
    // (the caller has zeroed lds.rhist and lds.n_list, and a barrier has passed since)
    // Values on a lattice put thousands of candidates on a few dozen keys, and LDS
    // atomics of one instruction that meet on one address are served one after the
    // other: lane l adds to copy l % kRep of the histogram, which divides those queues.
    kept.each(C, tau, [&](uint32_t bin, int) {
        if (bin != 0xFFFFu) atomicAdd(fine_counter(lds, bin), 1u);
    });
    __syncthreads();
    uint32_t bin, want, in_bin;
    find_rank_bin<kFineBins, kRep>(lds.rhist, lds.scan, lds.bcast, K, bin, want, in_bin);
    if (in_bin > (uint32_t)kKeyBins) return false;                  // uniform
    // the last bin is open-ended: its members' keys do not fit the exact-key histogram
    if (in_bin > (uint32_t)kRankCap && bin == (uint32_t)(kFineBins - 1)) return false;

    uint32_t* mkey = lds.rhist;                   // find_rank_bin ended with a barrier: the histogram is free
    uint32_t* mpos = lds.rhist + kKeyBins;
    {
        // the members, in no particular order: a wavefront takes room for its own with one atomic, and nobody waits
        uint32_t mine = 0;
        kept.each(C, tau, [&](uint32_t b, int) { mine += (b == bin); });
        uint32_t p = 0;
        if (__ballot(mine != 0u) != 0ull) {       // wave-uniform
            const uint32_t incl = wave_incl_scan(mine);
            if (lane == kWave - 1) p = atomicAdd(&lds.n_list, incl);
            p = from_lane(p, kWave - 1) + incl - mine;
        }
        if (mine)
            kept.each(C, tau, [&](uint32_t b, int q) {
                if (b == bin) {
                    if constexpr (Kept::kWhole) {
                        mkey[p] = kept.entry[q].x;
                        mpos[p++] = kept.entry[q].y;
                    } else {
                        mpos[p++] = (uint32_t)q * kRowThreads + t;   // for now its place in the list
                    }
                }
            });
    }
    __syncthreads();
    if constexpr (!Kept::kWhole) {
        for (uint32_t p = t; p < in_bin; p += kRowThreads) {         // all lanes together: one round trip
            const u32x2 c = crow[mpos[p]];
            mkey[p] = c.x;
            mpos[p] = c.y;
        }
        __syncthreads();
    }
    if (in_bin <= (uint32_t)kRankCap) {           // uniform
        // few members: ranked by counting under (magnitude desc, coordinate asc);
        // the one with exactly want-1 others ahead is the last of the top K
        if (t < 4) {                              // pad to a multiple of 4 with entries ranked last
            mkey[in_bin + t] = 0;
            mpos[in_bin + t] = 0xFFFFFFFFu;
        }
        __syncthreads();
        if (t < in_bin) {
            const uint32_t mk = mkey[t], mi = mpos[t];
            const u32x4* hk = reinterpret_cast<const u32x4*>(mkey);
            const u32x4* hi = reinterpret_cast<const u32x4*>(mpos);
            uint32_t ahead = 0;
#pragma unroll 4
            for (uint32_t j = 0; j < (in_bin + 3) / 4; ++j) {
                const u32x4 ok = hk[j], oi = hi[j];
                ahead += (ok.x > mk) || (ok.x == mk && oi.x < mi);
                ahead += (ok.y > mk) || (ok.y == mk && oi.y < mi);
                ahead += (ok.z > mk) || (ok.z == mk && oi.z < mi);
                ahead += (ok.w > mk) || (ok.w == mk && oi.w < mi);
            }
            if (ahead == want - 1) {
                lds.bcast[0] = mk;
                lds.bcast[1] = mi;
            }
        }
        __syncthreads();
        kth = lds.bcast[0];
        tie_cut = lds.bcast[1];
        __syncthreads();
        return true;
    }
    // Values on a lattice put hundreds of EQUAL magnitudes there: if all members share one
    // key, that key is the K-th largest and only the tie cut is left to find.
    if (t == 0) lds.bcast[2] = 0;
    __syncthreads();
    {
        bool differs = false;
        const uint32_t k0 = mkey[0];
        for (uint32_t p = t; p < in_bin; p += kRowThreads) {
            differs |= mkey[p] != k0;
            lds.ties[p] = mpos[p];                // in_bin <= kKeyBins <= kTieCap
        }
        if (differs) lds.bcast[2] = 1;
    }
    __syncthreads();
    if (lds.bcast[2] == 0) {                      // uniform
        kth = mkey[0];
        __syncthreads();                          // everyone has read bcast and mkey
        tie_cut = want < in_bin ? smallest_coordinate(lds, lds.ties, in_bin, want) : 0xFFFFFFFFu;
        return true;
    }
    // up to 4096 members: the bin spans exactly 4096 key values, so a histogram over the
    // members' exact keys finds the K-th largest, and its ties' coordinates are in LDS
    uint32_t* h2 = lds.rhist + 2 * kKeyBins;
    const uint32_t bin_lo = tau + (bin << kFineShift);
    for (int b = t; b < kKeyBins; b += kRowThreads) h2[b] = 0;
    __syncthreads();
    for (uint32_t p0 = 0; p0 < in_bin; p0 += kRowThreads) {          // wave-wide grouping: many keys are equal
        const uint32_t p = p0 + t;
        tally_digit(h2, p < in_bin, p < in_bin ? (mkey[p] - bin_lo) & (uint32_t)(kKeyBins - 1) : 0u, lane);
    }
    __syncthreads();
    uint32_t sub, take_eq, n_eq;
    find_rank_bin<kKeyBins>(h2, lds.scan, lds.bcast, want, sub, take_eq, n_eq);
    kth = bin_lo + sub;
    tie_cut = 0xFFFFFFFFu;
    if (take_eq < n_eq) {                         // uniform: only the take_eq lowest coordinates of the ties
        if (t == 0) lds.n_list = 0;
        __syncthreads();
        for (uint32_t p0 = 0; p0 < in_bin; p0 += kRowThreads) {
            const uint32_t p = p0 + t;
            const bool mine = p < in_bin && mkey[p] == kth;
            const uint32_t s = wave_slots(mine, &lds.n_list, lane);
            if (mine) lds.ties[s] = mpos[p];
        }
        __syncthreads();
        tie_cut = smallest_coordinate(lds, lds.ties, n_eq, take_eq);
    }
    return true;
}

// The votes of the entries q with q % parts == part, those that are taken: all the atomics, then what depends on
// their results (see cast_votes).
template <int KEEP>
__device__ __forceinline__ void cast_votes_from_registers(u32x2 (&entry)[KEEP], uint32_t C, uint32_t kth, uint32_t tie_cut,
                                                          uint32_t part, uint32_t parts, uint32_t* __restrict__ votes32,
                                                          uint32_t* lvl, SegmentTallies tallies)
{
    uint32_t taken = 0;
    uint32_t next = part;                         // the workgroup's next q
#pragma unroll
    for (int q = 0; q < KEEP; ++q)
        if ((uint32_t)q == next && (uint32_t)q * kRowThreads < C) {                // uniform
            next += parts;
            if ((uint32_t)q * kRowThreads + threadIdx.x < C && is_taken(entry[q], kth, tie_cut)) {
                taken |= 1u << q;
                entry[q].x = atomicAdd(&votes32[entry[q].y >> 2], 1u << ((entry[q].y & 3u) * 8u));   // key done with
            }
        }
    next = part;
#pragma unroll
    for (int q = 0; q < KEEP; ++q)
        if ((uint32_t)q == next && (uint32_t)q * kRowThreads < C) {                // uniform
            next += parts;
            const bool mine = taken >> q & 1u;
            if (mine) atomicAdd(&lvl[((entry[q].x >> ((entry[q].y & 3u) * 8u)) & 255u) + 1u], 1u);
            if (tallies.taken)
                tally_groups((uint32_t)q * kRowThreads + threadIdx.x < C ? segment_of(entry[q].y, tallies.shift) : 0xFFFFFFFFu,
                             mine, [&](uint32_t s, uint32_t n) { tallies.add(s, n); });
        }
}

// Exact select of a whole row from memory by one workgroup: the K-th largest magnitude by a radix select and the tie
// cut, the row's vote in ascending order (out, may be null) and its votes (votes32, may be null: they are not cast
// here).  (Lds: the scratch of the kernel at hand.)
template <typename Lds>
__device__ __forceinline__ void select_row_from_memory(Lds& lds, const float* __restrict__ arow, int64_t d, uint32_t K,
                                                       uint32_t* __restrict__ out, uint32_t* __restrict__ votes32,
                                                       uint32_t* __restrict__ lvl_sets, uint32_t* __restrict__ kth_out,
                                                       uint32_t* __restrict__ tie_cut_out)
{
    const uint32_t t = threadIdx.x;
    for (int i = t; i < 257; i += kRowThreads) lds.lvl[i] = 0;   // ordered by the select's first barrier
    uint32_t take_eq, n_eq;
    auto at = [arow](uint64_t i) { return __float_as_uint(arow[i]) & kAbsMask; };
    const KeysInMemory<decltype(at)> src{at, (uint64_t)d};
    const uint32_t kth = block_radix_select(src, K, lds.hist, lds.scan, lds.bcast, take_eq, n_eq);
    if (t == 0) *kth_out = kth;
    if (!out && !votes32) {
        // only the membership test is needed: the tie cut is the take_eq-th
        // smallest coordinate among the row's ties, selected from memory
        uint32_t tie_cut = 0xFFFFFFFFu;
        if (take_eq < n_eq) {
            uint32_t t_eq, t_n;
            auto tie_at = [arow, kth](uint64_t i) {
                return (__float_as_uint(arow[i]) & kAbsMask) == kth ? kAbsMask - (uint32_t)i : 0u;
            };
            const KeysInMemory<decltype(tie_at)> ties_src{tie_at, (uint64_t)d};
            tie_cut = kAbsMask - block_radix_select(ties_src, take_eq, lds.hist, lds.scan, lds.bcast, t_eq, t_n);
        }
        if (t == 0) *tie_cut_out = tie_cut;
        return;
    }
    uint32_t gt_before = 0, eq_before = 0;
    for (int64_t j0 = 0; j0 < d; j0 += (int64_t)kRowThreads * 4) {
        const int64_t j = j0 + (int64_t)t * 4;
        uint32_t kk[4];
        uint32_t gt = 0, eq = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool valid = (j + c < d);
            kk[c] = valid ? (__float_as_uint(arow[j + c]) & kAbsMask) : 0u;
            gt += (valid && kk[c] > kth);
            eq += (valid && kk[c] == kth);
        }
        uint64_t total;
        const uint64_t ex = block_excl_scan64<kRowThreads>(pack2(gt, eq), lds.scan, total);
        uint32_t g0 = gt_before + (uint32_t)(ex >> 32), e0 = eq_before + (uint32_t)ex;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (j + c < d) {
                const bool is_gt = kk[c] > kth, is_eq = kk[c] == kth;
                if (is_gt || (is_eq && e0 < take_eq)) {
                    const uint32_t pos = g0 + min(e0, take_eq);
                    if (out && pos < K) out[pos] = (uint32_t)(j + c);
                    if (votes32) cast_vote(votes32, (uint32_t)(j + c), lds.lvl);
                    if (is_eq && e0 == take_eq - 1) *tie_cut_out = (uint32_t)(j + c);       // the last tie taken
                }
                g0 += is_gt;
                e0 += is_eq;
            }
        }
        gt_before += (uint32_t)(total >> 32);
        eq_before += (uint32_t)total;
        __syncthreads();   // lds.scan is reused by the next round
    }
    if (votes32) merge_levels(lds.lvl, lvl_sets, blockIdx.x);
}

// parts workgroups per row; the grid is one-dimensional and workgroup ids are laid
// out so that the workgroups of one row have equal id % 8: consecutive ids go to
// different XCDs (each with an L2 of its own), so a row's list is then read from
// memory once and served to the row's other workgroups from that L2.
// Usual case: EVERY workgroup of a row runs the same exact select over the row's
// candidate list (the work is repeated rather than shared so that no workgroup
// waits for another): the K-th largest magnitude kth[row] and tie_cut[row], the
// largest coordinate taken among the candidates tied with it (0xFFFFFFFF: all ties
// taken).  Each workgroup then casts the votes of its share of the list.  With
// thresholds_only (add-drop voting) no vote is cast.  Longer lists go through
// mv_sel_hist, mv_sel_split and mv_sel_finish.
// If the candidate count is < K or overflowed the list (for instance a row of
// equal magnitudes), the row's first workgroup selects it exactly from memory (e
// already holds a = g + e), emits and casts its vote; slow_flag[row] = 1 tells the
// later kernels to skip the row.
// n_spec (<= KEEP): how many of a thread's list entries are fetched before the
// row's count is known (the list's storage holds cap entries; what lies at or
// beyond the count is ignored), so that the two loads do not queue up.
template <int KEEP>
__global__ __launch_bounds__(kRowThreads) void mv_row_select(
    const float* __restrict__ e, int64_t ld_e, int64_t d, uint32_t N, uint32_t K,
    const u32x2* __restrict__ cand, uint32_t cap, const uint32_t* __restrict__ row_count_sets,
    uint32_t row_count_set_words, const uint32_t* __restrict__ step_no,
    const unsigned long long* __restrict__ tau_pub, const uint32_t* __restrict__ row_poison,
    uint32_t* __restrict__ cand_count, uint32_t* __restrict__ tau_bits, uint32_t* __restrict__ kth_out, uint32_t* __restrict__ tie_cut_out,
    uint32_t* __restrict__ worker_idx, uint32_t* __restrict__ votes32,
    uint32_t* __restrict__ run_tallies, uint32_t n_runs, RowSegments segs, uint32_t* __restrict__ lvl_sets,
    uint32_t* __restrict__ slow_flag, uint32_t parts, uint32_t n_spec, int thresholds_only)
{
    __shared__ SelectLds lds;
    const uint32_t t = threadIdx.x;
    const uint32_t within = blockIdx.x % (8u * parts);
    const uint32_t row = (blockIdx.x / (8u * parts)) * 8u + within % 8u, part = within / 8u;
    if (row >= N) return;                         // whole workgroup
    const u32x2* crow = cand + (size_t)row * cap;
    constexpr bool kWhole = KEEP <= 16;           // whole entries are kept, else bins
    KeptEntries<kWhole ? KEEP : 1> whole;
    uint32_t key[kWhole ? 1 : KEEP];
    auto fetch = [&](int q) {
        const u32x2* at = &crow[min((uint32_t)q * kRowThreads + t, cap - 1)];
        if constexpr (kWhole) whole.entry[q] = *at;
        else                  key[q] = at->x;
    };
#pragma unroll
    for (int q = 0; q < KEEP; ++q) {
        if ((uint32_t)q < n_spec) fetch(q);
        if ((q & 7) == 7) __builtin_amdgcn_sched_barrier(0);   // keep address arithmetic from piling up
    }
    // where bins are kept, the first whole entries of the workgroup's share as well, for the votes (4 x 2^20, K =
    // 10,486: 48.7 -> 48.1 us)
    constexpr int kOwn = kWhole ? 1 : 4;
    u32x2 own[kOwn];
    if constexpr (!kWhole) {
#pragma unroll
        for (int i = 0; i < kOwn; ++i) own[i] = crow[min((part + i * parts) * kRowThreads + t, cap - 1)];
    }
    // (the streaming kernel counted into the counter set of this step's parity)
    const uint32_t epoch = step_no[0] + 1u;
    uint32_t C = row_count_sets[(epoch & 1u) * row_count_set_words + row * kCounterStride];
    const uint32_t tau = (uint32_t)tau_pub[row * (kCounterStride / 2)];   // with the count, not after it
    // a row whose streaming wavefronts did not all see tau in time: its list is incomplete
    const bool poisoned = row_poison[row] == epoch;
    // the fine histogram is cleared while those loads are under way
    clear_fine_histogram(lds);
    if (t == 0) lds.n_list = 0;
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    if (poisoned) C = kRowPoison | C;             // reads as overflowed, here and for every later reader
    if (part == 0 && t == 0) {                    // for the kernels that follow, and the row statistics
        cand_count[row] = C;
        tau_bits[row] = tau;
        slow_flag[row] = 0;
    }
    const bool from_list = C >= K && C <= cap;
    if (!from_list && part != 0) return;          // whole workgroup

    if (from_list) {
        uint32_t kth = 0, tie_cut = 0, path = 0;
        bool done = false;
        if (tau != 0 && C <= (uint32_t)KEEP * kRowThreads) {
#pragma unroll
            for (int q = 0; q < KEEP; ++q)        // longer than expected
                if ((uint32_t)q >= n_spec && (uint32_t)q * kRowThreads < C) fetch(q);      // uniform
            if constexpr (kWhole) {
                done = select_from_registers(whole, crow, C, K, tau, lds, kth, tie_cut);
            } else {
                KeptBins<KEEP> bins;
#pragma unroll
                for (int q = 0; q < KEEP; ++q)
                    bins.set(q, (uint32_t)q * kRowThreads + t < C ? fine_bin(key[q], tau) : 0xFFFFu);
                done = select_from_registers(bins, crow, C, K, tau, lds, kth, tie_cut);
            }
        }
        if (!done) {                              // uniform
            __syncthreads();
            path = 2;
            auto at = [crow](uint64_t i) { return crow[i].x; };
            const KeysInMemory<decltype(at)> src{at, C};
            uint32_t p2;
            select_among_candidates(src, crow, C, K, tau, lds, kth, tie_cut, p2);
        }
        if (part == 0 && t == 0) {
            kth_out[row] = kth;
            tie_cut_out[row] = tie_cut;
            if (path) slow_flag[row] = path;      // diagnostic only
        }
        if (!thresholds_only) {
            for (int i = t; i < 257; i += kRowThreads) lds.lvl[i] = 0;
            __syncthreads();
            const SegmentTallies tallies = {run_tallies ? run_tallies + (size_t)row * (n_runs / 2) : nullptr, segs.shift(row)};
            bool cast = false;
            uint32_t first = part;
            if constexpr (KEEP <= 8) {
                cast = done;
                if (done) cast_votes_from_registers(whole.entry, C, kth, tie_cut, part, parts, votes32, lds.lvl, tallies);
            }
            if constexpr (!kWhole) {
                uint32_t taken = 0;
#pragma unroll
                for (int i = 0; i < kOwn; ++i)
                    taken |= ((part + i * parts) * kRowThreads + t < C && is_taken(own[i], kth, tie_cut) ? 1u : 0u) << i;
                cast_votes<kOwn, false>(own, taken, votes32, lds.lvl, tallies);
                first = part + kOwn * parts;
            }
            if (!cast) cast_votes_of_share(crow, C, kth, tie_cut, first, parts, votes32, lds.lvl, tallies);
            __syncthreads();
            merge_levels(lds.lvl, lvl_sets, blockIdx.x);
        }
        return;
    }

    if (t == 0) slow_flag[row] = 1;
    select_row_from_memory(lds, e + (int64_t)row * ld_e, d, K, worker_idx ? worker_idx + (size_t)row * K : nullptr,
                           thresholds_only ? nullptr : votes32, lvl_sets, kth_out + row, tie_cut_out + row);
}

// ---- exact select over a long list with many workgroups ----------------------
// Finds the `want` largest keys of a list and does something with them: (1) a histogram
// of the keys over the list (see list_bin), (2) every workgroup locates the bin of the
// want-th largest, acts on its entries of higher bins, and moves that bin's members
// to a second list, (3) these are ranked exactly and those that are taken are acted on.
// The rows' top K when K is large (to act = cast the vote, or leave it to mv_vote_count), the add and drop candidates
// of add-drop voting, and the random selection all come this way.
//
// (3) for the rows' top K is a launch of its own: several workgroups rank the same members, each
// acts on its share.  It costs an ordinary row nothing (10 x 11.2 M, K = 111,740: 332 us with it and
// without), and a tie group of a hundred thousand members, which values on a lattice have, is no
// longer one workgroup's to act on (4 x 10 M, K = 300,000 on a lattice: 297 us, so 193; 2 x 10^6 equal values,
// K = 500,001: 4040 and 159).  The other lists are shorter: their last workgroup ranks and acts, or
// the only one, with the histogram in LDS, where one workgroup reads the list in a moment.
//
// What the last workgroup reads of the others -- the second list and its length -- goes
// through atomics, which are performed in memory; the workgroups count themselves done
// behind them, and nobody waits.
constexpr int kListUnroll = 4;                    // entries per thread in flight together
constexpr int kListBatch = kRowThreads * kListUnroll;
// members of the want-th largest's bin that are ranked in LDS: the first lets two workgroups share a compute unit
constexpr int kMembers = 3072, kMembersMost = 8192;
constexpr int kTallyBlocks = 1024;
constexpr uint32_t kAloneList = 4 * kListBatch;   // lists of up to so many entries are left to one workgroup

struct ListView {
    const u32x2* list;
    uint32_t  n;              // entries, at least `want`
    uint32_t  want;
    uint32_t  base, fine, coarse;   // the histogram's bins, see list_bin
    uint32_t* hist;           // kListBins counters, zero between steps
    uint32_t* count2;         // length of the second list, zero between steps
    uint32_t* done;           // workgroups that have passed, zero between steps (on a line of its own)
    u32x2*    list2;          // room for `room` members; step2 = -1: growing downwards
    int       step2;
    uint32_t  room;
    // the rows' lists only: counters of the members per block of 2^block_shift coordinates (segments) and, at count2[1] and
    // [2], the largest of their keys and of the keys' complements (see BigGroup); zero between steps
    uint32_t* blocks;
    uint32_t  block_shift, shift;     // (of the row's segments)
};
constexpr int kCoordBlocks = 2048;                // block_shift is such that there are at most so many

template <int MEMBERS>
struct SplitLds {
    static constexpr uint32_t kMost = MEMBERS;
    __attribute__((aligned(16))) uint32_t hist[kKeyBins];
    __attribute__((aligned(16))) uint32_t key[2][MEMBERS + 4];
    __attribute__((aligned(16))) uint32_t at[2][MEMBERS + 4];
    union {
        uint32_t lvl[257];                        // the rows' votes: see merge_levels
        uint32_t tally[kTallyBlocks];             // the other lists: see BlockTally
    };
    uint32_t bcast[3];
    uint32_t n_list, last;
    uint64_t scan[kRowThreads / kWave];
};

// Counts taken entries per block of coordinates: in LDS and merged at the end, since the taken ones concentrate in
// few blocks and their counters in memory would be the bottleneck (counted there one group of lanes at a time, the
// random selection's pick took 19.8 us instead of 12.7 at 16 x 11.2 M, K = 11,174, the add-drop pick 63 instead of 27 at
// 10 x 11.2 M, K = 111,740); in memory when there are more blocks than LDS has
// counters.
struct BlockTally {
    uint32_t* lds;
    uint32_t* counters;       // of block b at counters[b * stride]
    uint32_t  stride, n_blocks;
    __device__ __forceinline__ void clear() const       // a barrier must follow before the first add
    {
        for (uint32_t b = threadIdx.x; b < n_blocks && b < (uint32_t)kTallyBlocks; b += kRowThreads) lds[b] = 0;
    }
    __device__ __forceinline__ void add(uint32_t block, bool marked) const
    {
        if (n_blocks <= (uint32_t)kTallyBlocks)          // uniform
            tally_groups(block, marked, [&](uint32_t b, uint32_t n) { atomicAdd(&lds[b], n); });
        else
            tally_groups(block, marked, [&](uint32_t b, uint32_t n) { atomicAdd(&counters[b * stride], n); });
    }
    __device__ __forceinline__ void merge() const        // all threads of the workgroup
    {
        if (n_blocks > (uint32_t)kTallyBlocks) return;
        __syncthreads();
        for (uint32_t b = threadIdx.x; b < n_blocks; b += kRowThreads) {
            const uint32_t c = lds[b];
            if (c) atomicAdd(&counters[b * stride], c);
        }
    }
};

// Bins of a list's histogram, ordered like the keys: kListBins / 2 of 2^fine keys from `base` on (keys below
// count there as well), then as many of 2^coarse keys, the last one open-ended.  Where the wanted key is expected
// the bins are narrow, and a workgroup's share of a list still meets few of them: every one it meets is an atomic
// in the merge (10 lists of 145,000: 9.4 us, with 2048 equal bins 10.9).
constexpr int kListBins = 1024;
__device__ __forceinline__ uint32_t list_bin(const ListView& v, uint32_t key)
{
    const uint32_t x = key > v.base ? key - v.base : 0u, half = kListBins / 2;
    const uint32_t in_fine = x >> v.fine;
    return in_fine < half ? in_fine : half + min((x - (half << v.fine)) >> v.coarse, half - 1u);
}
// the keys of bin b: from lo on, 2^bits of them at most
__device__ __forceinline__ void list_bin_range(const ListView& v, uint32_t b, uint32_t& lo, uint32_t& bits)
{
    const uint32_t half = kListBins / 2;
    lo = v.base + (b < half ? b << v.fine : (half << v.fine) + ((b - half) << v.coarse));
    bits = b < half ? v.fine : v.coarse;
    if (b == 0) lo = 0;
    if (b == 0 || b == (uint32_t)(kListBins - 1)) bits = 31;
}

__device__ __forceinline__ u32x2 load_past_caches(const u32x2* p)
{
    const unsigned long long w = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    return u32x2{(uint32_t)w, (uint32_t)(w >> 32)};
}
__device__ __forceinline__ void store_past_caches(u32x2* p, u32x2 v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)v.y << 32 | v.x, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// The histogram of the list's share of workgroup `part` of `parts`
__device__ __forceinline__ void list_hist(const ListView& v, uint32_t part, uint32_t parts, uint32_t* hist_lds)
{
    const uint32_t t = threadIdx.x;
    if (part * (uint32_t)kListBatch >= v.n) return;                 // whole workgroup
    hist_lds[t] = 0;
    __syncthreads();
    for (uint64_t i0 = (uint64_t)part * kListBatch; i0 < v.n; i0 += (uint64_t)parts * kListBatch) {
        uint32_t k[kListUnroll];
#pragma unroll
        for (int u = 0; u < kListUnroll; ++u) {
            const uint64_t i = i0 + (uint32_t)u * kRowThreads + t;
            k[u] = (i < v.n) ? v.list[i].x : 0xFFFFFFFFu;           // keys are at most 0x7FFFFFFF
        }
#pragma unroll
        for (int u = 0; u < kListUnroll; ++u)
            if (k[u] != 0xFFFFFFFFu) atomicAdd(&hist_lds[list_bin(v, k[u])], 1u);
    }
    __syncthreads();
    const uint32_t c = hist_lds[t];
    if (c) atomicAdd(&v.hist[t], c);
}

// The want-th of n members (key[0], at[0] in LDS, a barrier behind them), whose keys lie in
// [lo, lo + 2^bits), under (key descending, coordinate ascending): its key and its coordinate, or
// 0xFFFFFFFF when all with that key are taken.  Ranked by counting when few; else narrowed by
// histograms of the next 12 bits until they are few or all equal.
template <typename Lds>
__device__ __forceinline__ void rank_members(Lds& lds, uint32_t n, uint32_t want, uint32_t lo, uint32_t bits,
                                             uint32_t& kth, uint32_t& tie_cut)
{
    const uint32_t t = threadIdx.x, lane = lane_id();
    for (int cur = 0;; cur ^= 1) {                // uniform
        uint32_t* key = lds.key[cur];
        uint32_t* at = lds.at[cur];
        if (n <= (uint32_t)kRankCap) {
            if (t < 4) {                          // pad to a multiple of 4 with entries ranked last
                key[n + t] = 0;
                at[n + t] = 0xFFFFFFFFu;
            }
            __syncthreads();
            if (t < n) {
                const uint32_t mk = key[t], mi = at[t];
                const u32x4* hk = reinterpret_cast<const u32x4*>(key);
                const u32x4* hi = reinterpret_cast<const u32x4*>(at);
                uint32_t ahead = 0;
#pragma unroll 4
                for (uint32_t j = 0; j < (n + 3) / 4; ++j) {
                    const u32x4 ok = hk[j], oi = hi[j];
                    ahead += (ok.x > mk) || (ok.x == mk && oi.x < mi);
                    ahead += (ok.y > mk) || (ok.y == mk && oi.y < mi);
                    ahead += (ok.z > mk) || (ok.z == mk && oi.z < mi);
                    ahead += (ok.w > mk) || (ok.w == mk && oi.w < mi);
                }
                if (ahead == want - 1) {
                    lds.bcast[0] = mk;
                    lds.bcast[1] = mi;
                }
            }
            __syncthreads();
            kth = lds.bcast[0];
            tie_cut = lds.bcast[1];
            __syncthreads();
            return;
        }
        if (bits == 0) {
            kth = lo;
            tie_cut = want < n ? smallest_coordinate(lds, at, n, want) : 0xFFFFFFFFu;
            return;
        }
        const uint32_t rest = bits > 12u ? bits - 12u : 0u;
        for (int b = t; b < kKeyBins; b += kRowThreads) lds.hist[b] = 0;
        if (t == 0) lds.n_list = 0;
        __syncthreads();
        for (uint32_t p0 = 0; p0 < n; p0 += kRowThreads) {           // wave-wide grouping: many keys may be equal
            const uint32_t p = p0 + t;
            tally_digit(lds.hist, p < n, p < n ? (key[p] - lo) >> rest : 0u, lane);
        }
        __syncthreads();
        uint32_t sub, in_sub;
        find_rank_bin<kKeyBins>(lds.hist, lds.scan, lds.bcast, want, sub, want, in_sub);
        for (uint32_t p0 = 0; p0 < n; p0 += kRowThreads) {
            const uint32_t p = p0 + t;
            const bool mine = p < n && (key[p] - lo) >> rest == sub;
            const uint32_t s = wave_slots(mine, &lds.n_list, lane);
            if (mine) {
                lds.key[cur ^ 1][s] = key[p];
                lds.at[cur ^ 1][s] = at[p];
            }
        }
        __syncthreads();
        n = in_sub;
        lo += sub << rest;
        bits = rest;
    }
}

// The same over n entries in memory, entry(i) = (key, coordinate): those in [lo, lo + 2^bits) are `count`
// members, more than LDS holds.  Narrowed by histograms of the next 12 bits until they fit (or are all equal).
template <typename Lds, typename Entry>
__device__ __forceinline__ void rank_in_memory(Lds& lds, Entry entry, uint32_t n, uint32_t count, uint32_t want,
                                               uint32_t lo, uint32_t bits, uint32_t& kth, uint32_t& tie_cut)
{
    const uint32_t t = threadIdx.x, lane = lane_id();
    // f(entry, member) the same number of times in every lane, eight loads in flight
    auto each = [&](auto f) {
        for (uint64_t i0 = 0; i0 < n; i0 += (uint64_t)kRowThreads * 8) {
            u32x2 c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint64_t i = i0 + (uint32_t)u * kRowThreads + t;
                const u32x2 none = {0u, 0u};
                c[u] = i < n ? entry(i) : none;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                f(c[u], i0 + (uint32_t)u * kRowThreads + t < n && c[u].x - lo < 1u << bits);
        }
    };
    while (count > Lds::kMost && bits != 0) {                // uniform
        const uint32_t rest = bits > 12u ? bits - 12u : 0u;
        for (int b = t; b < kKeyBins; b += kRowThreads) lds.hist[b] = 0;
        __syncthreads();
        each([&](u32x2 c, bool member) { tally_digit(lds.hist, member, member ? (c.x - lo) >> rest : 0u, lane); });
        __syncthreads();
        uint32_t sub;
        find_rank_bin<kKeyBins>(lds.hist, lds.scan, lds.bcast, want, sub, want, count);
        lo += sub << rest;
        bits = rest;
    }
    if (count <= Lds::kMost) {            // uniform
        if (t == 0) lds.n_list = 0;
        __syncthreads();
        each([&](u32x2 c, bool member) {
            const uint32_t p = wave_slots(member, &lds.n_list, lane);
            if (member) {
                lds.key[0][p] = c.x;
                lds.at[0][p] = c.y;
            }
        });
        __syncthreads();
        rank_members(lds, count, want, lo, bits, kth, tie_cut);
        return;
    }
    kth = lo;
    tie_cut = 0xFFFFFFFFu;
    if (want < count) {                           // uniform; entries that are not ties are mapped below every tie
        auto tie_at = [&](uint64_t i) {
            const u32x2 c = entry(i);
            return c.x == lo ? kAbsMask - c.y : 0u;
        };
        const KeysInMemory<decltype(tie_at)> ties{tie_at, n};
        uint32_t a, b;
        tie_cut = kAbsMask - block_radix_select(ties, want, lds.hist, lds.scan, lds.bcast, a, b);
    }
}

// What of a list is still to be decided when its histogram has been read and every entry of a higher bin has been
// acted on: the members of one bin, of which the first `want` under (key descending, coordinate ascending) are taken.
struct ListRest {
    uint32_t bin, want, n;
};

// Members that the second list has no room for are found in the first one again.
__device__ __forceinline__ bool members_stored(const ListView& v, const ListRest& r) { return r.n <= v.room; }

// A member; PAST: past the caches, as this launch's other workgroups have stored it.
template <bool PAST>
__device__ __forceinline__ u32x2 member_at(const ListView& v, uint64_t i)
{
    const u32x2* at = v.list2 + (int64_t)i * v.step2;
    if constexpr (PAST) return load_past_caches(at);
    return *at;
}

// By one workgroup, with the members in the second list (or in the first): their ranking, ...
template <bool PAST, typename Lds>
__device__ __forceinline__ void rank_rest(const ListView& v, const ListRest& r, Lds& lds, uint32_t& kth, uint32_t& tie_cut)
{
    uint32_t lo, bits;
    list_bin_range(v, r.bin, lo, bits);
    if (r.want == r.n) {                          // uniform: all of them are taken
        kth = lo;
        tie_cut = 0xFFFFFFFFu;
        return;
    }
    const bool stored = members_stored(v, r);
    if (stored && r.n <= Lds::kMost) {            // uniform
        for (uint32_t p = threadIdx.x; p < r.n; p += kRowThreads) {
            const u32x2 m = member_at<PAST>(v, p);
            lds.key[0][p] = m.x;
            lds.at[0][p] = m.y;
        }
        __syncthreads();
        rank_members(lds, r.n, r.want, lo, bits, kth, tie_cut);
    } else if (stored) {
        rank_in_memory(lds, [&](uint64_t i) { return member_at<PAST>(v, i); }, r.n, r.n, r.want, lo, bits, kth, tie_cut);
    } else {
        rank_in_memory(lds,
                       [&](uint64_t i) {          // what is no member gets a key outside every range
                           u32x2 m = v.list[i];
                           if (list_bin(v, m.x) != r.bin) m.x = 0xFFFFFFFFu;
                           return m;
                       },
                       v.n, r.n, r.want, lo, bits, kth, tie_cut);
    }
}

// ... and act for the taken ones among the share of workgroup `part` of `parts`.
template <bool PAST, typename Act>
__device__ __forceinline__ void act_on_rest(const ListView& v, const ListRest& r, uint32_t kth, uint32_t tie_cut,
                                            uint32_t part, uint32_t parts, Act act)
{
    const bool stored = members_stored(v, r);
    const uint32_t n = stored ? r.n : v.n;
    for (uint64_t i0 = (uint64_t)part * kListBatch; i0 < n; i0 += (uint64_t)parts * kListBatch) {
        u32x2 c[kListUnroll];
        uint32_t taken = 0;
#pragma unroll
        for (int u = 0; u < kListUnroll; ++u) {
            const uint64_t i = i0 + (uint32_t)u * kRowThreads + threadIdx.x;
            const u32x2 none = {0u, 0xFFFFFFFFu};
            c[u] = i < n ? (stored ? member_at<PAST>(v, i) : v.list[i]) : none;
        }
#pragma unroll
        for (int u = 0; u < kListUnroll; ++u)
            taken |= (c[u].y != 0xFFFFFFFFu && (stored || list_bin(v, c[u].x) == r.bin) && is_taken(c[u], kth, tie_cut)
                          ? 1u : 0u) << u;
        if (__ballot(taken != 0u) != 0ull) act(c, taken);            // wave-uniform
    }
}

// A bin with more members than LDS holds: nearly always a tie group (values on a lattice, a row of equal values),
// of which the lowest coordinates are taken.  Read member by member by one workgroup such a group of a million costs
// milliseconds, so the workgroups that find the members also count them per block of coordinates and note
// whether all keys are the same.
template <typename Lds>
struct BigGroup {
    Lds&     lds;
    uint32_t largest = 0, largest_not = 0;
    __device__ __forceinline__ void clear()       // a barrier must follow before the first add
    {
        for (uint32_t b = threadIdx.x; b < (uint32_t)kCoordBlocks; b += kRowThreads) lds.hist[b] = 0;
        if (threadIdx.x < 2) lds.bcast[threadIdx.x] = 0;
    }
    __device__ __forceinline__ void add(const ListView& v, u32x2 c, bool member)
    {
        if (member) {
            largest = max(largest, c.x);
            largest_not = max(largest_not, ~c.x);
        }
        tally_groups((c.y + v.shift) >> v.block_shift, member, [&](uint32_t b, uint32_t n) { atomicAdd(&lds.hist[b], n); });
    }
    __device__ __forceinline__ void merge(const ListView& v)         // all threads of the workgroup
    {
        for (int o = 1; o < kWave; o <<= 1) {
            largest = max(largest, (uint32_t)__shfl_xor(largest, o, kWave));
            largest_not = max(largest_not, (uint32_t)__shfl_xor(largest_not, o, kWave));
        }
        if (lane_id() == 0) {
            atomicMax(&lds.bcast[0], largest);
            atomicMax(&lds.bcast[1], largest_not);
        }
        __syncthreads();
        if (threadIdx.x < 2) atomicMax(&v.count2[1 + threadIdx.x], lds.bcast[threadIdx.x]);
        for (uint32_t b = threadIdx.x; b < (uint32_t)kCoordBlocks; b += kRowThreads) {
            const uint32_t n = lds.hist[b];
            if (n) atomicAdd(&v.blocks[b], n);
        }
    }
};

// The coordinate of the want-th of a row's candidates with this key, in coordinate order, `count` being the
// thread's two counters of v.blocks: the block it lies in, its run among the block's, its place in the
// run (runs are ascending).
template <typename Lds>
__device__ __forceinline__ uint32_t tie_cut_by_blocks(const ListView& v, const uint32_t (&count)[2], uint32_t key,
                                                      uint32_t want, const u32x2* __restrict__ runs, uint32_t n_segs, uint32_t n_dealt,
                                                      Lds& lds)
{
    static_assert(kCoordBlocks == 2 * kRowThreads, "two blocks to a thread");
    const uint32_t t = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave);
    uint32_t total;
    uint32_t ex = block_excl_scan<kRowThreads>(count[0] + count[1], lds.scan, total);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (ex < want && want <= ex + count[q]) {
            lds.bcast[0] = 2u * t + q;
            lds.bcast[1] = want - ex;
        }
        ex += count[q];
    }
    __syncthreads();
    static_assert(((1ll << 31) + kSeg) >> 21 < kCoordBlocks && (1 << 21) / kSeg == 2 * kRowThreads,
                  "at most two runs to a thread in a block of a row of up to 2^31 coordinates");
    const uint32_t per_block = (1u << v.block_shift) / kSeg;         // runs: at most 2048
    const uint32_t r0 = lds.bcast[0] * per_block, n_here = min(per_block, n_segs - r0);
    want = lds.bcast[1];
    __syncthreads();
    if (n_here > 1) {                             // uniform: a wavefront per run counts
        for (uint32_t i = wave; i < n_here; i += kRowThreads / kWave) {
            const u32x2 run = runs[run_place(r0 + i, n_dealt)];
            uint32_t k[kSeg / kWave];
            uint32_t n = 0;
#pragma unroll
            for (int q = 0; q < kSeg / kWave; ++q) {
                const uint32_t j = (uint32_t)q * kWave + lane;
                k[q] = j < run.y ? v.list[run.x + j].x : 0xFFFFFFFFu;
            }
#pragma unroll
            for (int q = 0; q < kSeg / kWave; ++q) n += (uint32_t)__popcll(__ballot(k[q] == key));
            if (lane == 0) lds.hist[i] = n;
        }
        __syncthreads();
        const uint32_t mine[2] = {2 * t < n_here ? lds.hist[2 * t] : 0u, 2 * t + 1 < n_here ? lds.hist[2 * t + 1] : 0u};
        ex = block_excl_scan<kRowThreads>(mine[0] + mine[1], lds.scan, total);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (ex < want && want <= ex + mine[q]) {
                lds.bcast[0] = 2 * t + q;
                lds.bcast[1] = want - ex;
            }
            ex += mine[q];
        }
        __syncthreads();
        want = lds.bcast[1];
    } else if (t == 0) {
        lds.bcast[0] = 0;
    }
    __syncthreads();
    const u32x2 run = runs[run_place(r0 + lds.bcast[0], n_dealt)];
    __syncthreads();
    static_assert(kSeg == kRowThreads, "a thread per entry of a run");
    const bool tie = t < run.y && v.list[run.x + t].x == key;
    ex = block_excl_scan<kRowThreads>(tie ? 1u : 0u, lds.scan, total);
    if (tie && ex == want - 1) lds.bcast[0] = v.list[run.x + t].y;
    __syncthreads();
    const uint32_t cut = lds.bcast[0];
    __syncthreads();
    return cut;
}

// How list_split ends: with the histogram taken here by the list's only workgroup; by the last of the list's
// workgroups; or not at all -- the next launch ranks the members and acts on them.
enum class SplitEnd { Alone, Last, Later };

// Workgroup `part` of `parts` of a list.  act(c, taken): the marked ones of a batch of kListUnroll entries per
// thread are among the `want` largest; every one of these is marked in exactly one call, by one workgroup.  A
// wavefront calls it for the batches in which it has marked ones; it must hold no barrier.
// Returns true to all threads of the one workgroup that finished the list, with kth / tie_cut (the membership
// test is is_taken).  SplitEnd::Later: false to all, with `rest`.
template <SplitEnd END, typename Lds, typename Act>
__device__ __forceinline__ bool list_split(const ListView& v, uint32_t part, uint32_t parts, Lds& lds, Act act,
                                           uint32_t& kth, uint32_t& tie_cut, ListRest& rest)
{
    constexpr bool ALONE = END == SplitEnd::Alone, LATER = END == SplitEnd::Later;
    const uint32_t t = threadIdx.x, lane = lane_id();
    const u32x2 none = {0u, 0xFFFFFFFFu};
    u32x2 c[kListUnroll];
    auto load = [&](uint64_t i0) {
#pragma unroll
        for (int u = 0; u < kListUnroll; ++u) {
            const uint64_t i = i0 + (uint32_t)u * kRowThreads + t;
            c[u] = i < v.n ? v.list[i] : none;
        }
    };
    const uint64_t first = (uint64_t)part * kListBatch;
    load(first);
    if (t == 0) lds.n_list = 0;
    if (ALONE) {
        lds.hist[t] = 0;
        __syncthreads();
        for (uint64_t i0 = 0; i0 < v.n; i0 += kListBatch) {
            if (i0) load(i0);
#pragma unroll
            for (int u = 0; u < kListUnroll; ++u)
                if (c[u].y != 0xFFFFFFFFu) atomicAdd(&lds.hist[list_bin(v, c[u].x)], 1u);
        }
        if (v.n > (uint32_t)kListBatch) load(0);
    } else {
        lds.hist[t] = v.hist[t];
    }
    __syncthreads();
    find_rank_bin<kListBins>(lds.hist, lds.scan, lds.bcast, v.want, rest.bin, rest.want, rest.n);
    // Space in the second list is reserved once per workgroup, or per workgroup and batch when the members are many:
    // reservations of one list follow each other at the memory side, about 9 ns apart (once per wavefront
    // instead, random selection took 452 us at 16 x 11.2 M, K = 11,174, for 441 so, and at 3 x 10 M, K = 150,000,
    // 207 for 169).
    const bool few = rest.n <= Lds::kMost;        // uniform
    BigGroup<Lds> group = {lds};
    if (LATER && !few) group.clear();             // (a barrier follows before the first add)
    for (uint64_t i0 = first; i0 < v.n; i0 += (uint64_t)parts * kListBatch) {
        if (i0 != first) load(i0);
        uint32_t above = 0, member = 0;
#pragma unroll
        for (int u = 0; u < kListUnroll; ++u) {
            const uint32_t b = list_bin(v, c[u].x);
            const bool there = c[u].y != 0xFFFFFFFFu;
            above |= (there && b > rest.bin ? 1u : 0u) << u;
            member |= (there && b == rest.bin ? 1u : 0u) << u;
        }
        if (ALONE || few) {
            // (few members in the whole list: they all fit; in a list alone, as many as fit)
#pragma unroll
            for (int u = 0; u < kListUnroll; ++u) {
                const bool mine = member >> u & 1u;
                const uint32_t p = wave_slots(mine, &lds.n_list, lane);
                if (mine && p < Lds::kMost) {
                    lds.key[0][p] = c[u].x;
                    lds.at[0][p] = c[u].y;
                }
            }
            if (__ballot(above != 0u) != 0ull) act(c, above);        // wave-uniform
        } else {
            uint32_t total;
            uint32_t p = block_excl_scan<kRowThreads>((uint32_t)__popc(member), lds.scan, total);
            uint32_t base = 0;
            if (t == 0 && total != 0u) base = atomicAdd(v.count2, total);
            if (__ballot(above != 0u) != 0ull) act(c, above);        // wave-uniform
            if (LATER)
#pragma unroll
                for (int u = 0; u < kListUnroll; ++u) group.add(v, c[u], member >> u & 1u);
            if (t == 0) lds.n_list = base;
            __syncthreads();
            p += lds.n_list;
#pragma unroll
            for (int u = 0; u < kListUnroll; ++u)
                if (member >> u & 1u) {
                    if (p < v.room) store_past_caches(v.list2 + (int64_t)p * v.step2, c[u]);
                    ++p;
                }
            __syncthreads();                      // (lds.n_list has been read)
        }
    }
    if (!ALONE && few) {                          // uniform
        __syncthreads();
        const uint32_t n = lds.n_list;
        if (t == 0 && n != 0u) lds.bcast[0] = atomicAdd(v.count2, n);
        __syncthreads();
        for (uint32_t p = t; p < n; p += kRowThreads) {
            const uint32_t to = lds.bcast[0] + p;
            const u32x2 m = {lds.key[0][p], lds.at[0][p]};
            if (to < v.room) store_past_caches(v.list2 + (int64_t)to * v.step2, m);
        }
    }
    if (LATER) {
        if (!few && first < v.n) group.merge(v);
        return false;
    }
    if (ALONE) {
        __syncthreads();
        uint32_t lo, bits;
        list_bin_range(v, rest.bin, lo, bits);
        ListView again = v;                       // more members than LDS holds are found in the list again
        again.room = 0;
        if (rest.n <= Lds::kMost) rank_members(lds, rest.n, rest.want, lo, bits, kth, tie_cut);   // uniform
        else                      rank_rest<false>(again, rest, lds, kth, tie_cut);
        act_on_rest<false>(again, rest, kth, tie_cut, 0, 1, act);
        return true;
    }
    // every store and atomic of this workgroup has been performed before it is counted as done
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (t == 0) lds.last = atomicAdd(v.done, 1u) == parts - 1u;
    __syncthreads();
    if (!lds.last) return false;
    // what the next step must find at zero
    v.hist[t] = 0;
    if (t == 0) {
        *v.count2 = 0;
        *v.done = 0;
    }
    if (few) {                                    // uniform
        rank_rest<true>(v, rest, lds, kth, tie_cut);
        act_on_rest<true>(v, rest, kth, tie_cut, 0, 1, act);
    } else {
        // many members are read several times: with this unit's and its L2's copies dropped, plain loads find what
        // was stored past the caches, and find it in the cache the next time (dropped by the last workgroup of
        // every list, a step of 16 x 300,001, K = 30,000, K_ad = 3000 took 139 us instead of 118)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        rank_rest<false>(v, rest, lds, kth, tie_cut);
        act_on_rest<false>(v, rest, kth, tie_cut, 0, 1, act);
    }
    return true;
}

// ---- the rows' top-K when K is large: grid (workgroups of a list, rows)
// A row whose list is too short or overflowed (or that was marked) is left to its first workgroup of
// mv_sel_split, which selects it from memory.
constexpr uint32_t kHistRow = kHistBins;          // words of a row's sample histogram, which lends its storage below
constexpr uint32_t kCtlWords = 3 * kListBins;      // behind three histograms: the counters, a line each
// The sample histograms are at zero when the streaming kernel has ended: list number `which` (0, 1, 2) of a
// row keeps its histogram and its two counters there, and leaves them at zero as well.
__device__ __forceinline__ void lend_storage(ListView& v, uint32_t* __restrict__ sample_hist, uint32_t row, uint32_t which)
{
    uint32_t* h = sample_hist + (size_t)row * kHistRow;
    v.hist = h + which * kListBins;
    v.count2 = h + kCtlWords + (2 * which) * kCounterStride;
    v.done = h + kCtlWords + (2 * which + 1) * kCounterStride;
    v.step2 = 1;
    v.room = v.n;
    v.blocks = nullptr;
    v.block_shift = 0;
    v.shift = 0;
}
static_assert(kListBins == kRowThreads, "a bin per thread");
static_assert(kHistRow >= kCtlWords + 6 * kCounterStride, "three lists' storage fits a row's sample histogram");

// A row's list as mv_sel_hist, mv_sel_split and mv_sel_finish see it.  2048 bins to an octave above the row's
// threshold, beyond a quarter octave 32; without a threshold (nearly all of the row is wanted) 4 to an octave.
__device__ __forceinline__ ListView row_list(u32x2* __restrict__ cand, uint32_t cap, uint32_t row, uint32_t n, uint32_t K,
                                             uint32_t tau, uint32_t* __restrict__ sample_hist, uint32_t block_shift,
                                             uint32_t shift)
{
    ListView v;
    v.list = cand + (size_t)row * cap;  v.n = n;
    v.want = K;
    v.base = tau;
    v.fine = tau ? 12 : 21;
    v.coarse = tau ? 18 : 21;
    lend_storage(v, sample_hist, row, 0);
    v.list2 = cand + (size_t)row * cap + (cap - 1);                 // the end of the row's storage, downwards
    v.step2 = -1;
    v.room = cap - v.n;
    v.blocks = v.hist + kListBins;                // (the other two lists' storage: add-drop voting uses it later)
    v.block_shift = block_shift;
    v.shift = shift;
    return v;
}
static_assert(kCoordBlocks <= 2 * kListBins, "the blocks' counters fit two lists' histograms");

__global__ __launch_bounds__(kRowThreads) void mv_sel_hist(
    u32x2* __restrict__ cand, uint32_t cap, uint32_t K, const uint32_t* __restrict__ row_count_sets,
    uint32_t row_count_set_words, const uint32_t* __restrict__ step_no, const unsigned long long* __restrict__ tau_pub,
    const uint32_t* __restrict__ row_poison, uint32_t* __restrict__ sample_hist, uint32_t* __restrict__ cand_count,
    uint32_t* __restrict__ tau_bits, uint32_t* __restrict__ slow_flag)
{
    __shared__ uint32_t hist[kListBins];
    const uint32_t row = blockIdx.y;
    const uint32_t epoch = step_no[0] + 1u;
    uint32_t C = row_count_sets[(epoch & 1u) * row_count_set_words + row * kCounterStride];
    const uint32_t tau = (uint32_t)tau_pub[row * (kCounterStride / 2)];
    if (row_poison[row] == epoch) C |= kRowPoison;                   // reads as overflowed, here and for later readers
    const bool from_list = C >= K && C <= cap;
    if (blockIdx.x == 0 && threadIdx.x == 0) {                       // for the kernels that follow, and the row statistics
        cand_count[row] = C;
        tau_bits[row] = tau;
        slow_flag[row] = from_list ? 0u : 1u;
    }
    if (!from_list) return;                                          // whole workgroup
    list_hist(row_list(cand, cap, row, C, K, tau, sample_hist, 0, 0), blockIdx.x, gridDim.x, hist);
}

// Votes for the marked entries of a batch; unless CAST (add-drop voting, or mv_vote_count behind) none are cast.
template <bool CAST>
struct CastVotes {
    uint32_t *votes32, *lvl;
    SegmentTallies tallies;
    __device__ __forceinline__ void operator()(const u32x2 (&c)[kListUnroll], uint32_t taken) const
    {
        if constexpr (CAST) cast_votes<kListUnroll, true>(c, taken, votes32, lvl, tallies);
    }
};

// What mv_sel_split leaves of a row to mv_sel_finish: behind the row's published threshold, on the line it has
// to itself.
__device__ __forceinline__ uint32_t* row_rest(unsigned long long* tau_pub, uint32_t row)
{
    return reinterpret_cast<uint32_t*>(tau_pub + row * (kCounterStride / 2) + 1);
}

// Chunks of coordinates with so many list entries that mv_vote_count deals them out in pieces.
struct CrowdedChunks {
    uint32_t* n;                                  // how many there are
    uint32_t* entries;                            // of each chunk (null: they are not looked for)
    uint32_t* list;                               // of them, in any order
    uint32_t  n_chunks, chunk_shift;
    uint32_t  least;                              // what a row has less of in a chunk is passed over
};
constexpr uint32_t kCrowdedEntries = 8192;        // a chunk is crowded from so many entries on

// The streaming pass leaves a row's runs as its workgroups noted them; the kernels behind mv_sel_split read them in the
// order of the segments, a few neighbouring ones at a time, where they go by chunks of coordinates.  Workgroup `part`
// of a row's puts some groups of 64 in order: a wavefront has a whole one in its registers, so it stays in place.  The
// addition that takes a chunk's entries to kCrowdedEntries puts it on the list.
constexpr int kOrderGroups = 4;                   // groups per wavefront
constexpr uint32_t kOrderRuns = kRowThreads * kOrderGroups;
__device__ __forceinline__ void order_runs(u32x2* __restrict__ row_runs, uint32_t n, uint32_t part,
                                           const CrowdedChunks& crowd)
{
    const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t g0 = (part * (kRowThreads / kWave) + wave) * kOrderGroups;
    const uint32_t from = run_place(lane, kWave);                    // of the group's segment number `lane`
    u32x2 r[kOrderGroups];
#pragma unroll
    for (int q = 0; q < kOrderGroups; ++q) {
        r[q] = u32x2{0u, 0u};
        if ((g0 + q) * kWave + lane < n) r[q] = row_runs[(g0 + q) * kWave + lane];
    }
#pragma unroll
    for (int q = 0; q < kOrderGroups; ++q)
        if ((g0 + q + 1) * kWave <= n) {           // uniform; less than a group at the row's end is in order
            r[q].x = __shfl(r[q].x, from, kWave);
            r[q].y = __shfl(r[q].y, from, kWave);
            row_runs[(g0 + q) * kWave + lane] = r[q];
        }
    if (!crowd.entries) return;                    // uniform
    const uint32_t own = (1u << crowd.chunk_shift) / kSeg;           // segments to a chunk: 1, 2 or 4
#pragma unroll
    for (int q = 0; q < kOrderGroups; ++q) {
        uint32_t sum = r[q].y;
        if (own > 1) sum += __shfl_xor(sum, 1, kWave);
        if (own > 2) sum += __shfl_xor(sum, 2, kWave);
        const uint32_t c = ((g0 + q) * kWave + lane) / own;          // (a shifted row may have a segment behind the last)
        if ((lane & (own - 1)) != 0u || sum < crowd.least || c >= crowd.n_chunks) continue;
        const uint32_t before = atomicAdd(crowd.entries + c, sum);
        if (before < kCrowdedEntries && before + sum >= kCrowdedEntries) crowd.list[atomicAdd(crowd.n, 1u)] = c;
    }
}
static_assert(kGroupSegs == kWave, "a lane per segment of a group");

// The members of the K-th's bin are left to mv_sel_finish.  Workgroups (split_blocks + part, row) put the row's runs in
// order.
template <bool CAST>
__global__ __launch_bounds__(kRowThreads) void mv_sel_split(
    const float* __restrict__ e, int64_t ld_e, int64_t d, u32x2* cand, uint32_t cap, uint32_t K,
    const uint32_t* __restrict__ cand_count, const uint32_t* __restrict__ tau_bits,
    const uint32_t* __restrict__ slow_flag, uint32_t* __restrict__ sample_hist,
    uint32_t* __restrict__ kth_out, uint32_t* __restrict__ tie_cut_out, uint32_t* __restrict__ worker_idx,
    uint32_t* __restrict__ votes32, uint32_t* __restrict__ run_tallies, u32x2* __restrict__ runs, uint32_t n_runs,
    RowSegments segs, uint32_t* __restrict__ lvl_sets, unsigned long long* __restrict__ tau_pub,
    uint32_t block_shift, uint32_t split_blocks, CrowdedChunks crowd)
{
    __shared__ SplitLds<kMembers> lds;
    const uint32_t row = blockIdx.y, t = threadIdx.x;
    if (blockIdx.x >= split_blocks) {
        if (slow_flag[row] == 1u) crowd.entries = nullptr;           // (its runs are not read)
        order_runs(runs + (size_t)row * n_runs, segs.count(row), blockIdx.x - split_blocks, crowd);
        return;
    }
    if (slow_flag[row] == 1u) {
        if (blockIdx.x == 0)
            select_row_from_memory(lds, e + (int64_t)row * ld_e, d, K, worker_idx ? worker_idx + (size_t)row * K : nullptr,
                                   CAST ? votes32 : nullptr, lvl_sets, kth_out + row, tie_cut_out + row);
        return;
    }
    const ListView v = row_list(cand, cap, row, cand_count[row], K, tau_bits[row], sample_hist, block_shift,
                                segs.shift(row));
    for (int i = t; i < 257; i += kRowThreads) lds.lvl[i] = 0;       // ordered by the barriers before the first act
    const CastVotes<CAST> act = {votes32, lds.lvl, {run_tallies ? run_tallies + (size_t)row * (n_runs / 2) : nullptr, v.shift}};
    uint32_t kth, tie_cut;
    ListRest rest;
    (void)list_split<SplitEnd::Later>(v, blockIdx.x, split_blocks, lds, act, kth, tie_cut, rest);
    if (blockIdx.x == 0 && t == 0) {
        uint32_t* r = row_rest(tau_pub, row);
        r[0] = rest.bin;
        r[1] = rest.want;
        r[2] = rest.n;
    }
    if constexpr (CAST) {
        __syncthreads();
        merge_levels(lds.lvl, lvl_sets, blockIdx.y * split_blocks + blockIdx.x);
    }
}

// The end of the rows' select: grid (parts, rows).  Every workgroup of a row ranks the members -- the work
// is repeated rather than shared so that no workgroup waits for another -- and casts the votes of its share.
template <bool CAST>
__global__ __launch_bounds__(kRowThreads) void mv_sel_finish(
    u32x2* cand, uint32_t cap, uint32_t K, const uint32_t* __restrict__ cand_count, const uint32_t* __restrict__ tau_bits,
    const uint32_t* __restrict__ slow_flag, uint32_t* __restrict__ sample_hist, uint32_t* __restrict__ kth_out,
    uint32_t* __restrict__ tie_cut_out, uint32_t* __restrict__ votes32, uint32_t* __restrict__ run_tallies, uint32_t n_runs,
    RowSegments segs, uint32_t* __restrict__ lvl_sets, unsigned long long* __restrict__ tau_pub,
    const u32x2* __restrict__ runs, int in_order, uint32_t block_shift)
{
    __shared__ SplitLds<kMembers> lds;
    const uint32_t row = blockIdx.y, t = threadIdx.x;
    if (slow_flag[row] == 1u) return;
    const ListView v = row_list(cand, cap, row, cand_count[row], K, tau_bits[row], sample_hist, block_shift,
                                segs.shift(row));
    const uint32_t* left = row_rest(tau_pub, row);
    const ListRest rest = {left[0], left[1], left[2]};
    const uint32_t share = members_stored(v, rest) ? rest.n : v.n;
    if (blockIdx.x != 0 && blockIdx.x * (uint32_t)kListBatch >= share) return;      // nothing to act on
    if (blockIdx.x == 0) {                        // what the next step must find at zero
        v.hist[t] = 0;
        if (t == 0) *v.count2 = 0;
    }
    for (int i = t; i < 257; i += kRowThreads) lds.lvl[i] = 0;       // ordered by the next barrier
    const CastVotes<CAST> act = {votes32, lds.lvl, {run_tallies ? run_tallies + (size_t)row * (n_runs / 2) : nullptr, v.shift}};
    uint32_t kth, tie_cut;
    if (rest.n <= (uint32_t)kMembers && members_stored(v, rest)) {   // uniform; usual: this is the row's only workgroup
        static_assert(kMembers <= kListBatch, "a batch holds them");
        u32x2 c[kListUnroll];
        const u32x2 none = {0u, 0xFFFFFFFFu};
#pragma unroll
        for (int u = 0; u < kListUnroll; ++u) {
            const uint32_t i = (uint32_t)u * kRowThreads + t;
            c[u] = i < rest.n ? member_at<false>(v, i) : none;
        }
#pragma unroll
        for (int u = 0; u < kListUnroll; ++u)
            if (c[u].y != 0xFFFFFFFFu) {
                lds.key[0][u * kRowThreads + t] = c[u].x;
                lds.at[0][u * kRowThreads + t] = c[u].y;
            }
        __syncthreads();
        uint32_t lo, bits;
        list_bin_range(v, rest.bin, lo, bits);
        rank_members(lds, rest.n, rest.want, lo, bits, kth, tie_cut);
        if (t == 0) {
            kth_out[row] = kth;
            tie_cut_out[row] = tie_cut;
        }
        if constexpr (!CAST) return;
        uint32_t taken = 0;
#pragma unroll
        for (int u = 0; u < kListUnroll; ++u)
            taken |= (c[u].y != 0xFFFFFFFFu && is_taken(c[u], kth, tie_cut) ? 1u : 0u) << u;
        if (__ballot(taken != 0u) != 0ull) act(c, taken);            // wave-uniform
        __syncthreads();
        merge_levels(lds.lvl, lvl_sets, row);
        return;
    }
    __syncthreads();                              // (a bin that is wanted whole is acted on without another)
    bool ranked = false;
    if (rest.n > (uint32_t)kMembers) {            // uniform: a big group
        const uint32_t count[2] = {v.blocks[2 * t], v.blocks[2 * t + 1]};
        const uint32_t largest = v.count2[1], smallest = ~v.count2[2];
        // these values are there before the workgroup is counted
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (t == 0) lds.last = atomicAdd(v.done, 1u) + 1u == min(gridDim.x, (share + kListBatch - 1) / kListBatch);
        __syncthreads();
        if (lds.last) {                           // every workgroup of the row has read them
            v.blocks[2 * t] = 0;
            v.blocks[2 * t + 1] = 0;
            if (t < 2) v.count2[1 + t] = 0;
            if (t == 0) *v.done = 0;
        }
        if (largest == smallest && rest.want < rest.n) {
            kth = largest;
            tie_cut = tie_cut_by_blocks(v, count, kth, rest.want, runs + (size_t)row * n_runs, segs.count(row),
                                        in_order ? 0u : segs.count(row), lds);
            ranked = true;
        }
    }
    if (!ranked) rank_rest<false>(v, rest, lds, kth, tie_cut);
    kth = max(kth, v.base);                       // (where a bin is wanted whole: what is not in the list stays outside)
    if (blockIdx.x == 0 && t == 0) {
        kth_out[row] = kth;
        tie_cut_out[row] = tie_cut;
    }
    if constexpr (!CAST) return;
    act_on_rest<false>(v, rest, kth, tie_cut, blockIdx.x, gridDim.x, act);
    __syncthreads();
    merge_levels(lds.lvl, lvl_sets, blockIdx.y * gridDim.x + blockIdx.x);
}

}  // namespace mvk
