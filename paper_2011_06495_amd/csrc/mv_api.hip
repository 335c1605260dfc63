// Host side of the C ABI declared in include/mv.h: argument checks, scratch
// layout, and the launch sequence of one vote step (Algorithm 1 of the paper,
// error compensation .. error update).  Every step of the method runs in the
// kernels of mv_kernels.hpp; nothing is computed on the host.
#include "../../include/mv.h"
#include "mv_kernels.hpp"

#include <hip/hip_runtime.h>
#include <new>
#include <stdint.h>
#include <string.h>
#include <math.h>

namespace {

enum KernelId {
    KID_STREAM = 0,
    KID_ROW_SELECT,
    // rows' select with many workgroups (large K) in place of the one above
    KID_SEL_HIST,
    KID_SEL_SPLIT,
    KID_SEL_FINISH,
    KID_VOTE_COUNT,
    KID_MASK_COUNT,
    KID_GATHER,
    // add-drop voting only
    KID_AD_COLLECT,
    KID_AD_CHUNKS,                                // long, dense lists, in place of the one above
    KID_AD_HIST,
    KID_AD_PICK,
    KID_AD_EMIT,
    // random selection only
    KID_RS_KEYS,
    KID_RS_HIST,
    KID_RS_PICK,
    // short vectors only, in place of all the others
    KID_SMALL_ROWS,
    KID_SMALL_MASK,
    KID_COUNT
};
const char* const kKernelNames[KID_COUNT] = {
    "mv_stream_collect", "mv_row_select",        "mv_sel_hist", "mv_sel_split",  "mv_sel_finish", "mv_vote_count",
    "mv_mask_count",     "mv_gather_update",     "mv_ad_collect", "mv_ad_collect_chunks", "mv_ad_hist", "mv_ad_pick",
    "mv_ad_emit",        "mv_rs_keys",           "mv_rs_hist",  "mv_rs_pick",    "mv_small_rows", "mv_small_mask"};

constexpr size_t kAlign = 256;
constexpr int kEventRing = 64;   // steps whose kernel durations stay readable
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Everything that follows from (N, d, K) alone.
struct Plan {
    uint32_t N, K;
    int64_t  d;
    uint32_t n_runs;            // segments of 1024 coordinates per row, however they are shifted, in whole workgroups of 8
    uint32_t stride;            // every stride-th 32-coordinate chunk is sampled
    uint32_t n_sampled_chunks;  // per row
    uint64_t n_sampled;         // sampled coordinates per row
    uint32_t m_target;          // sampled coordinates that must lie at or above the threshold bin
    uint32_t cap;               // candidate list capacity per row
    uint32_t n_vote_blocks;     // workgroups of the mask kernels: blocks of 16384 vote_q coordinates
    uint32_t vote_q;            // quads of 16 vote bytes per thread of the mask kernels (1, 2, 3, 4, 6 or 8)
    uint32_t rs_blocks;         // workgroups of mv_rs_keys: blocks of kVoteBlock coordinates
    uint32_t list_blocks;       // workgroups per row of mv_ad_collect that walk the candidate list
    uint32_t split_blocks;      // workgroups per row of the many-workgroup select
    uint32_t emit_blocks;       // workgroups per row that write the sorted vote list
    uint32_t select_parts;      // workgroups per row of mv_row_select when they also cast the votes
    uint32_t n_spec;            // list entries per thread that mv_row_select fetches ahead of the row's count
    // add-drop voting (only with MV_FLAG_ADD_DROP)
    bool     add_drop;
    uint32_t nwords, nwords_pad;  // 32-bit words of a row's vote bitmap, and padded to a multiple of 4
    uint32_t cap_d;               // capacity of a row's list of removal candidates
    uint32_t bit_blocks;          // workgroups of kBitBlockWords bitmap words per row
    uint32_t collect_threads, collect_blocks;   // of mv_ad_collect: threads per workgroup, workgroups per row for the bitmap
    bool     collect_chunks;      // mv_ad_collect_chunks in its place
    // rows' select with many workgroups: when about 2K candidates are far more than one workgroup keeps in registers
    bool     multi_select;
    uint32_t block_shift;         // its blocks of coordinates: 2^block_shift, at most kCoordBlocks of them
    bool     vote_chunks;         // their votes are counted by mv_vote_count
    uint32_t chunk_shift, n_chunks, chunks_per_wg;   // of mv_vote_count
    uint32_t crowd_least;                            // see CrowdedChunks
    // random selection
    uint32_t rs_cap;              // most coordinates that can hold a vote: min(N K, d)
    size_t   off_rscount, off_rsbits, off_rsblk, off_rslist, off_rslist2;
    // scratch offsets (bytes)
    uint32_t sample_wgs;        // workgroups per row that sample it (the head of the streaming kernel's grid)
    bool     keep_samples;      // several sampling workgroups store what they read
    uint32_t crowded;           // samples in tau's bin or above it beyond which tau is placed inside the bin
    uint64_t vector_bytes;      // gradients and errors
    uint64_t through_most;      // up to so many bytes that a step touches the streaming pass stores past the caches
    uint32_t head_wgs;          // streaming workgroups behind them that wait for the sampling before they load
    size_t off_samples, off_sampledone, off_readsdone, off_taupub, off_poison, off_stepno, off_candcount;
    size_t off_crowd, off_crowdlist;
    size_t off_hist, off_tau, off_rowcnt, off_slow, off_kth, off_tiecut, off_lvlsets, off_runs, off_runtaken,
        off_alist, off_dlist, off_adcount, off_adbits, off_adblk, off_cand, off_votes, off_blockcnt, off_subcnt, off_votethr, off_emitfail,
        off_lookback;
    uint32_t n_zero_words;      // words from off_lvlsets on that a step's first kernel zeroes
    size_t total_bytes;
};

bool config_valid(const mv_config* c)
{
    if (!c) return false;
    if (c->struct_size != sizeof(mv_config)) return false;
    if (c->n_workers < 1 || c->n_workers > 255) return false;
    if (c->d < 1 || c->d > 0x7FFFFFFFll) return false;
    if (c->k < 1 || c->k > c->d) return false;
    if (c->grad_dtype != MV_F32 && c->grad_dtype != MV_BF16) return false;
    if (c->reduce != MV_REDUCE_MEAN && c->reduce != MV_REDUCE_SUM) return false;
    if ((c->flags & ~MV_FLAG_ADD_DROP) != 0) return false;
    if (c->device < 0) return false;
    return true;
}

Plan make_plan(const mv_config* c)
{
    Plan p;
    memset(&p, 0, sizeof p);
    p.N = (uint32_t)c->n_workers;
    p.K = (uint32_t)c->k;
    p.d = c->d;
    const uint64_t per_wg = (uint64_t)mvk::kSeg * mvk::kSegPerBlock;
    p.n_runs = (uint32_t)(((uint64_t)p.d + mvk::kMostShift + per_wg - 1) / per_wg * mvk::kSegPerBlock);

    // A row with exactly K coordinates above the threshold shows K * frac of them in a sample of frac * d
    // coordinates on average.  Ask for m sampled ones with m - 7 sqrt(m) = K * frac, never fewer than 128:
    // falling short of K is then a 7-sigma event of the sample count, and the candidates exceed K by about
    // 7 sqrt(m) / frac (a factor 2 at K = d/1000, 1.3 at d/100).
    auto sampled_above = [&](double frac) {
        const double root_m = 3.5 + sqrt(12.25 + (double)p.K * frac), m = ceil(root_m * root_m);
        return m < 128.0 ? 128.0 : m;
    };
    // list entries to be ready for when so many are expected
    auto with_room = [](double expected) { return expected * 1.25 + 1.0; };
    // Sample about d/128 coordinates of each row, at least 32K and at most the 128K that 16 workgroups take in one
    // round (kSampleQuads quads per thread: the first row's stream waits for every further round, and scattered lines
    // cost the memory more than a longer list does; d/128 everywhere : so, 1 x 200 M, K = 200,000 626 : 602 us, 1 x 50
    // M 178.3 : 172.5, 3 x 25.6 M 206.1 : 203.3, 32 x 25.6 M bf16 1368.5 : 1366.0, 16 of them with add-drop 760.9 :
    // 757.4; 96K at most 1363.8 and 755.2 there, but 24 x 20 M bf16, K = 6000 803.0 : 807.0) -- or, where the list does
    // not grow too long for it, 8K by ONE workgroup in one round, whose histogram need not be merged in memory: the
    // step of a short row waits for the estimate.  The line follows the lists, one workgroup's against several's (steps
    // of 2, 4 and 16 rows, time with several : time with one):
    //   up to 8192 entries, whatever the others':   2.7K for 0.9K 1.04 1.04 1.02; 6.3K for 1.6K 1.04 1.04 0.99;
    //                        beyond it, at four times theirs:   14K for 3.5K 0.92 0.90 0.93
    //   up to half as long again, as far as mv_row_select serves them: 20K for 13K 1.05 1.03 1.02; 25K for 17K 1.07 1.03
    //                        1.02; beyond, where several workgroups have to select: 27K for 20K 1.08 1.02 1.04, but
    //                        with 40 rows and add-drop voting 0.90
    const uint64_t nchunks = (uint64_t)(p.d + mvk::kChunk - 1) / mvk::kChunk;
    const uint64_t per_round = (uint64_t)mvk::kSampleQuads * mvk::kStreamThreads;      // quads
    // More than a round where the list would take more than a quarter of its storage otherwise (fewer than a few
    // thousand of tens of millions: 128 sampled ones stand for 128 d / 131,072 entries).
    uint64_t cap = 16ull * p.K;
    if (cap < 65536) cap = 65536;
    if (cap > (uint64_t)p.d) cap = (uint64_t)p.d;
    uint64_t want = (uint64_t)p.d / 128 > 32768 ? (uint64_t)p.d / 128 : 32768;
    uint64_t most_sampled = 4 * per_round * mvk::kSampleWgs;
    while (most_sampled < want) {
        const double frac = (double)most_sampled / (double)p.d;
        if (sampled_above(frac) / frac <= 0.25 * (double)cap) break;
        most_sampled *= 2;
    }
    if (want > most_sampled) want = most_sampled;
    const double one = 4.0 * (double)per_round / (double)p.d, many = (double)want / (double)p.d;   // fractions
    const double list_one = sampled_above(one) / one, list_many = sampled_above(many) / many;
    uint64_t stride;
    if (list_one <= 8192.0 || (list_one <= 1.5 * list_many && with_room(list_one) <= (double)mvk::kKeepMost * mvk::kRowThreads)) {
        const uint64_t chunks = per_round / (mvk::kChunk / 4);
        stride = (nchunks + chunks - 1) / chunks;
        p.sample_wgs = 1;
    } else {
        const uint64_t chunks = (want + mvk::kChunk - 1) / mvk::kChunk;
        stride = nchunks / chunks;
        if (stride < 1) stride = 1;
        if (stride > 128) stride = 128;
        const uint64_t most = most_sampled / mvk::kChunk;
        if ((nchunks + stride - 1) / stride > most) stride = (nchunks + most - 1) / most;
        const uint64_t bx = ((nchunks + stride - 1) / stride * (mvk::kChunk / 4) + per_round - 1) / per_round;
        p.sample_wgs = (uint32_t)(bx > mvk::kSampleWgs ? mvk::kSampleWgs : bx);
    }
    // Loads of the grid's head beside the sampling bring a short grid's data earlier and the estimate later.  One
    // sampling workgroup per row has little to fetch: no loads are held back (7 x 272,475 bf16: 33.7 -> 33.0 us;
    // 4 x 2^20, K = 10,486: 49.9 -> 48.9; 40 x 1,000,003, K = 10,000: 132.7 -> 131.9).  Several do better with the
    // memory to themselves, in any grid: two rounds of resident workgroups (of four to a unit) wait (2 x 1,000,003,
    // K = 1000: 35.4 us, 36.3 if none did; 4 x 1,500,003: 44.5 and 47.0; 16 x 2,000,003: 97.5 and 99.3; 3 x 25.6 M:
    // 217.0 and 219.3).
    p.head_wgs = p.sample_wgs == 1 ? 0 : 2048;
    // Where a step's vectors lie in the last-level cache (256 MB), stores past the dies' L2s spare the kernel's end the
    // writing back of what they left there.  The line follows the bytes of gradients and errors and of what the step
    // touches beside them: the votes and their copy, in random selection the votes once more (they are read twice) and
    // the clocks' lines that it needs (enqueue_step).  Steps on three sets of inputs in turn, with those bytes (MiB) and
    // the time written back : past the caches; first with scratch and outputs of their own, then shared.
    //   fp32: 10 x 2.3 M 181: 79.7 78.5, 79.2 77.3; 4 x 5.8 M 182: 102.2 100.6, 83.2 79.7; 2 x 10.9 M 188: 88.5 89.3, 86.7
    //   83.9; 30 x 0.85 M 197: 102.3 104.6, 80.3 81.5; 1 x 20.6 M 197: 115.4 119.0, 114.5 111.8; 894 MB 332 360.
    //   bf16: 10 x 2.25 M 133: 93.0 91.8, 73.7 71.4; 4 x 5.6 M 139: 78.7 79.0, 80.5 78.1; 30 x 0.8 M 140: 71.0 71.0, 77.8
    //   76.8; 4 x 6 M 144: 87.8 88.6, 76.1 74.0; 30 x 0.86 M 149: 94.7 96.7, 82.9 83.7; 216 MB 112 116.
    //   Random selection: 10 x 2.2 M 181: 110.8 112.3; 10 x 2.2 M 179: 95.5 94.6, 95.2 93.0; 1 x 17.5 M 184: 97.3 101.7,
    //   102.0 98.3; 1 x 20.6 M 218: 112.3 119.2; bf16 10 x 2.1 M 128: 84.6 83.2, 133: 89.7 87.5; 30 x 0.8 M 144: 86.5 89.4, 86.2
    //   88.0.
    // Over 560 steps around the line this rule is 0.1 and 0.4 % from the better of the two; one by the bytes of the
    // vectors alone 0.7 and 0.6; one with all of the clocks, 160 MiB and, in bf16, 128 0.3 and 1.0 (4 x 5.8 M bf16 75.1 ->
    // 77.5, with add-drop 121.9 -> 125.6, random selection 1 x 12.5 M 92.3 -> 96.1).
    p.vector_bytes = (uint64_t)p.N * (uint64_t)p.d * (c->grad_dtype == MV_BF16 ? 6 : 8);
    p.through_most = (c->grad_dtype == MV_BF16 ? 140ull : 184ull) << 20;
    // With few workers the mask is nearly what each of them asked for, every coordinate grows until it is sent, and
    // the magnitudes pile up below the K-th: there several sampling workgroups keep their samples.  That costs every such
    // step a little (2 x 1,000,003 0.3 us of 35.4, 2 x 9 M 0.7 of 88.3, 1 x 16 M 1.1 of 90.1, 3 x 25.6 M 1.6 of 217) and
    // spares a long run on the same gradients lists that overflow, at 0.1 ms per million coordinates of the row.  With
    // more workers the residuals spread: over four thousand steps on the same normal gradients lists of 5 to 32 rows grew
    // from 2 to 5 K entries to at most 7 K of the 16 K that fit, and keeping the samples would only cost the step
    // (10 x 11.2 M: 1.4 us, 32 x 25.6 M 9).  Values on a lattice can overflow there after some thousand steps.
    p.keep_samples = p.sample_wgs > 1 && p.N <= 4;
    p.stride = (uint32_t)stride;
    p.n_sampled_chunks = (uint32_t)((nchunks + stride - 1) / stride);
    // all sampled chunks are full except possibly the row's last chunk
    p.n_sampled = (uint64_t)p.n_sampled_chunks * mvk::kChunk;
    if (((nchunks - 1) % stride) == 0) p.n_sampled -= (uint64_t)(nchunks * mvk::kChunk - (uint64_t)p.d);

    const double frac = (double)p.n_sampled / (double)p.d;
    const double m = sampled_above(frac) + 1.0;
    p.m_target = (m >= 4294967295.0) ? 0xFFFFFFFFu : (uint32_t)m;

    p.cap = (uint32_t)cap;
    {
        // A crowded bin makes the list longer than it has to be, and the search inside it holds the row's stream up:
        // it is made where the list would be twice as long (one sampling workgroup, whose samples are at hand) or three
        // times (several, whose samples one has to fetch: up to 32,768 quads of them; K = d / 1000, lists of 6K to 8K
        // entries kept : searched: 1 x 8 M 86.3 us 73.0; 1 x 14 M 100.8 99.9), and in longer rows only where the list nears
        // its storage.  (Samples that grew with the row made the search the slower way there.  With those of one round it
        // gains, after thousands of steps on the same gradients: 1 x 25 M 140.4 : 132.9, 2 x 20 M bf16 171.3 : 152.0,
        // 1 x 200 M 586.0 : 558.7.)
        const bool long_row = (uint64_t)p.d > 128ull * 4 * per_round * mvk::kSampleWgs;
        double most = p.sample_wgs == 1 ? 2.0 * m : 3.0 * m;
        if (long_row && 0.875 * (double)p.cap * frac > most) most = 0.875 * (double)p.cap * frac;
        p.crowded = (p.sample_wgs > 1 && !p.keep_samples) || most >= 4294967295.0 ? 0xFFFFFFFFu : (uint32_t)most;
    }

    p.rs_blocks = (uint32_t)((p.d + mvk::kVoteBlock - 1) / mvk::kVoteBlock);
    {
        // the mask kernels: as few vote bytes per thread as keep the vote blocks at two workgroups per compute unit, all
        // resident at once, which the exchange of counts between the blocks likes (a limit of 500 beats 250 by 3 us
        // on 16 x 11.2 M and by 13 on 32 x 25.6 M; 750 and more lose again on d = 11 M), and leave some units to the
        // lists' workgroups, which come behind them in the grid
        static const uint32_t kQs[] = {1, 2, 3, 4, 6, 8};
        uint32_t q = 8;
        for (uint32_t cand_q : kQs)
            if ((uint64_t)p.d <= (uint64_t)(500 - (p.N < 128 ? p.N : 128)) * mvk::kMaskThreads * 16 * cand_q) {
                q = cand_q;
                break;
            }
        p.vote_q = q;
        const uint64_t per = (uint64_t)mvk::kMaskThreads * 16 * q;
        p.n_vote_blocks = (uint32_t)(((uint64_t)p.d + per - 1) / per);
    }
    {
        // about 2K candidates are expected; fetch 3K per row ahead (never beyond the list's storage),
        // and give every workgroup of a row about four list entries per thread to cast votes for
        const uint64_t expect = (uint64_t)with_room((double)p.m_target / frac);      // candidates per row
        uint64_t slots = (expect + mvk::kRowThreads - 1) / mvk::kRowThreads;        // list entries per thread
        const uint64_t in_cap = ((uint64_t)p.cap + mvk::kRowThreads - 1) / mvk::kRowThreads;
        if (slots > in_cap) slots = in_cap;
        if (slots < 1) slots = 1;
        p.n_spec = (uint32_t)(slots < (uint64_t)mvk::kKeepMost ? slots : (uint64_t)mvk::kKeepMost);
        uint64_t parts = (slots + 3) / 4;
        if (parts > 16) parts = 16;
        if (parts * p.N > 240) parts = 240 / p.N;      // all at once: with its registers a workgroup has a unit to itself
        if (parts < 1) parts = 1;
        p.select_parts = (uint32_t)parts;
        // beyond what one workgroup keeps in registers the lists go through the many-workgroup select
        p.multi_select = slots > (uint64_t)mvk::kKeepMost;
        p.block_shift = 10;                       // a segment at least
        while (((p.d - 1 + mvk::kMostShift) >> p.block_shift) >= mvk::kCoordBlocks) ++p.block_shift;
        // mv_vote_count: chunks of 4096 coordinates (a chunk shares a segment with the next one: of 2048, 10 x 11.2 M,
        // K = 111,740 takes 17.0 us for 14.7 and 32 x 25.6 M 24.5 for 20.2), shorter ones where those are fewer than
        // the chip's units; as many to a workgroup as leave four workgroups to a unit (three there 14.7 us, two 16.0,
        // one 20.2; at 32 x 25.6 M six 20.2, four 21.8, two 24.5), and as LDS and the runs have room for
        static_assert(204 * 5 <= mvk::kVotesRunsMost && 255 * 3 <= mvk::kVotesRunsMost, "the runs of a chunk of 4096, of 2048");
        p.chunk_shift = p.d >= (1 << 20) && p.N <= 204 ? 12 : p.d >= (1 << 19) ? 11 : 10;
        p.n_chunks = (uint32_t)((p.d - 1) >> p.chunk_shift) + 1;
        const uint32_t of_chunk = (1u << p.chunk_shift) / mvk::kSeg + 1;    // segments
        uint32_t most = (uint32_t)mvk::kVotesBytesMost >> p.chunk_shift;
        if (most > mvk::kVotesRunsMost / (p.N * of_chunk)) most = mvk::kVotesRunsMost / (p.N * of_chunk);
        p.chunks_per_wg = (p.n_chunks + 1023) / 1024;
        if (p.chunks_per_wg > most) p.chunks_per_wg = most;
        p.crowd_least = mvk::kCrowdedEntries / (2 * p.N);
        {
            // Counted so, the votes cost a launch more and no atomics: worth it from half a million votes on, where the
            // list entries of a workgroup's chunks, those it shares among them, are not too many.  Steps with the votes
            // cast from the lists : counted in chunks: 16 x 6 M, K = 40,000 258.2 : 250.8 us; 24 x 3 M, K = 30,000
            // 210.4 : 205.9; 4 x 10 M on a lattice, K = 300,000 177.9 : 170.3; random selection 10 x 11.2 M, K =
            // 111,740 345.6 : 335.5; 20 x 2 M, K = 40,000 from a zero buffer (2.7 K entries) 153 : 150; fewer votes:
            // random selection 12 x 2 M, K = 33,333 114.7 : 117.0, 2 x 10 M, K = 150,000 117.3 : 119.8.  With more
            // entries either may be faster, with carried errors and from a zero buffer: 40 x 1 M, K = 25,000 (3.9 K)
            // 157 : 152 and 147 : 155; 64 x 2 M, K = 22,000 (5.2 K) 376 : 362 and 354 : 370; 2 x 2 M, K = 10^6 (5.4 K)
            // 110 : 101 and 121 : 111; 20 x 300,001, K = 30,000 (4.6 K) 61.1 : 64.9; 50 x 400,003, K = 40,000 (12 K)
            // 136 : 138; 8 x 600,000, K = 300,000 (13 K) 117 : 108; 100 x 200,000, K = 30,000 (34 K) 163 : 183.
            // The gain is that of steps with carried errors.  From a zero buffer, where votes share atomics, and of fewer
            // than about three workgroups to a unit the counted votes can be the slower ones; with carried errors and from
            // a zero buffer: 10 x 2.5 M, K = 100,000 133 : 128.5 and 123 : 129.5; 33 x 2.2 M, K = 20,000 218 : 212 and
            // 213 : 220; 20 x 4 M, K = 27,000 221 : 217 and 220 : 226; 8 x 2 M, K = 80,000 95.6 : 94.0 and 88 : 98;
            // 4 x 2 M, K = 200,000 78.7 : 80.5 and 84 : 91; 5 x 2^20, K = 100,000 61.6 : 63.3 and 67 : 72; from 3 M
            // coordinates and 600,000 votes on 6 x 6 M, K = 150,000 160 : 153 and 150 : 152; 20 x 5 M, K = 50,000
            // 292 : 280 and 280 : 279; 40 x 4 M, K = 20,000 396 : 386 and 402 : 402.
            const double wgs = (double)((p.n_chunks + p.chunks_per_wg - 1) / p.chunks_per_wg);
            const double entries = (double)p.N * (double)p.m_target / frac * (double)of_chunk / (double)(of_chunk - 1) / wgs;
            p.vote_chunks = p.multi_select && (uint64_t)p.N * p.K >= 500000 && entries <= 3000.0;
        }
        // one batch of list entries per thread in the many-workgroup select, two when writing the sorted lists
        uint64_t sb = (slots + mvk::kListUnroll - 1) / mvk::kListUnroll, eb2 = (slots + 3) / 4;
        if (sb > 256) sb = 256;
        if (eb2 * p.N > 512) eb2 = 512 / p.N;      // (10 x 11.2 M, K = 111,740: 346.7 us, with 256 349.6)
        if (eb2 < 1) eb2 = 1;
        p.split_blocks = (uint32_t)sb;
        // likewise in mv_ad_collect (a row's bitmap in one workgroup of more threads, where it fits), which goes by
        // chunks of coordinates where lists are long and dense and a workgroup's chunks hold not too many entries of
        // them (steps with candidates looked up one by one : by chunks; 2 x 4 M, K = 400,000 (9 K entries to a
        // workgroup) 162 : 140; 8 x 1.5 M, K = 200,000 (12 K) 195 : 174; 4 x 3 M, K = 450,000 (14 K) 220 : 192; 16 x
        // 600,000, K = 100,000 (14 K) 172 : 162; 2 x 1.5 M, K = 300,000 (18 K) 177 : 149; 32 x 131,000, K = 50,000 (33
        // K) 193 : 185; sparser: 16 x 11.2 M, K = 30,000 452 : 456, 32 x 25.6 M bf16, K = 25,557 1459 : 1487; fuller,
        // either: 40 x 65,536, K = 25,000 (33 K) 135 : 154, 2 x 2 M, K = 800,000 (34 K) 242 : 221, 100 x 60,003, K =
        // 30,000 (39 K) 249 : 289)
        const uint64_t per_wg = 32ull * mvk::collect_words(mvk::kCollectThreads);
        p.collect_chunks = p.multi_select && 256ull * p.K >= (uint64_t)p.d &&
                           expect <= 25000 * (((uint64_t)p.d + per_wg - 1) / per_wg);
        const bool one = !p.collect_chunks && (uint64_t)p.d <= 32ull * mvk::collect_words(mvk::kCollectThreadsShort);
        p.collect_threads = one ? mvk::kCollectThreadsShort : mvk::kCollectThreads;
        const uint64_t batch = mvk::add_batch((int)p.collect_threads);
        uint64_t lb = (expect + batch - 1) / batch;
        if (lb > 256) lb = 256;
        p.list_blocks = (uint32_t)lb;
        p.emit_blocks = (uint32_t)eb2;
    }

    size_t off = 0;
    p.off_hist = off;     off += align_up((size_t)p.N * mvk::kHistBins * 4);
    p.off_tau = off;      off += align_up((size_t)p.N * 4);
    p.off_sampledone = off; off += align_up((size_t)p.N * mvk::kCounterStride * 4);
    p.off_readsdone = off; off += align_up((size_t)p.N * mvk::kCounterStride * 4);
    p.off_taupub = off;   off += align_up((size_t)p.N * (mvk::kCounterStride / 2) * 8);
    p.off_poison = off;   off += align_up((size_t)p.N * 4);
    p.off_stepno = off;   off += align_up(4);
    p.off_candcount = off; off += align_up((size_t)p.N * 4);
    p.off_rowcnt = off;   off += 2 * align_up((size_t)p.N * mvk::kCounterStride * 4);   // one set per step parity
    p.off_slow = off;     off += align_up((size_t)p.N * 4);
    p.off_kth = off;      off += align_up((size_t)p.N * 4);
    p.off_tiecut = off;   off += align_up((size_t)p.N * 4);
    // the vote-level counters and, behind them, what mv_mask_count's blocks publish to each other (a flag word
    // and two 64-bit words per block): one stretch of words that every step's first kernel leaves at zero
    p.off_lvlsets = off;  off += (size_t)mvk::kLvlSets * 256 * 4;
    p.off_emitfail = off; off += 8;
    // (and how many chunks are crowded, in two words, and their list entries)
    p.off_crowd = off;    off += 8 + (p.vote_chunks ? ((size_t)p.n_chunks + 1) / 2 * 8 : 0);
    p.off_lookback = off; off += (size_t)p.n_vote_blocks * 16;
    // (and the counts per block of the winners of the random selection and of the additions and removals)
    p.add_drop = (c->flags & MV_FLAG_ADD_DROP) != 0;
    p.nwords = (uint32_t)((p.d + 31) / 32);
    p.nwords_pad = (p.nwords + 3) / 4 * 4;
    p.cap_d = p.K;
    const uint32_t stretch = mvk::collect_words((int)p.collect_threads);
    p.collect_blocks = (p.nwords_pad + stretch - 1) / stretch;
    p.bit_blocks = (p.nwords_pad + mvk::kBitBlockWords - 1) / mvk::kBitBlockWords;
    if (p.add_drop) {
        p.off_adblk = off; off += (size_t)p.N * p.bit_blocks * 8;
    }
    p.off_rsblk = off;    off += align_up((size_t)p.n_vote_blocks * 4);
    p.n_zero_words = (uint32_t)((off - p.off_lvlsets) / 4);
    off = align_up(off);
    p.off_runs = off;     off += align_up((size_t)p.N * p.n_runs * 8);
    if (p.vote_chunks) {
        p.off_crowdlist = off; off += align_up((size_t)p.n_chunks * 4);
    }
    p.off_runtaken = off; off += align_up((size_t)p.N * p.n_runs * 2);
    if (p.keep_samples) {                         // their magnitudes
        p.off_samples = off; off += align_up((size_t)p.N * p.n_sampled_chunks * mvk::kChunk * 4);
    }
    p.off_cand = off;     off += align_up((size_t)p.N * p.cap * 8);
    p.off_votes = off;    off += align_up(((size_t)p.d + 15) / 16 * 16);
    p.off_blockcnt = off; off += align_up((size_t)p.n_vote_blocks * 8);
    p.off_subcnt = off;   off += align_up((size_t)p.n_vote_blocks * (mvk::kMaskThreads / mvk::kWave) * 8);
    p.off_votethr = off;  off += align_up(2 * 4);
    if (p.add_drop) {
        p.off_alist = off;   off += align_up((size_t)p.N * p.cap * 8);
        p.off_dlist = off;   off += align_up((size_t)p.N * p.cap_d * 8);
        p.off_adcount = off; off += align_up((size_t)p.N * 2 * mvk::kCounterStride * 4);
        p.off_adbits = off;  off += align_up((size_t)p.N * p.nwords_pad * 4);
    }
    const uint64_t voted_max = (uint64_t)p.N * p.K;
    p.rs_cap = (uint32_t)(voted_max < (uint64_t)p.d ? voted_max : (uint64_t)p.d);
    p.off_rscount = off; off += align_up(4);
    p.off_rsbits = off;  off += align_up((size_t)p.nwords_pad * 4);
    p.off_rslist = off;  off += align_up((size_t)p.rs_cap * 8);
    p.off_rslist2 = off; off += align_up((size_t)p.rs_cap * 8);
    p.total_bytes = off;
    return p;
}

}  // namespace

struct mv_ctx {
    mv_config  cfg;
    Plan       plan;
    char*      ws;          // device scratch
    bool       owns_ws;
    bool       ended;
    bool       broken;      // a step's launch sequence failed: the scratch invariants no longer hold
    int32_t    profiling;
    // event pairs around kernels, a ring over the last kEventRing steps
    hipEvent_t ev[kEventRing][KID_COUNT][2];
    bool       ev_recorded[kEventRing][KID_COUNT];
    uint64_t   steps_done;
    uint32_t   spin_limit;  // polls a streaming wavefront makes for its row's threshold before it gives up
    hipStream_t last_stream;
};

namespace {

template <typename T>
T* ws_ptr(mv_ctx* c, size_t off) { return reinterpret_cast<T*>(c->ws + off); }

struct DeviceGuard {
    int  prev;
    bool ok;
    explicit DeviceGuard(int dev) : prev(0), ok(false)
    {
        if (hipGetDevice(&prev) != hipSuccess) return;
        if (prev != dev && hipSetDevice(dev) != hipSuccess) return;
        ok = true;
    }
    ~DeviceGuard() { if (ok) (void)hipSetDevice(prev); }
};

}  // namespace

extern "C" {

size_t mv_workspace_bytes(const mv_config* cfg)
{
    if (!config_valid(cfg)) return 0;
    return make_plan(cfg).total_bytes;
}

mv_status mv_begin(const mv_config* cfg, mv_ctx** out_ctx)
{
    if (!out_ctx) return MV_ERR_INVALID_ARG;
    *out_ctx = nullptr;
    if (!config_valid(cfg)) return MV_ERR_INVALID_ARG;
    const Plan plan = make_plan(cfg);
    if (cfg->workspace) {
        if (cfg->workspace_bytes < plan.total_bytes) return MV_ERR_INVALID_ARG;
        if ((reinterpret_cast<uintptr_t>(cfg->workspace) & (kAlign - 1)) != 0) return MV_ERR_INVALID_ARG;
    }

    mv_ctx* c = new (std::nothrow) mv_ctx;
    if (!c) return MV_ERR_ALLOC;
    memset(c, 0, sizeof *c);
    c->cfg = *cfg;
    c->plan = plan;
    c->spin_limit = 1u << 20;   // of about a microsecond each; a threshold is normally there within ten

    DeviceGuard guard(cfg->device);
    if (!guard.ok) {
        delete c;
        return MV_ERR_DEVICE;
    }
    if (cfg->workspace) {
        c->ws = static_cast<char*>(cfg->workspace);
        c->owns_ws = false;
    } else {
        void* p = nullptr;
        if (hipMalloc(&p, plan.total_bytes) != hipSuccess) {
            (void)hipGetLastError();
            delete c;
            return MV_ERR_ALLOC;
        }
        c->ws = static_cast<char*>(p);
        c->owns_ws = true;
    }
    // The histogram and the packed vote words must start at zero; the kernels
    // leave them at zero after every step.
    bool ok = hipMemset(c->ws + plan.off_hist, 0, plan.off_tau - plan.off_hist) == hipSuccess &&
              hipMemset(c->ws + plan.off_votes, 0, ((size_t)plan.d + 15) / 16 * 16) == hipSuccess &&
              hipMemset(c->ws + plan.off_tau, 0, plan.off_runs - plan.off_tau) == hipSuccess;
    if (ok && plan.add_drop)   // the scratch bitmaps start at zero and are left at zero by every step
        ok = hipMemset(c->ws + plan.off_adcount, 0,
                       plan.off_adbits - plan.off_adcount + (size_t)plan.N * plan.nwords_pad * 4) == hipSuccess;
    // random selection: the list's length and the bitmap start at zero and are left at zero
    ok = ok && hipMemset(c->ws + plan.off_rscount, 0, plan.off_rslist - plan.off_rscount) == hipSuccess;
    ok = ok && hipDeviceSynchronize() == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        if (c->owns_ws) (void)hipFree(c->ws);
        delete c;
        return MV_ERR_DEVICE;
    }
    *out_ctx = c;
    return MV_OK;
}

}  // extern "C"

namespace {

// What the two step entry points pass down.
struct StepArgs {
    const void* grads; int64_t ld_g;
    float* err;        int64_t ld_e;
    uint32_t* worker_idx;
    uint8_t*  votes;
    uint32_t* mask_idx;
    float*    agg_vals;
    // add-drop voting (k_ad == 0: plain majority voting)
    int64_t   k_ad;
    uint32_t* vote_bits; int64_t ld_bits;
    uint8_t*  msum;
    uint32_t* add_idx;
    uint32_t* drop_idx;
    uint32_t* counts;
    // random selection (null: the mask is the K most voted coordinates)
    const float* rand_exp;
};

mv_status check_common(mv_ctx* c, const StepArgs& a)
{
    if (!c) return MV_ERR_INVALID_ARG;
    if (c->ended || c->broken) return MV_ERR_STATE;
    if (!a.grads || !a.err || !a.mask_idx || !a.agg_vals) return MV_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(a.rand_exp) & 3) return MV_ERR_INVALID_ARG;
    const Plan& p = c->plan;
    const bool bf16 = c->cfg.grad_dtype == MV_BF16;
    if (a.ld_g < p.d || a.ld_e < p.d) return MV_ERR_INVALID_ARG;
    if (a.ld_g % (bf16 ? 8 : 4) != 0 || a.ld_e % 4 != 0) return MV_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(a.grads) & 15) || (reinterpret_cast<uintptr_t>(a.err) & 15))
        return MV_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(a.mask_idx) & 3) || (reinterpret_cast<uintptr_t>(a.agg_vals) & 3) ||
        (reinterpret_cast<uintptr_t>(a.worker_idx) & 3))
        return MV_ERR_INVALID_ARG;
    return MV_OK;
}

// Enqueues one step: the part common to both voting schemes (threshold estimate,
// streaming pass, exact per-row select), then either the plain vote count or the
// add-drop update of the standing votes, then the mask and the aggregate.
mv_status enqueue_step(mv_ctx* c, const StepArgs& a, void* stream_v)
{
    const Plan& p = c->plan;
    const bool bf16 = c->cfg.grad_dtype == MV_BF16;
    const bool add_drop = a.k_ad > 0;
    const bool random_sel = a.rand_exp != nullptr;
    const mvk::RowSegments segs = {(uint32_t)(reinterpret_cast<uintptr_t>(a.err) / 4 % mvk::kSeg),
                                   (uint32_t)((uint64_t)a.ld_e % mvk::kSeg), (uint32_t)p.d};
    DeviceGuard guard(c->cfg.device);
    if (!guard.ok) return MV_ERR_DEVICE;
    // an error the caller left pending is not this step's: nothing is enqueued and the context stays usable
    if (hipPeekAtLastError() != hipSuccess) return MV_ERR_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream_v);

    uint32_t* hist = ws_ptr<uint32_t>(c, p.off_hist);
    uint32_t* tau = ws_ptr<uint32_t>(c, p.off_tau);
    // the rows' candidate counters while the streaming pass runs (two sets, used in turn; the step's
    // number on the device says which), and the counts as mv_row_select leaves them for everyone after it
    const uint32_t rowcnt_set_words = (uint32_t)(align_up((size_t)p.N * mvk::kCounterStride * 4) / 4);
    uint32_t* rowcnt_sets = ws_ptr<uint32_t>(c, p.off_rowcnt);
    uint32_t* stepno = ws_ptr<uint32_t>(c, p.off_stepno);
    uint32_t* rowcnt = ws_ptr<uint32_t>(c, p.off_candcount);
    uint32_t* slow = ws_ptr<uint32_t>(c, p.off_slow);
    uint32_t* lvlsets = ws_ptr<uint32_t>(c, p.off_lvlsets);
    uint32_t* kth = ws_ptr<uint32_t>(c, p.off_kth);
    uint32_t* tiecut = ws_ptr<uint32_t>(c, p.off_tiecut);
    mvk::u32x2* runs = ws_ptr<mvk::u32x2>(c, p.off_runs);
    uint32_t* run_taken = ws_ptr<uint32_t>(c, p.off_runtaken);
    mvk::u32x2* cand = ws_ptr<mvk::u32x2>(c, p.off_cand);
    uint32_t* votes32 = ws_ptr<uint32_t>(c, p.off_votes);
    mvk::u32x2* blockcnt = ws_ptr<mvk::u32x2>(c, p.off_blockcnt);
    uint32_t* rsblk = ws_ptr<uint32_t>(c, p.off_rsblk);
    mvk::u32x2* subcnt = ws_ptr<mvk::u32x2>(c, p.off_subcnt);
    uint32_t* emitfail = ws_ptr<uint32_t>(c, p.off_emitfail);
    unsigned long long* lookback = ws_ptr<unsigned long long>(c, p.off_lookback);
    uint32_t* votethr = ws_ptr<uint32_t>(c, p.off_votethr);
    mvk::u32x2* alist = p.add_drop ? ws_ptr<mvk::u32x2>(c, p.off_alist) : nullptr;
    mvk::u32x2* dlist = p.add_drop ? ws_ptr<mvk::u32x2>(c, p.off_dlist) : nullptr;
    uint32_t* adcount = p.add_drop ? ws_ptr<uint32_t>(c, p.off_adcount) : nullptr;
    uint32_t* adbits = p.add_drop ? ws_ptr<uint32_t>(c, p.off_adbits) : nullptr;
    mvk::u32x2* adblk = p.add_drop ? ws_ptr<mvk::u32x2>(c, p.off_adblk) : nullptr;

    const int slot = (int)(c->steps_done % kEventRing);
    for (int i = 0; i < KID_COUNT; ++i) c->ev_recorded[slot][i] = false;
    const int prof = c->profiling;
    bool ev_ok = true;
    auto wanted = [&](int kid) { return prof >= 2 || (prof == 1 && (kid == KID_STREAM || kid == KID_SMALL_ROWS)); };
    auto before = [&](int kid) {
        if (!wanted(kid)) return;
        for (int j = 0; j < 2; ++j)   // events are created on first use
            if (!c->ev[slot][kid][j] && hipEventCreate(&c->ev[slot][kid][j]) != hipSuccess) ev_ok = false;
        if (ev_ok && hipEventRecord(c->ev[slot][kid][0], st) != hipSuccess) ev_ok = false;
    };
    auto after = [&](int kid) {
        if (!wanted(kid) || !ev_ok) return;
        if (hipEventRecord(c->ev[slot][kid][1], st) == hipSuccess) c->ev_recorded[slot][kid] = true;
    };

    // the step ends here: nothing was left out, or the context is given up
    auto finish = [&]() {
        c->last_stream = st;
        c->steps_done += 1;
        if (hipGetLastError() != hipSuccess) {
            // Some kernel of the sequence was not launched: counters that every step leaves at zero, and the
            // step's number on the device, may be off.  The context refuses further steps.
            c->broken = true;
            return MV_ERR_DEVICE;
        }
        return ev_ok ? MV_OK : MV_ERR_DEVICE;
    };

    // Short vectors: two launches for any scheme.  (Every step of a context takes the same way, so the two
    // ways' scratch need not agree: the rows' bitmaps lie where long vectors have their candidate lists.)
    if (p.d <= mvk::kSmallMaxD) {
        const uint32_t d = (uint32_t)p.d;
        uint32_t* row_bits = ws_ptr<uint32_t>(c, p.off_cand);
        mvk::SmallAddDrop ad;
        memset(&ad, 0, sizeof ad);
        if (add_drop) {
            ad.vote_bits = a.vote_bits;  ad.ld_bits = a.ld_bits;
            ad.msum32 = reinterpret_cast<uint32_t*>(a.msum);
            ad.k_ad = (uint32_t)a.k_ad;  ad.add_idx = a.add_idx;  ad.drop_idx = a.drop_idx;  ad.counts = a.counts;
        }
        before(KID_SMALL_ROWS);
#define MV_LAUNCH_SMALL_ROWS(GT, U)                                                                              \
        hipLaunchKernelGGL((mvk::mv_small_rows<GT, U>), dim3(p.N), dim3(mvk::kSmallThreads), 0, st,               \
                           static_cast<const GT*>(a.grads), a.ld_g, a.err, a.ld_e, d, p.K,                        \
                           add_drop ? (uint32_t*)nullptr : a.worker_idx, row_bits, p.nwords, rowcnt, tau, slow, ad)
        const uint32_t quads = (d + 4 * mvk::kSmallThreads - 1) / (4 * mvk::kSmallThreads);   // per thread
        if (bf16) {
            if (quads <= 1) MV_LAUNCH_SMALL_ROWS(uint16_t, 1);
            else if (quads <= 2) MV_LAUNCH_SMALL_ROWS(uint16_t, 2);
            else if (quads <= 4) MV_LAUNCH_SMALL_ROWS(uint16_t, 4);
            else MV_LAUNCH_SMALL_ROWS(uint16_t, 8);
        } else {
            if (quads <= 1) MV_LAUNCH_SMALL_ROWS(float, 1);
            else if (quads <= 2) MV_LAUNCH_SMALL_ROWS(float, 2);
            else if (quads <= 4) MV_LAUNCH_SMALL_ROWS(float, 4);
            else MV_LAUNCH_SMALL_ROWS(float, 8);
        }
#undef MV_LAUNCH_SMALL_ROWS
        after(KID_SMALL_ROWS);
        // every workgroup finds the whole mask again: one round of positions each while that keeps them within
        // one per compute unit
        const uint32_t kb = mvk::kSmallThreads / p.N;
        uint32_t rounds = (p.K + kb * 256 - 1) / (kb * 256);
        if (rounds > (uint32_t)mvk::kGatherRounds) rounds = mvk::kGatherRounds;
        before(KID_SMALL_MASK);
        auto* mask_kernel = random_sel ? &mvk::mv_small_mask<true> : &mvk::mv_small_mask<false>;
        hipLaunchKernelGGL(mask_kernel, dim3((p.K + kb * rounds - 1) / (kb * rounds)),
                           dim3(mvk::kSmallThreads), 0, st, a.err, a.ld_e, d, p.N, p.K, (const uint32_t*)row_bits,
                           p.nwords, (const uint32_t*)ad.msum32, a.rand_exp, add_drop ? (uint8_t*)nullptr : a.votes,
                           a.mask_idx, 1.0f / (float)p.N, c->cfg.reduce == MV_REDUCE_MEAN ? 1 : 0, a.agg_vals, rounds);
        after(KID_SMALL_MASK);
        return finish();
    }

    // 1. one kernel: sample histogram and threshold estimate per row (its first workgroups, which
    // also reset the per-step counters), and the streaming pass a = g + e over e, candidates out
    uint32_t* sampledone = ws_ptr<uint32_t>(c, p.off_sampledone);
    uint32_t* readsdone = ws_ptr<uint32_t>(c, p.off_readsdone);
    uint64_t step_bytes = p.vector_bytes;         // what the step touches: see make_plan
    if (!add_drop) step_bytes += (a.votes ? 2ull : 1ull) * (uint64_t)p.d;
    if (random_sel) {
        const uint64_t lines = 128ull * p.N * p.K, clocks = 4ull * (uint64_t)p.d;
        step_bytes += (uint64_t)p.d + (lines < clocks ? lines : clocks);
    }
    const int through = step_bytes <= p.through_most ? 1 : 0;
    uint32_t* samples = p.keep_samples ? ws_ptr<uint32_t>(c, p.off_samples) : nullptr;
    unsigned long long* taupub = ws_ptr<unsigned long long>(c, p.off_taupub);
    uint32_t* poison = ws_ptr<uint32_t>(c, p.off_poison);
    {
        uint32_t* zero_votes = add_drop || p.vote_chunks ? nullptr : votes32;     // (mv_vote_count writes all of them)
        const dim3 grid(p.N * p.sample_wgs + p.N * (p.n_runs / mvk::kSegPerBlock));
        before(KID_STREAM);
        if (bf16)
            hipLaunchKernelGGL(mvk::mv_stream_collect<uint16_t>, grid, dim3(mvk::kStreamThreads), 0, st,
                               static_cast<const uint16_t*>(a.grads), a.ld_g, a.err, a.ld_e, p.d, p.N, p.sample_wgs,
                               p.stride, p.n_sampled_chunks, p.m_target, p.crowded, hist, sampledone, readsdone, taupub, stepno,
                               c->spin_limit, poison, lvlsets, p.n_zero_words, adcount, samples, cand, p.cap,
                               rowcnt_sets, rowcnt_set_words, runs, run_taken, p.n_runs, segs, p.head_wgs, through,
                               zero_votes, (int64_t)(((size_t)p.d + 15) / 16 * 16));
        else
            hipLaunchKernelGGL(mvk::mv_stream_collect<float>, grid, dim3(mvk::kStreamThreads), 0, st,
                               static_cast<const float*>(a.grads), a.ld_g, a.err, a.ld_e, p.d, p.N, p.sample_wgs,
                               p.stride, p.n_sampled_chunks, p.m_target, p.crowded, hist, sampledone, readsdone, taupub, stepno,
                               c->spin_limit, poison, lvlsets, p.n_zero_words, adcount, samples, cand, p.cap,
                               rowcnt_sets, rowcnt_set_words, runs, run_taken, p.n_runs, segs, p.head_wgs, through,
                               zero_votes, (int64_t)(((size_t)p.d + 15) / 16 * 16));
        after(KID_STREAM);
    }
    // 2. exact per-row select; in plain voting and random selection the votes are cast in the same launch (short
    // lists: every workgroup of a row casts those of its share; long lists: many workgroups per row)
    const bool sorted = a.worker_idx != nullptr;
    uint32_t* tallies = sorted ? run_taken : nullptr;
    const int thresholds_only = add_drop ? 1 : 0;
    // (the runs are put in order for the kernels that go through them by chunks of coordinates)
    const bool in_order = add_drop ? p.collect_chunks : p.vote_chunks;
    if (p.multi_select) {
        before(KID_SEL_HIST);
        hipLaunchKernelGGL(mvk::mv_sel_hist, dim3(p.split_blocks, p.N), dim3(mvk::kRowThreads), 0, st, cand, p.cap, p.K,
                           rowcnt_sets, rowcnt_set_words, stepno, taupub, poison, hist, rowcnt, tau, slow);
        after(KID_SEL_HIST);
        before(KID_SEL_SPLIT);
        const bool cast_here = !add_drop && !p.vote_chunks;
        uint32_t* n_crowded = ws_ptr<uint32_t>(c, p.off_crowd);
        const mvk::CrowdedChunks crowd = {n_crowded, !add_drop && p.vote_chunks ? n_crowded + 2 : nullptr,
                                          ws_ptr<uint32_t>(c, p.off_crowdlist), p.n_chunks, p.chunk_shift, p.crowd_least};
        const uint32_t order_blocks = in_order ? (p.n_runs + mvk::kOrderRuns - 1) / mvk::kOrderRuns : 0;
        hipLaunchKernelGGL((cast_here ? &mvk::mv_sel_split<true> : &mvk::mv_sel_split<false>),
                           dim3(p.split_blocks + order_blocks, p.N), dim3(mvk::kRowThreads), 0, st, a.err, a.ld_e, p.d,
                           cand, p.cap, p.K, (const uint32_t*)rowcnt, (const uint32_t*)tau, (const uint32_t*)slow, hist,
                           kth, tiecut, a.worker_idx, votes32, tallies, runs, p.n_runs, segs, lvlsets, taupub,
                           p.block_shift, p.split_blocks, crowd);
        after(KID_SEL_SPLIT);
        uint32_t parts = cast_here ? 256 / p.N : 1;
        parts = parts > 16 ? 16 : parts < 1 ? 1 : parts;
        before(KID_SEL_FINISH);
        hipLaunchKernelGGL((cast_here ? &mvk::mv_sel_finish<true> : &mvk::mv_sel_finish<false>), dim3(parts, p.N),
                           dim3(mvk::kRowThreads), 0, st, cand, p.cap, p.K,
                           (const uint32_t*)rowcnt, (const uint32_t*)tau, (const uint32_t*)slow, hist, kth, tiecut,
                           votes32, tallies, p.n_runs, segs, lvlsets, taupub, (const mvk::u32x2*)runs, in_order ? 1 : 0,
                           p.block_shift);
        after(KID_SEL_FINISH);
        if (!add_drop && p.vote_chunks) {
            before(KID_VOTE_COUNT);
            hipLaunchKernelGGL(mvk::mv_vote_count, dim3((p.n_chunks + p.chunks_per_wg - 1) / p.chunks_per_wg),
                               dim3(mvk::kVotesThreads), 0, st, (const float*)a.err, a.ld_e, p.d, p.N,
                               (const mvk::u32x2*)cand, p.cap, (const mvk::u32x2*)runs, p.n_runs, segs,
                               (const uint32_t*)kth, (const uint32_t*)tiecut, (const uint32_t*)slow, crowd,
                               p.chunks_per_wg, votes32, reinterpret_cast<uint16_t*>(tallies), lvlsets);
            after(KID_VOTE_COUNT);
        }
    } else {
        const uint32_t parts = add_drop ? 1 : p.select_parts;
        before(KID_ROW_SELECT);
        auto* kernel = p.n_spec <= 8 ? &mvk::mv_row_select<8> : p.n_spec <= 16 ? &mvk::mv_row_select<16>
                                                                               : &mvk::mv_row_select<mvk::kKeepMost>;
        hipLaunchKernelGGL(kernel, dim3((p.N + 7) / 8 * 8 * parts), dim3(mvk::kRowThreads), 0, st, a.err,
                           a.ld_e, p.d, p.N, p.K, cand, p.cap, rowcnt_sets, rowcnt_set_words, stepno, taupub, poison,
                           rowcnt, tau, kth, tiecut, a.worker_idx, votes32, tallies, p.n_runs, segs, lvlsets, slow, parts,
                           p.n_spec, thresholds_only);
        after(KID_ROW_SELECT);
    }

    uint32_t* mask_votes32 = votes32;     // the packed vote bytes the mask is selected from
    if (add_drop) {
        // 3'. add-drop voting: candidates for addition and removal, exact K_ad-selects with the update of msum,
        // then the sorted add / drop lists, the standing votes and the levels of msum
        const uint32_t k_ad = (uint32_t)a.k_ad;
        uint32_t* msum32 = reinterpret_cast<uint32_t*>(a.msum);
        const int kid_collect = p.collect_chunks ? KID_AD_CHUNKS : KID_AD_COLLECT;
        before(kid_collect);
        if (p.collect_chunks)
            hipLaunchKernelGGL(mvk::mv_ad_collect_chunks, dim3(p.collect_blocks, p.N), dim3(p.collect_threads), 0, st,
                               a.err, a.ld_e, p.d, cand, p.cap, (const mvk::u32x2*)runs, p.n_runs, segs, kth, tiecut,
                               slow, a.vote_bits, a.ld_bits, p.nwords_pad, alist, dlist, p.cap_d, adcount);
        else
            hipLaunchKernelGGL((p.collect_threads == (uint32_t)mvk::kCollectThreads
                                ? &mvk::mv_ad_collect<mvk::kCollectThreads>
                                : &mvk::mv_ad_collect<mvk::kCollectThreadsShort>),
                           dim3(p.list_blocks + p.collect_blocks, p.N), dim3(p.collect_threads), 0,
                           st, a.err, a.ld_e, p.d, cand, p.cap, rowcnt, kth, tiecut, slow, a.vote_bits, a.ld_bits,
                           p.nwords_pad, alist, dlist, p.cap_d, adcount, p.list_blocks);
        after(kid_collect);
        // (a list has at most K entries; the candidate lists have been used and lend their storage)
        const bool alone = p.K <= mvk::kAloneList;
        uint32_t parts = (p.K + mvk::kListBatch - 1) / mvk::kListBatch;
        parts = alone ? 1 : parts > 64 ? 64 : parts;
        const dim3 grid(parts, 2 * p.N);
        if (!alone) {
            before(KID_AD_HIST);
            hipLaunchKernelGGL(mvk::mv_ad_hist, grid, dim3(mvk::kRowThreads), 0, st, alist, p.cap, dlist, p.cap_d,
                               adcount, k_ad, kth, hist);
            after(KID_AD_HIST);
        }
        before(KID_AD_PICK);
        hipLaunchKernelGGL((alone ? &mvk::mv_ad_pick<true> : &mvk::mv_ad_pick<false>), grid, dim3(mvk::kRowThreads), 0,
                           st, alist, p.cap, dlist, p.cap_d, adcount, k_ad, kth, hist, cand, adbits, p.nwords_pad,
                           p.bit_blocks, adblk, msum32, a.counts);
        after(KID_AD_PICK);
        before(KID_AD_EMIT);
        hipLaunchKernelGGL(mvk::mv_ad_emit, dim3(p.N * p.bit_blocks + p.rs_blocks), dim3(mvk::kVoteThreads), 0, st,
                           adbits, p.nwords_pad, p.bit_blocks, adblk, k_ad, a.add_idx, a.drop_idx, a.vote_bits, a.ld_bits,
                           p.N * p.bit_blocks, (const uint32_t*)msum32, p.d, lvlsets);
        after(KID_AD_EMIT);
        mask_votes32 = msum32;
    }
    // the sorted vote lists, written by extra workgroups of one of the kernels from here on
    const mvk::RowLists row_lists = {p.emit_blocks, cand, p.cap, rowcnt, runs, in_order ? 1 : 0, run_taken, p.n_runs, segs,
                                     kth, tiecut, slow, a.worker_idx};
    const uint32_t n_list = sorted && !add_drop ? p.N * p.emit_blocks : 0;
    uint32_t* rsbits = ws_ptr<uint32_t>(c, p.off_rsbits);
    if (random_sel) {
        // 3''. random selection: keys of the voted coordinates, exact select of the K soonest into a bitmap
        uint32_t* rscount = ws_ptr<uint32_t>(c, p.off_rscount);
        mvk::u32x2* rslist = ws_ptr<mvk::u32x2>(c, p.off_rslist);
        mvk::u32x2* rslist2 = ws_ptr<mvk::u32x2>(c, p.off_rslist2);
        before(KID_RS_KEYS);
        hipLaunchKernelGGL(mvk::mv_rs_keys, dim3(p.rs_blocks), dim3(mvk::kVoteThreads), 0, st, votes32, p.d,
                           a.rand_exp, rslist, p.rs_cap, rscount);
        after(KID_RS_KEYS);
        const bool alone = p.rs_cap <= mvk::kAloneList;
        uint32_t parts = (p.rs_cap + mvk::kListBatch - 1) / mvk::kListBatch;
        parts = alone ? 1 : parts > 256 ? 256 : parts;
        if (!alone) {
            before(KID_RS_HIST);
            hipLaunchKernelGGL(mvk::mv_rs_hist, dim3(parts), dim3(mvk::kRowThreads), 0, st, rslist, p.rs_cap, rscount,
                               p.K, hist);
            after(KID_RS_HIST);
        }
        // The sorted vote lists are written beside this kernel, however many workgroups that makes: its own are few, or
        // long, and leave units idle, while beside the mask kernel and the gather, which fill the chip, the lists made the
        // step longer (beside the gather : so: 2 x 1,353,211 bf16, K = 3206: 58.3 us 55.6; 12 x 1 M, K = 16,000: 84.0
        // 80.5; 1 x 100,000, K = 1000: 34.3 33.0; 16 x 11.2 M, K = 11,174: 409.5 405.1; with 768 workgroups, 10 x 11.2 M,
        // K = 111,740: 333.2 331.3; 24 x 3 M, K = 30,000: 225.8 224.1).
        before(KID_RS_PICK);
        hipLaunchKernelGGL((alone ? &mvk::mv_rs_pick<true> : &mvk::mv_rs_pick<false>), dim3(parts + n_list),
                           dim3(mvk::kRowThreads), 0, st, rslist, p.rs_cap, rscount, p.K, hist, rslist2, rsbits,
                           (uint32_t)mvk::kMaskThreads * 16 * p.vote_q, p.n_vote_blocks, rsblk, parts, row_lists);
        after(KID_RS_PICK);
    }
    // 4. global mask: the vote threshold, the counts per stretch of the vote bytes and the mask's coordinates, or the
    // winners of the random selection in order; then 5. every workgroup of the last kernel gathers its part of the
    // mask, takes the mean and updates the error buffers.  Extra workgroups of one of the two write the sorted vote lists.
    {
        // Random selection's lists are under way beside mv_rs_pick.  The others run beside the mask kernel, whose blocks
        // wait for each other's counts anyway (steps beside the mask : beside the gather: 4 x 2^20, K = 10,486: 43.4 us
        // 46.1; 16 x 11.2 M, K = 11,174: 389.3 392.7; 16 x 1,000,003, K = 16,000: 74.5 77.9; 3 x 20 M, K = 200,000: 207.0
        // 209.2; 10 x 11.2 M, K = 111,740: 331.6 330.9), but not where its blocks are short ones of one quad per thread
        // and do not leave the lists room on the chip (16 x 6 M, K = 40,000: 267.3 263.5; 32 x 5 M, K = 20,000: 390.4
        // 387.2; 24 x 3 M, K = 30,000: 216.3 214.1; with room, K = 20,000: 201.5 203.2).
        const bool beside_mask = !random_sel && (p.vote_q > 1 || p.n_vote_blocks + n_list <= 512);
        const dim3 grid_c(p.n_vote_blocks + (beside_mask ? n_list : 0));
        const dim3 block(mvk::kMaskThreads);
        uint8_t* votes_out = add_drop ? nullptr : a.votes;
        const float inv_n = 1.0f / (float)p.N;
        const uint32_t kb = mvk::kMaskThreads / p.N;
        // Up to kGatherRounds rounds of kb mask positions per gathering workgroup, as few as keep the grid to a
        // thousand: many short workgroups beat few long ones (10 x 11.2 M, K = 111,740: two rounds 4 us faster than
        // four; with two rounds where they bring 312 to 390 workgroups to half as many, and with one: 12 x 2 M,
        // K = 33,000 104.6 us 103.4; 6 x 4 M, K = 66,000 109.9 108.4; random selection 8 x 4 M, K = 40,000 137.8 135.4;
        // 40 x 1 M, K = 10,000 131.6 130.9; 32 x 10 M, K = 10,000 665.5 667.2).
        uint32_t rounds = (uint32_t)(((uint64_t)p.K + 1000ull * kb - 1) / (1000ull * kb));
        if (rounds > (uint32_t)mvk::kGatherRounds) rounds = mvk::kGatherRounds;
        const uint32_t n_gather = (p.K + kb * rounds - 1) / (kb * rounds);
        const dim3 grid_g(n_gather + (beside_mask || random_sel ? 0 : n_list));
#define MV_LAUNCH_MASK(Q)                                                                                        \
        before(KID_MASK_COUNT);                                                                                  \
        hipLaunchKernelGGL((random_sel ? &mvk::mv_mask_count<Q, true> : &mvk::mv_mask_count<Q, false>), grid_c,   \
                           block, 0, st, mask_votes32, p.d, p.N, p.K, lvlsets,                                   \
                           subcnt, blockcnt, votethr, votes_out, p.n_vote_blocks, row_lists,                     \
                           add_drop || p.vote_chunks ? 1 : 0, lookback, emitfail, c->spin_limit, a.mask_idx,     \
                           reinterpret_cast<uint16_t*>(rsbits), (const uint32_t*)rsblk);             \
        after(KID_MASK_COUNT);                                                                                   \
        before(KID_GATHER);                                                                                      \
        hipLaunchKernelGGL(mvk::mv_gather_update<Q>, grid_g, block, 0, st, a.err, a.ld_e, p.d, p.N, p.K,          \
                           (const uint32_t*)mask_votes32, (const mvk::u32x2*)subcnt,                             \
                           (const mvk::u32x2*)blockcnt, p.n_vote_blocks,                                         \
                           (const uint32_t*)votethr, a.mask_idx, random_sel ? 1 : 0,                             \
                           (const uint32_t*)emitfail, inv_n,                                                     \
                           c->cfg.reduce == MV_REDUCE_MEAN ? 1 : 0, a.agg_vals, rounds, n_gather, row_lists, stepno);         \
        after(KID_GATHER);
        switch (p.vote_q) {
            case 1: { MV_LAUNCH_MASK(1) } break;
            case 2: { MV_LAUNCH_MASK(2) } break;
            case 3: { MV_LAUNCH_MASK(3) } break;
            case 4: { MV_LAUNCH_MASK(4) } break;
            case 6: { MV_LAUNCH_MASK(6) } break;
            default: { MV_LAUNCH_MASK(8) } break;
        }
#undef MV_LAUNCH_MASK
    }
    return finish();
}

}  // namespace

extern "C" {

mv_status mv_vote_step(mv_ctx* c, const void* grads, int64_t ld_g, float* err, int64_t ld_e,
                       uint32_t* worker_idx, uint8_t* votes, uint32_t* mask_idx, float* agg_vals,
                       void* stream_v)
{
    StepArgs a;
    memset(&a, 0, sizeof a);
    a.grads = grads; a.ld_g = ld_g; a.err = err; a.ld_e = ld_e;
    a.worker_idx = worker_idx; a.votes = votes; a.mask_idx = mask_idx; a.agg_vals = agg_vals;
    const mv_status st = check_common(c, a);
    if (st != MV_OK) return st;
    return enqueue_step(c, a, stream_v);
}

mv_status mv_ad_vote_step(mv_ctx* c, const void* grads, int64_t ld_g, float* err, int64_t ld_e,
                          int64_t k_ad, uint32_t* vote_bits, int64_t ld_bits, uint8_t* msum,
                          uint32_t* add_idx, uint32_t* drop_idx, uint32_t* counts,
                          uint32_t* mask_idx, float* agg_vals, void* stream_v)
{
    StepArgs a;
    memset(&a, 0, sizeof a);
    a.grads = grads; a.ld_g = ld_g; a.err = err; a.ld_e = ld_e;
    a.mask_idx = mask_idx; a.agg_vals = agg_vals;
    a.k_ad = k_ad; a.vote_bits = vote_bits; a.ld_bits = ld_bits; a.msum = msum;
    a.add_idx = add_idx; a.drop_idx = drop_idx; a.counts = counts;
    const mv_status st = check_common(c, a);
    if (st != MV_OK) return st;
    if (!c->plan.add_drop) return MV_ERR_STATE;              // the context was not begun with MV_FLAG_ADD_DROP
    if (k_ad < 1 || k_ad > (int64_t)c->plan.K) return MV_ERR_INVALID_ARG;
    if (!vote_bits || !msum || !add_idx || !drop_idx || !counts) return MV_ERR_INVALID_ARG;
    if (ld_bits < (int64_t)c->plan.nwords_pad || ld_bits % 4 != 0) return MV_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(vote_bits) & 15) || (reinterpret_cast<uintptr_t>(msum) & 15))
        return MV_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(add_idx) & 3) || (reinterpret_cast<uintptr_t>(drop_idx) & 3) ||
        (reinterpret_cast<uintptr_t>(counts) & 3))
        return MV_ERR_INVALID_ARG;
    return enqueue_step(c, a, stream_v);
}

mv_status mv_rs_vote_step(mv_ctx* c, const void* grads, int64_t ld_g, float* err, int64_t ld_e,
                          const float* rand_exp, uint32_t* worker_idx, uint8_t* votes, uint32_t* mask_idx,
                          float* agg_vals, void* stream_v)
{
    StepArgs a;
    memset(&a, 0, sizeof a);
    a.grads = grads; a.ld_g = ld_g; a.err = err; a.ld_e = ld_e;
    a.worker_idx = worker_idx; a.votes = votes; a.mask_idx = mask_idx; a.agg_vals = agg_vals;
    a.rand_exp = rand_exp;
    if (!rand_exp) return MV_ERR_INVALID_ARG;
    const mv_status st = check_common(c, a);
    if (st != MV_OK) return st;
    return enqueue_step(c, a, stream_v);
}

mv_status mv_end(mv_ctx* c)
{
    if (!c) return MV_ERR_INVALID_ARG;
    if (c->ended) return MV_ERR_STATE;
    c->ended = true;
    DeviceGuard guard(c->cfg.device);
    if (!guard.ok) return MV_ERR_DEVICE;
    mv_status rc = MV_OK;
    // steps run in the order of their calls, so the last call's stream is the one that still holds work
    if (c->steps_done != 0 && hipStreamSynchronize(c->last_stream) != hipSuccess) rc = MV_ERR_DEVICE;
    for (int r = 0; r < kEventRing; ++r)
        for (int i = 0; i < KID_COUNT; ++i)
            for (int j = 0; j < 2; ++j)
                if (c->ev[r][i][j]) (void)hipEventDestroy(c->ev[r][i][j]);
    if (c->owns_ws && c->ws && hipFree(c->ws) != hipSuccess) rc = MV_ERR_DEVICE;
    c->ws = nullptr;
    return rc;
}

void mv_release(mv_ctx* c)
{
    if (!c) return;
    if (!c->ended) (void)mv_end(c);
    delete c;
}

const char* mv_status_string(mv_status s)
{
    switch (s) {
        case MV_OK: return "ok";
        case MV_ERR_INVALID_ARG: return "invalid argument";
        case MV_ERR_UNSUPPORTED: return "unsupported";
        case MV_ERR_ALLOC: return "allocation failed";
        case MV_ERR_DEVICE: return "device error";
        case MV_ERR_STATE: return "context already ended";
    }
    return "unknown status";
}

int32_t mv_kernel_count(void) { return KID_COUNT; }

const char* mv_kernel_name(int32_t i) { return (i >= 0 && i < KID_COUNT) ? kKernelNames[i] : ""; }

mv_status mv_set_profiling(mv_ctx* c, int32_t level)
{
    if (!c || level < 0 || level > 2) return MV_ERR_INVALID_ARG;
    if (c->ended) return MV_ERR_STATE;
    c->profiling = level;
    return MV_OK;
}

mv_status mv_set_spin_limit(mv_ctx* c, uint32_t polls)
{
    if (!c) return MV_ERR_INVALID_ARG;
    if (c->ended) return MV_ERR_STATE;
    c->spin_limit = polls;
    return MV_OK;
}

mv_status mv_step_kernel_ms(mv_ctx* c, int32_t steps_back, float* ms, int32_t n)
{
    if (!c || !ms || n < KID_COUNT) return MV_ERR_INVALID_ARG;
    if (c->ended) return MV_ERR_STATE;
    if (steps_back < 0 || steps_back >= kEventRing || (uint64_t)steps_back >= c->steps_done)
        return MV_ERR_INVALID_ARG;
    DeviceGuard guard(c->cfg.device);
    if (!guard.ok) return MV_ERR_DEVICE;
    const int slot = (int)((c->steps_done - 1 - (uint64_t)steps_back) % kEventRing);
    for (int i = 0; i < KID_COUNT; ++i) {
        ms[i] = -1.0f;
        if (!c->ev_recorded[slot][i]) continue;
        if (hipEventSynchronize(c->ev[slot][i][1]) != hipSuccess) return MV_ERR_DEVICE;
        if (hipEventElapsedTime(&ms[i], c->ev[slot][i][0], c->ev[slot][i][1]) != hipSuccess)
            return MV_ERR_DEVICE;
    }
    return MV_OK;
}

mv_status mv_last_step_row_stats(mv_ctx* c, uint32_t* cand_count, uint32_t* threshold_bits, uint32_t* slow_path)
{
    if (!c) return MV_ERR_INVALID_ARG;
    if (c->ended) return MV_ERR_STATE;
    if (c->steps_done == 0) return MV_ERR_STATE;
    DeviceGuard guard(c->cfg.device);
    if (!guard.ok) return MV_ERR_DEVICE;
    if (hipStreamSynchronize(c->last_stream) != hipSuccess) return MV_ERR_DEVICE;
    const size_t nb = (size_t)c->plan.N * 4;
    if (cand_count && hipMemcpy(cand_count, c->ws + c->plan.off_candcount, nb, hipMemcpyDeviceToHost) != hipSuccess)
        return MV_ERR_DEVICE;
    if (threshold_bits && hipMemcpy(threshold_bits, c->ws + c->plan.off_tau, nb, hipMemcpyDeviceToHost) != hipSuccess)
        return MV_ERR_DEVICE;
    if (slow_path && hipMemcpy(slow_path, c->ws + c->plan.off_slow, nb, hipMemcpyDeviceToHost) != hipSuccess)
        return MV_ERR_DEVICE;
    return MV_OK;
}

mv_status mv_probe_copy(void* dst, const void* src, size_t bytes, void* stream)
{
    if (!dst || !src || bytes == 0 || (bytes & 15) != 0) return MV_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(dst) & 15) || (reinterpret_cast<uintptr_t>(src) & 15))
        return MV_ERR_INVALID_ARG;
    const uint64_t n16 = bytes / 16;
    const uint64_t blocks = (n16 + 1023) / 1024;
    if (blocks > 0x7FFFFFFFull) return MV_ERR_INVALID_ARG;
    hipLaunchKernelGGL(mvk::mv_probe_copy_kernel, dim3((uint32_t)blocks), dim3(256), 0,
                       static_cast<hipStream_t>(stream), static_cast<const mvk::u32x4*>(src),
                       static_cast<mvk::u32x4*>(dst), n16);
    return hipGetLastError() == hipSuccess ? MV_OK : MV_ERR_DEVICE;
}

}  // extern "C"
