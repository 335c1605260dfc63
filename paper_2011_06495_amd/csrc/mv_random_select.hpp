// Majority voting with random selection (Algorithm 1, the S_rand-weighted line).
#pragma once

#include "mv_common.hpp"
#include "mv_select.hpp"
#include "mv_mask.hpp"

namespace mvk {

// ----------------------------------------------------------------------------
// 8. majority voting with random selection (Algorithm 1, the S_rand-weighted line;
//    Sec. 2, paragraph after Algorithm 1; Sec. 4.2)
// ----------------------------------------------------------------------------
// Winners are drawn in proportion to their votes until K distinct ones are
// selected.  Stated without an order of draws: every voted coordinate j gets an
// exponential clock of rate votes[j], i.e. the time rand_exp[j] / votes[j] with
// rand_exp[j] ~ Exp(1) from the caller, and the K clocks that ring first win
// (equal times: lowest coordinate first).  The time is one correctly rounded fp32
// division; its bit pattern, complemented, is a key for the same exact select
// that serves long lists of candidates (list_split).  Selected coordinates are marked in
// a bitmap that the mask kernel turns into the ascending mask.

// Scan of the packed vote bytes (grid as for the mask kernels): every voted
// coordinate is appended to the list with its key.  rs_count[0] = list length.
__device__ __forceinline__ u32x2 rs_entry(const float* __restrict__ rand_exp, uint32_t j, uint32_t v)
{
    const float time = __fdiv_rn(rand_exp[j], (float)v);
    u32x2 c;
    c.x = kAbsMask - (__float_as_uint(time) & kAbsMask);            // sooner = larger key
    c.y = j;
    return c;
}
// The voted coordinates are parked in LDS as (offset, votes) and their random numbers then fetched by all
// lanes together: one dependent load per entry inside each thread's own loop made this kernel 2.5x
// slower, and 8x slower on crowded blocks.
__global__ __launch_bounds__(kVoteThreads) void mv_rs_keys(const uint32_t* __restrict__ votes32, int64_t d,
                                                           const float* __restrict__ rand_exp,
                                                           u32x2* __restrict__ list, uint32_t list_cap,
                                                           uint32_t* __restrict__ rs_count)
{
    static_assert(kVoteBlock == kVoteThreads * 16, "16 coordinates per thread");
    __shared__ uint32_t stage[kVoteBlock];                         // all of the block's coordinates may hold a vote
    __shared__ uint64_t scan_lds[kVoteThreads / kWave];
    __shared__ uint32_t base_sh;
    const int64_t base = (int64_t)blockIdx.x * kVoteBlock;
    const uint32_t off0 = threadIdx.x * 16;
    const u32x4 z = {0u, 0u, 0u, 0u};
    const u32x4 w = base + off0 < d ? *reinterpret_cast<const u32x4*>(votes32 + ((base + off0) >> 2)) : z;   // zero past d
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
    uint32_t n = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) n += ((ww[q >> 2] >> (8 * (q & 3))) & 255u) != 0u;
    uint32_t total;
    uint32_t sp = block_excl_scan<kVoteThreads>(n, scan_lds, total);
    if (total == 0) return;                                        // whole workgroup
    if (threadIdx.x == 0) base_sh = atomicAdd(&rs_count[0], total);
    if (n)
        for (int q = 0; q < 16; ++q) {
            const uint32_t v = (ww[q >> 2] >> (8 * (q & 3))) & 255u;
            if (v) stage[sp++] = ((off0 + (uint32_t)q) << 8) | v;
        }
    __syncthreads();
    const uint32_t at = base_sh;
    for (uint32_t i = threadIdx.x; i < total; i += kVoteThreads) {
        const uint32_t s = stage[i];
        if (at + i < list_cap) list[at + i] = rs_entry(rand_exp, (uint32_t)base + (s >> 8), s & 255u);
    }
}

// ---- one list; its storage is row 0's
__device__ __forceinline__ ListView rs_list(const u32x2* __restrict__ list, uint32_t list_cap,
                                            const uint32_t* __restrict__ rs_count, uint32_t K,
                                            uint32_t* __restrict__ sample_hist)
{
    ListView v;
    v.list = list;
    v.n = min(rs_count[0], list_cap);
    v.want = K;
    v.base = kAbsMask - 0x42800000u;              // times from 64 down: 64 bins to an octave for eight octaves, then 32
    v.fine = 17;
    v.coarse = 18;
    lend_storage(v, sample_hist, 0, 0);
    return v;
}

// Long lists only (see list_split): the histogram
__global__ __launch_bounds__(kRowThreads) void mv_rs_hist(const u32x2* __restrict__ list, uint32_t list_cap,
                                                          const uint32_t* __restrict__ rs_count, uint32_t K,
                                                          uint32_t* __restrict__ sample_hist)
{
    __shared__ uint32_t hist[kListBins];
    const ListView v = rs_list(list, list_cap, rs_count, K, sample_hist);
    list_hist(v, blockIdx.x, gridDim.x, hist);
}

// Workgroups [0, n_pick): mark the winners in the bitmap and count them per block of the mask kernel (`per_block`
// coordinates), and leave the list's length at zero for the next step.  Workgroups beyond write the sorted vote lists,
// where they run beside this kernel.
template <bool ALONE>
__global__ __launch_bounds__(kRowThreads) void mv_rs_pick(const u32x2* __restrict__ list, uint32_t list_cap,
                                                          uint32_t* __restrict__ rs_count, uint32_t K,
                                                          uint32_t* __restrict__ sample_hist, u32x2* __restrict__ list2,
                                                          uint32_t* __restrict__ rs_bits, uint32_t per_block, uint32_t n_blocks,
                                                          uint32_t* __restrict__ winners_per_block, uint32_t n_pick,
                                                          RowLists lists)
{
    __shared__ union { SplitLds<kMembersMost> pick; EmitLds emit; } shared;   // few workgroups, each with a compute unit to itself
    if (blockIdx.x >= n_pick) {
        __shared__ uint64_t scan_lds[kMaskThreads / kWave];
        static_assert(kMaskThreads == kRowThreads, "both kinds of workgroup have as many threads");
        write_row_lists(lists, blockIdx.x - n_pick, K, shared.emit, scan_lds);
        return;
    }
    SplitLds<kMembersMost>& lds = shared.pick;
    ListView v = rs_list(list, list_cap, rs_count, K, sample_hist);
    v.list2 = list2;
    if (v.n < K) return;                          // whole grid; cannot happen: every row votes K coordinates
    const BlockTally tally = {lds.tally, winners_per_block, 1, n_blocks};
    tally.clear();                                // (list_split has barriers before it acts)
    uint32_t kth, tie_cut;
    ListRest rest;
    const bool finished = list_split<ALONE ? SplitEnd::Alone : SplitEnd::Last>(
        v, blockIdx.x, n_pick, lds,
        [&](const u32x2 (&c)[kListUnroll], uint32_t taken) {
#pragma unroll
            for (int u = 0; u < kListUnroll; ++u) {
                const bool mine = taken >> u & 1u;
                if (mine) atomicOr(&rs_bits[c[u].y >> 5], 1u << (c[u].y & 31u));
                tally.add(c[u].y / per_block, mine);
            }
        },
        kth, tie_cut, rest);
    tally.merge();
    if (finished && threadIdx.x == 0) rs_count[0] = 0;   // (all workgroups have read it)
}

}  // namespace mvk
