// Short vectors (up to kSmallMaxD coordinates): a whole step in two launches, for all three
// voting schemes.
#pragma once

#include "mv_common.hpp"
#include "mv_mask.hpp"

namespace mvk {

// ----------------------------------------------------------------------------
// 9. short vectors
// ----------------------------------------------------------------------------
// Up to 32,768 coordinates a row fits the registers of one workgroup, and what a step
// costs is launches and dependent round trips, not bytes.  So no estimate, no candidate
// lists and no segment tables:
//   mv_small_rows   a workgroup per row: a = g + e, the exact top K from registers, the
//                   sorted vote list and the vote as a bitmap (d bits); with add-drop
//                   voting the row's additions and removals as well
//   mv_small_mask   every workgroup counts the votes from the N bitmaps (32 coordinates
//                   per thread, bit-sliced), finds the mask -- the same work in each,
//                   instead of another launch -- and gathers its own positions
// Step of 4 x 10,007 coordinates, K = 101: 35.2 us in the four launches of long vectors, 17.4 us so
// (8.8 + 7.6 in the kernels).  At the limit, 16 x 32,768, K = 546: 28.0 us (one compute unit reads a
// row, 15.8 us), against 38.8 the long way; add-drop 41 against 61.  Beyond it a row no longer fits one
// workgroup's registers.
constexpr int kSmallThreads = 1024;
constexpr int kSmallMaxD = 32 * kSmallThreads;
constexpr int kSmallBins = 8192;             // first digit: the 13 leading bits of a key
constexpr int kSmallShift = 31 - 13;
constexpr int kSmallDigit = 512;             // second and third digit: 9 bits each

struct SmallSelectLds {
    __attribute__((aligned(16))) uint32_t hist[kSmallBins];
    __attribute__((aligned(16))) uint32_t mkey[kRankCap + 4];
    __attribute__((aligned(16))) uint32_t mpos[kRankCap + 4];
    uint32_t ties[kSmallMaxD / 32];          // bitmap of the entries that tie with the last one taken
    uint64_t scan[kSmallThreads / kWave];
    uint32_t bcast[3];
    uint32_t n_list;
};

// With a histogram complete (a barrier has passed): the bin that holds the `want`-th largest entry, the
// rank inside it and the bin's count; returns the histogram's total (want > total: the rest is not set).
template <int BINS>
__device__ __forceinline__ uint32_t small_find(SmallSelectLds& lds, uint32_t want, uint32_t& bin, uint32_t& want_in_bin,
                                               uint32_t& in_bin)
{
    constexpr int per = BINS > kSmallThreads ? BINS / kSmallThreads : 1;
    const uint32_t t = threadIdx.x;
    uint32_t h[per];
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < per; ++q) {              // descending bins over threads
        const int b = BINS - 1 - ((int)t * per + q);
        h[q] = b >= 0 ? lds.hist[b] : 0u;
        sum += h[q];
    }
    uint32_t total;
    uint32_t acc = block_excl_scan<kSmallThreads>(sum, lds.scan, total);
    if (acc < want && want <= acc + sum) {
#pragma unroll
        for (int q = 0; q < per; ++q) {
            if (acc < want && want <= acc + h[q]) {
                lds.bcast[0] = (uint32_t)(BINS - 1 - ((int)t * per + q));
                lds.bcast[1] = want - acc;
                lds.bcast[2] = h[q];
            }
            acc += h[q];
        }
    }
    __syncthreads();
    bin = lds.bcast[0];
    want_in_bin = lds.bcast[1];
    in_bin = lds.bcast[2];
    return total;
}

// Marks the `want` largest of the workgroup's entries, equal keys in the order of place(i): thread t has
// NK entries, entry i exists if bit i of `active` is set, has key[i] (31 bits) and the place place(i)
// (below kSmallMaxD, all different).  1 <= want <= number of entries.  All threads must call it.
// A histogram of the 13 leading key bits (32 bins to an octave) finds the bin in which the last one taken
// lies; its members are ranked by counting when few, else two more digits of 9 bits follow, and ties are
// cut with a bitmap.  Zeros, which values on a lattice have by the thousand, are kept out of the
// histogram: equal keys queue up on one LDS address.
template <int NK, typename Place>
__device__ __forceinline__ uint32_t small_select(const uint32_t (&key)[NK], uint32_t active, uint32_t want, Place place,
                                                 SmallSelectLds& lds)
{
    const uint32_t t = threadIdx.x;
    {
        const u32x4 z = {0u, 0u, 0u, 0u};
        u32x4* hz = reinterpret_cast<u32x4*>(lds.hist);
        for (int b = t; b < kSmallBins / 4; b += kSmallThreads) hz[b] = z;
        if (t == 0) lds.n_list = 0;
    }
    __syncthreads();
    uint32_t bin, left, in_bin;
#pragma unroll
    for (int i = 0; i < NK; ++i)
        if ((active >> i & 1u) && key[i] != 0u) atomicAdd(&lds.hist[key[i] >> kSmallShift], 1u);
    __syncthreads();
    const uint32_t total = small_find<kSmallBins>(lds, want, bin, left, in_bin);

    uint32_t last = 0;                           // the smallest key taken
    uint32_t take_eq = want - total;             // how many of the keys equal to it (here: zeros)
    if (want <= total) {                         // uniform
        if (left == in_bin) {                    // the whole bin is taken, zeros are not
            last = max(bin << kSmallShift, 1u);
            uint32_t taken = 0;
#pragma unroll
            for (int i = 0; i < NK; ++i) taken |= (key[i] >= last ? 1u : 0u) << i;
            return taken & active;
        }
        if (in_bin <= (uint32_t)kRankCap) {      // uniform: rank the members by counting
#pragma unroll
            for (int i = 0; i < NK; ++i)
                if ((active >> i & 1u) && key[i] != 0u && key[i] >> kSmallShift == bin) {
                    const uint32_t p = atomicAdd(&lds.n_list, 1u);
                    lds.mkey[p] = key[i];
                    lds.mpos[p] = place(i);
                }
            if (t < 4) {                         // pad to a multiple of 4 with entries ranked last
                lds.mkey[in_bin + t] = 0;
                lds.mpos[in_bin + t] = 0xFFFFFFFFu;
            }
            __syncthreads();
            if (t < in_bin) {
                const uint32_t mk = lds.mkey[t], mp = lds.mpos[t];
                const u32x4* hk = reinterpret_cast<const u32x4*>(lds.mkey);
                const u32x4* hp = reinterpret_cast<const u32x4*>(lds.mpos);
                uint32_t ahead = 0;
#pragma unroll 4
                for (uint32_t j = 0; j < (in_bin + 3) / 4; ++j) {
                    const u32x4 ok = hk[j], op = hp[j];
                    ahead += (ok.x > mk) || (ok.x == mk && op.x < mp);
                    ahead += (ok.y > mk) || (ok.y == mk && op.y < mp);
                    ahead += (ok.z > mk) || (ok.z == mk && op.z < mp);
                    ahead += (ok.w > mk) || (ok.w == mk && op.w < mp);
                }
                if (ahead == left - 1) {
                    lds.bcast[0] = mk;
                    lds.bcast[1] = mp;
                }
            }
            __syncthreads();
            last = lds.bcast[0];
            const uint32_t cut = lds.bcast[1];
            uint32_t taken = 0;
#pragma unroll
            for (int i = 0; i < NK; ++i)
                taken |= (key[i] > last || (key[i] == last && place(i) <= cut) ? 1u : 0u) << i;
            return taken & active;
        }
        // many members: the remaining 18 bits, 9 at a time
        uint32_t prefix = bin << kSmallShift;
#pragma unroll
        for (int shift = kSmallShift - 9; shift >= 0; shift -= 9) {
            if (t < (uint32_t)kSmallDigit) lds.hist[t] = 0;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NK; ++i)
                if ((active >> i & 1u) && key[i] != 0u && (key[i] ^ prefix) >> (shift + 9) == 0u)
                    atomicAdd(&lds.hist[(key[i] >> shift) & (uint32_t)(kSmallDigit - 1)], 1u);
            __syncthreads();
            (void)small_find<kSmallDigit>(lds, left, bin, left, in_bin);
            prefix |= bin << shift;
        }
        last = prefix;
        take_eq = left;
    }
    // entries equal to `last`, taken in the order of their places
    lds.ties[t] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NK; ++i)
        if ((active >> i & 1u) && key[i] == last) atomicOr(&lds.ties[place(i) >> 5], 1u << (place(i) & 31u));
    __syncthreads();
    {
        uint32_t w = lds.ties[t];
        uint32_t all;
        const uint32_t before = block_excl_scan<kSmallThreads>((uint32_t)__popc(w), lds.scan, all);
        uint32_t keep = 0;
        for (uint32_t room = before < take_eq ? take_eq - before : 0u; w != 0u && room != 0u; --room) {
            keep |= w & (0u - w);
            w &= w - 1u;
        }
        lds.ties[t] = keep;
    }
    __syncthreads();
    uint32_t taken = 0;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
        const bool tie = key[i] == last && (lds.ties[place(i) >> 5] >> (place(i) & 31u) & 1u);
        taken |= (key[i] > last || tie ? 1u : 0u) << i;
    }
    return taken & active;
}

// What add-drop voting adds to a row's work (vote_bits null: plain voting)
struct SmallAddDrop {
    uint32_t* vote_bits;
    int64_t   ld_bits;
    uint32_t* msum32;
    uint32_t  k_ad;
    uint32_t* add_idx;
    uint32_t* drop_idx;
    uint32_t* counts;
};

struct SmallRowsLds {
    SmallSelectLds sel;
    uint32_t bits[kSmallMaxD / 32];
    uint32_t stand[kSmallMaxD / 32];
};

// four bits to the low bits of four bytes
__device__ __forceinline__ uint32_t nibble_to_bytes(uint32_t x) { return (x * 0x00204081u) & 0x01010101u; }

// U quads of coordinates per thread: coordinate u * 4096 + 4 t + c for u < U, c < 4.  Bound by its chain:
// loads, two barriers and an LDS round trip per digit, the list.
template <typename GT, int U>
__global__ __launch_bounds__(kSmallThreads) void mv_small_rows(
    const GT* __restrict__ g, int64_t ld_g, float* __restrict__ e, int64_t ld_e, uint32_t d, uint32_t K,
    uint32_t* __restrict__ worker_idx, uint32_t* __restrict__ row_bits, uint32_t n_words,
    uint32_t* __restrict__ cand_count, uint32_t* __restrict__ tau_bits, uint32_t* __restrict__ slow_flag,
    SmallAddDrop ad)
{
    __shared__ SmallRowsLds lds;
    const uint32_t row = blockIdx.x, t = threadIdx.x;
    const GT* grow = g + (int64_t)row * ld_g;
    float*    erow = e + (int64_t)row * ld_e;
    uint32_t* vrow = ad.vote_bits ? ad.vote_bits + (int64_t)row * ad.ld_bits : nullptr;
    if (t == 0) {                                // row statistics: every coordinate was a candidate
        cand_count[row] = d;
        tau_bits[row] = 0;
        slow_flag[row] = 0;
    }
    uint32_t key[4 * U];
    uint32_t inside = 0;
    {
        f32x4 gv[U], ev[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t j = (uint32_t)u * (4 * kSmallThreads) + t * 4;
            if (j + 4 <= d) {
                gv[u] = load4_grad(grow + j);
                ev[u] = *reinterpret_cast<const f32x4*>(erow + j);
            }
        }
        if (vrow) lds.stand[t] = t < n_words ? vrow[t] : 0u;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t j = (uint32_t)u * (4 * kSmallThreads) + t * 4;
            if (j + 4 <= d) {
                const f32x4 a = gv[u] + ev[u];
                *reinterpret_cast<f32x4*>(erow + j) = a;
                key[u * 4 + 0] = __float_as_uint(a.x) & kAbsMask;
                key[u * 4 + 1] = __float_as_uint(a.y) & kAbsMask;
                key[u * 4 + 2] = __float_as_uint(a.z) & kAbsMask;
                key[u * 4 + 3] = __float_as_uint(a.w) & kAbsMask;
                inside |= 15u << (4 * u);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    key[u * 4 + c] = 0;
                    if (j + c < d) {
                        const float a = load1_grad(grow + j + c) + erow[j + c];
                        erow[j + c] = a;
                        key[u * 4 + c] = __float_as_uint(a) & kAbsMask;
                        inside |= 1u << (4 * u + c);
                    }
                }
            }
        }
    }
    auto place = [t](int i) { return (uint32_t)(i >> 2) * (4 * kSmallThreads) + t * 4 + (uint32_t)(i & 3); };
    // the marked coordinates as a bitmap in lds.bits, word w = coordinates 32 w .. 32 w + 31; returns thread t's word
    auto bitmap_of = [&](uint32_t marked) {
        lds.bits[t] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t nib = marked >> (4 * u) & 15u;
            if (nib) atomicOr(&lds.bits[u * (kSmallThreads / 8) + (t >> 3)], nib << ((t & 7u) * 4u));
        }
        __syncthreads();
        return lds.bits[t];
    };
    // their coordinates, ascending, to out[0 .. limit)
    auto write_list = [&](uint32_t word, uint32_t* out, uint32_t limit) {
        uint32_t total;
        uint32_t pos = block_excl_scan<kSmallThreads>((uint32_t)__popc(word), lds.sel.scan, total);
        for (; word != 0u; word &= word - 1u, ++pos)
            if (pos < limit) out[pos] = t * 32u + (uint32_t)__ffs((int)word) - 1u;
    };

    const uint32_t top = small_select<4 * U>(key, inside, K, place, lds.sel);
    if (!vrow) {
        const uint32_t word = bitmap_of(top);
        if (t < n_words) row_bits[(size_t)row * n_words + t] = word;
        if (worker_idx) write_list(word, worker_idx + (size_t)row * K, K);
        return;
    }

    // Add-drop voting: the k_ad largest of the top K that are not in the standing vote join it, the k_ad
    // smallest of its members that are not in the top K leave it (keys complemented: largest first).
    uint32_t member = 0;
#pragma unroll
    for (int u = 0; u < U; ++u)
        member |= (lds.stand[u * (kSmallThreads / 8) + (t >> 3)] >> ((t & 7u) * 4u) & 15u) << (4 * u);
    uint32_t joins = top & ~member, leaves = member & inside & ~top;
    uint64_t found;
    __syncthreads();                             // the scan's scratch is free
    (void)block_excl_scan64<kSmallThreads>(pack2((uint32_t)__popc(joins), (uint32_t)__popc(leaves)), lds.sel.scan, found);
    __syncthreads();
    const uint32_t n_joins = (uint32_t)(found >> 32), n_leaves = (uint32_t)found;
    if (n_joins > ad.k_ad) joins = small_select<4 * U>(key, joins, ad.k_ad, place, lds.sel);
    if (n_leaves > ad.k_ad) {
#pragma unroll
        for (int i = 0; i < 4 * U; ++i) key[i] = kAbsMask - key[i];
        leaves = small_select<4 * U>(key, leaves, ad.k_ad, place, lds.sel);
    }
    const uint32_t add = bitmap_of(joins);
    write_list(add, ad.add_idx + (size_t)row * ad.k_ad, ad.k_ad);
    __syncthreads();
    const uint32_t drop = bitmap_of(leaves);
    write_list(drop, ad.drop_idx + (size_t)row * ad.k_ad, ad.k_ad);
    if ((add | drop) != 0u) {                    // words beyond the row's are zero
        vrow[t] = lds.stand[t] ^ add ^ drop;
        // M^sum moves with the standing votes: bytes packed four to a word; a byte never carries because
        // 0 <= msum <= N <= 255 holds before and after
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t up = nibble_to_bytes(add >> (4 * q) & 15u), down = nibble_to_bytes(drop >> (4 * q) & 15u);
            if (up) atomicAdd(&ad.msum32[t * 8u + q], up);
            if (down) atomicSub(&ad.msum32[t * 8u + q], down);
        }
    }
    if (t < 2) ad.counts[2 * row + t] = min(t ? n_leaves : n_joins, ad.k_ad);
}

struct SmallMaskLds {
    union {
        struct {                                              // random selection: the voted coordinates, ascending,
            uint16_t voted_at[kSmallMaxD];                    // and their votes
            uint8_t  voted_by[kSmallMaxD];
        };
        struct {                                              // then, for the gather:
            uint32_t slice[kGatherRounds * kSmallThreads];    // the workgroup's positions' coordinates
            float    tile[kTileFloats];
        };
    };
    uint64_t scan[2][kSmallThreads / kWave];
    uint32_t winners[kSmallMaxD / 32];                        // random selection: bitmap
    SmallSelectLds sel;
};

// sum and carry of three bits in every bit position
__device__ __forceinline__ void full_add(uint32_t a, uint32_t b, uint32_t c, uint32_t& sum, uint32_t& carry)
{
    const uint32_t x = a ^ b;
    carry = (a & b) | (x & c);
    sum = x ^ c;
}

// The winners of the random selection: the K soonest of the n <= NK * 1024 voted coordinates, to lds.winners.
template <int NK>
__device__ __forceinline__ void small_random_winners(const float* __restrict__ rand_exp, uint32_t n, uint32_t K,
                                                     SmallMaskLds& lds)
{
    const uint32_t t = threadIdx.x;
    uint32_t key[NK], at[NK];
    float    r[NK];
    uint32_t active = 0;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
        const uint32_t p = (uint32_t)i * kSmallThreads + t;
        at[i] = 0;
        r[i] = 0.0f;
        if (p < n) {
            at[i] = lds.voted_at[p];
            r[i] = rand_exp[at[i]];
            active |= 1u << i;
        }
    }
#pragma unroll
    for (int i = 0; i < NK; ++i) {
        key[i] = 0;
        if (active >> i & 1u) {
            const float time = __fdiv_rn(r[i], (float)lds.voted_by[(uint32_t)i * kSmallThreads + t]);
            key[i] = kAbsMask - (__float_as_uint(time) & kAbsMask);           // sooner = larger key
        }
    }
    // the list is in the order of the coordinates: places in it order ties
    const uint32_t won = small_select<NK>(key, active, K, [t](int i) { return (uint32_t)i * kSmallThreads + t; }, lds.sel);
#pragma unroll
    for (int i = 0; i < NK; ++i)
        if (won >> i & 1u) atomicOr(&lds.winners[at[i] >> 5], 1u << (at[i] & 31u));
}

// Votes, mask, gather.  msum32 null: the votes are counted from the rows' bitmaps; else they are its bytes.
// RANDOM: random selection with rand_exp.  votes_out may be null.
template <bool RANDOM>
__global__ __launch_bounds__(kSmallThreads) void mv_small_mask(
    float* __restrict__ e, int64_t ld_e, uint32_t d, uint32_t N, uint32_t K, const uint32_t* __restrict__ row_bits,
    uint32_t n_words, const uint32_t* __restrict__ msum32, const float* __restrict__ rand_exp,
    uint8_t* __restrict__ votes_out, uint32_t* __restrict__ mask_idx, float scale, int apply_scale,
    float* __restrict__ agg, uint32_t rounds)
{
    __shared__ SmallMaskLds lds;
    const uint32_t t = threadIdx.x;
    const uint32_t kb = kSmallThreads / N;       // N <= 255, so kb >= 4
    const uint32_t k0 = blockIdx.x * kb * rounds, k1 = min(K, k0 + kb * rounds);
    uint32_t inside = 0;                         // which of the thread's coordinates 32 t .. 32 t + 31 there are
    if (t < n_words) inside = d - t * 32u >= 32u ? 0xFFFFFFFFu : (1u << (d & 31u)) - 1u;

    // the votes of the thread's coordinates, bit p of all of them in plane[p]
    uint32_t plane[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (!msum32) {
        for (uint32_t n0 = 0; n0 < N; n0 += 7) {
            uint32_t x[7];
#pragma unroll
            for (int i = 0; i < 7; ++i)
                x[i] = n0 + i < N && t < n_words ? row_bits[(size_t)(n0 + i) * n_words + t] : 0u;
            uint32_t s0, s1, s, c0, c1, c2, c, f;
            full_add(x[0], x[1], x[2], s0, c0);
            full_add(x[3], x[4], x[5], s1, c1);
            full_add(s0, s1, x[6], s, c2);
            full_add(c0, c1, c2, c, f);          // the seven rows' sum = s + 2 c + 4 f
            uint32_t carry = plane[0] & s;
            plane[0] ^= s;
            full_add(plane[1], c, carry, plane[1], carry);
            full_add(plane[2], f, carry, plane[2], carry);
#pragma unroll
            for (int p = 3; p < 8; ++p) {
                const uint32_t up = plane[p] & carry;
                plane[p] ^= carry;
                carry = up;
            }
        }
    } else if (t < n_words) {
        // (msum is padded with zeros to a multiple of 16 bytes)
        const u32x4 z = {0u, 0u, 0u, 0u};
        const u32x4 lo = *reinterpret_cast<const u32x4*>(msum32 + t * 8u);
        const u32x4 hi = t * 32u + 16u < d ? *reinterpret_cast<const u32x4*>(msum32 + t * 8u + 4u) : z;
        const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int p = 0; p < 8; ++p)
#pragma unroll
            for (int q = 0; q < 8; ++q)          // bit p of four bytes to four neighbouring bits
                plane[p] |= ((w[q] >> p & 0x01010101u) * 0x10204080u) >> 28 << (4 * q);
    }
    const uint32_t n_planes = msum32 ? 8u : 32u - (uint32_t)__clz(N);
    uint32_t bytes[8];                           // four coordinates' votes each, where someone asks for them
    if (RANDOM || votes_out) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            bytes[q] = 0;
#pragma unroll
            for (int p = 0; p < 8; ++p)
                if ((uint32_t)p < n_planes) bytes[q] |= nibble_to_bytes(plane[p] >> (4 * q) & 15u) << p;
        }
        if (votes_out && t % gridDim.x == blockIdx.x && t < n_words) {         // the workgroups share the copy
            uint8_t* to = votes_out + t * 32u;
            if (inside == 0xFFFFFFFFu && (reinterpret_cast<uintptr_t>(votes_out) & 15) == 0) {
                reinterpret_cast<u32x4*>(to)[0] = u32x4{bytes[0], bytes[1], bytes[2], bytes[3]};
                reinterpret_cast<u32x4*>(to)[1] = u32x4{bytes[4], bytes[5], bytes[6], bytes[7]};
            } else {
#pragma unroll
                for (int b = 0; b < 32; ++b)
                    if (inside >> b & 1u) to[b] = (uint8_t)(bytes[b >> 2] >> (8 * (b & 3)));
            }
        }
    }

    // all coordinates in `above` are taken, and the first `take` of those in `at`
    uint32_t above = 0, at = inside, take = K;
    if constexpr (RANDOM) {
        uint32_t voted = 0;
#pragma unroll
        for (int p = 0; p < 8; ++p) voted |= plane[p];
        uint32_t n;
        uint32_t pos = block_excl_scan<kSmallThreads>((uint32_t)__popc(voted), lds.scan[0], n);
#pragma unroll
        for (int b = 0; b < 32; ++b)
            if (voted >> b & 1u) {
                lds.voted_at[pos] = (uint16_t)(t * 32u + b);
                lds.voted_by[pos++] = (uint8_t)(bytes[b >> 2] >> (8 * (b & 3)));
            }
        lds.winners[t] = 0;
        __syncthreads();
        if (n <= 4u * kSmallThreads) small_random_winners<4>(rand_exp, n, K, lds);       // uniform
        else                         small_random_winners<32>(rand_exp, n, K, lds);
        __syncthreads();
        above = lds.winners[t];
        at = 0;
        take = 0;
    } else {
        // the K-th largest number of votes, bit by bit from the top: one count per bit
        for (uint32_t i = 0; i < n_planes; ++i) {
            uint32_t bit = 0;
#pragma unroll
            for (int p = 0; p < 8; ++p)          // plane[n_planes - 1 - i], registers not being indexed
                bit = n_planes - 1u - i == (uint32_t)p ? plane[p] : bit;
            const uint32_t with = at & bit;
            uint32_t n;
            (void)block_excl_scan<kSmallThreads>((uint32_t)__popc(with), lds.scan[i & 1u], n);   // in turn: one barrier
            if (n >= take) {                     // uniform
                at = with;
            } else {
                above |= with;
                at &= ~bit;
                take -= n;
            }
        }
    }
    __syncthreads();
    uint64_t total;
    const uint64_t before = block_excl_scan64<kSmallThreads>(pack2((uint32_t)__popc(above), (uint32_t)__popc(at)),
                                                             lds.scan[0], total);
    {
        uint32_t g0 = (uint32_t)(before >> 32), e0 = (uint32_t)before;
        const uint32_t first = g0 + min(e0, take);
        uint32_t m = above | at;
        if (first >= k1) m = 0;                  // behind the workgroup's positions
        for (; m != 0u; m &= m - 1u) {
            const uint32_t low = m & (0u - m);
            const bool is_above = (above & low) != 0u;
            if (is_above || e0 < take) {
                const uint32_t pos = g0 + min(e0, take);
                if (pos >= k0 && pos < k1) {
                    const uint32_t j = t * 32u + (uint32_t)__ffs((int)low) - 1u;
                    lds.slice[pos - k0] = j;
                    mask_idx[pos] = j;
                }
            }
            if (is_above) ++g0;
            else ++e0;
        }
    }
    __syncthreads();
    gather_positions(lds.tile, lds.slice, e, ld_e, d, N, k0, k1, rounds, scale, apply_scale, agg);
}

}  // namespace mvk
