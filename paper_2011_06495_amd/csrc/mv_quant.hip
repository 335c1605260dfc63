// Fractional quantisation of the paper's Sec. 4.3.2 on the GPU, for batches of
// rows (for instance the N workers' K masked values).
//
// q bits per value: q-1 bits name one of L = 2^(q-1) geometric intervals of |v|
// between the row's largest and smallest non-zero magnitude, one bit is the sign;
// L means (of the magnitudes that fell into each interval) follow, and the
// receiver reproduces sign * mean.
//
// The interval edges are computed in fp64 from correctly rounded operations only
// (a division, q-1 square roots -- L is a power of two, so that is the L-th root --
// and L-1 divisions), so they are the same numbers on any IEEE machine:
//   alpha = (v_max / v_min)^(1/L),  edge_0 = v_max,  edge_l = edge_{l-1} / alpha,
//   interval of |v| = 1 + #{ j in 1..L-1 : |v| <= edge_j }   (a value on an edge
//   goes to the interval of the smaller magnitudes; zeros go to the last one).
// code = (interval - 1) | sign << (q-1); value k occupies bits [k q, (k+1) q) of the
// row's stream, bit b of a stream being bit b % 32 of word b / 32.
//
// Encoding is latency, not bandwidth (a row of 111,740 values is 447 KB): what counts is
// how many compute units share a row and how long the dependent chain is.  Rows of up to
// kTile values, and of up to row_most(q), are done whole by one workgroup in one launch; longer
// rows are cut into tiles of kTile values over up to kMaxBlocks workgroups, in three launches: the
// blocks' largest and smallest magnitudes; codes and the blocks' sums per interval; the means.
// 10 rows of 111,740 values, q = 4: 188 us with one workgroup per row, 12.6 us so (3.8 + 6.8 + 2.7
// us in the kernels).
#include "../../include/mv.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mvq {

constexpr int kTile = 2048;         // values a workgroup works on at a time
constexpr int kMaxBlocks = 256;     // workgroups per row: every one reads the ranges of all
constexpr int kRangeThreads = 256;
constexpr int kMeanThreads = 1024;

// values per packing group: the fewest whose codes fill whole words
__host__ __device__ constexpr int group_size(int q)
{
    int g = 32;
    while (g > 1 && ((g / 2) * q) % 32 == 0) g /= 2;
    return g;
}

// Wavefronts per workgroup of quant_codes_kernel: every wavefront has a table of L x 64 sums
// (8 bytes) and counts (4 bytes) in LDS, 96 KB of tables at most.
constexpr int code_waves(int q) { return q <= 6 ? 4 : q == 7 ? 2 : 1; }

// The values of a row that one workgroup of kRowWaves wavefronts takes whole.  The three launches take 12 us however
// short the row is: 10 rows of 2049 values, q = 2, 3, 4: 12.8, 12.5, 13.3 us, so 5.3, 5.9, 5.5; of 8192 values 12.9, 13.2,
// 12.9, so 5.8, 7.0, 6.9; of 16,384, q = 2, 3: 12.9, 12.7, so 7.3, 8.7.  With more intervals the tables of so many
// wavefronts would not fit.
constexpr int kRowWaves = 16;
__host__ __device__ constexpr int row_most(int q) { return q <= 3 ? 16384 : q == 4 ? 8192 : 0; }

struct Range {                      // of the non-zero magnitudes, as bit patterns (same order as the values)
    uint32_t vmax, vmin;            // 0 and 0xFFFFFFFF: none
};

__device__ __forceinline__ void widen(Range& r, float x)
{
    const uint32_t m = __float_as_uint(x) & 0x7FFFFFFFu;
    r.vmax = max(r.vmax, m);
    if (m) r.vmin = min(r.vmin, m);
}

// All lanes of the wavefront get the wavefront's range.
__device__ __forceinline__ Range wave_range(Range r)
{
    for (int o = 32; o >= 1; o >>= 1) {
        r.vmax = max(r.vmax, (uint32_t)__shfl_xor(r.vmax, o, 64));
        r.vmin = min(r.vmin, (uint32_t)__shfl_xor(r.vmin, o, 64));
    }
    return r;
}

// Tiles b, b + gridDim.x, ... of the row: their range.
__global__ __launch_bounds__(kRangeThreads) void quant_range_kernel(const float* __restrict__ vals, int64_t ld_vals,
                                                                    int64_t n, Range* __restrict__ ranges)
{
    __shared__ Range waves[kRangeThreads / 64];
    const uint32_t t = threadIdx.x;
    const float* v = vals + (int64_t)blockIdx.y * ld_vals;
    constexpr int kPer = kTile / kRangeThreads;
    Range r = {0u, 0xFFFFFFFFu};
    for (int64_t k0 = (int64_t)blockIdx.x * kTile; k0 < n; k0 += (int64_t)gridDim.x * kTile) {
        float x[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int64_t k = k0 + i * kRangeThreads + t;
            x[i] = k < n ? v[k] : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i) widen(r, x[i]);
    }
    r = wave_range(r);
    if ((t & 63u) == 0u) waves[t / 64] = r;
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < kRangeThreads / 64; ++w) {
            r.vmax = max(r.vmax, waves[w].vmax);
            r.vmin = min(r.vmin, waves[w].vmin);
        }
        ranges[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = r;
    }
}

// Codes of tiles b, b + gridDim.x, ... of the row, and the workgroup's sum and count per interval.
//  * The interval of a magnitude comes from a bisection of the edges (they descend, and when one of
//    them is not a number all behind it are not), q-1 steps instead of L-1 comparisons.
//  * A lane adds its magnitudes to sums of its own, table[interval][lane] of its wavefront: every
//    sum is formed in one order whatever the timing, and equal intervals do not queue up.
//  * Codes go through LDS bytes, so that loads are coalesced and a thread packs whole words.
// Alone and Row: the workgroup has the whole row: range, codes and means in this one launch.
// Bound by its dependent chain: q - 1 square roots and L divisions in fp64 before the first code
// (about 1 us at q = 4), LDS round trips behind it.
enum class Work { Tiles, Alone, Row };           // many workgroups to a row; rows of up to kTile; of up to row_most(q)
template <int q, Work WORK>
__global__ __launch_bounds__(64 * (WORK == Work::Row ? kRowWaves : code_waves(q))) void quant_codes_kernel(
    const float* __restrict__ vals, int64_t ld_vals, int64_t n, uint32_t* __restrict__ streams, int64_t ld_words,
    const Range* __restrict__ ranges, double* __restrict__ partial, uint32_t* __restrict__ pcount,
    float* __restrict__ means)
{
    constexpr int L = 1 << (q - 1);
    constexpr bool ALONE = WORK != Work::Tiles;
    constexpr int kWaves = WORK == Work::Row ? kRowWaves : code_waves(q), kThreads = 64 * kWaves;
    constexpr int kTile = WORK == Work::Row ? row_most(q) : mvq::kTile;
    constexpr int kPer = kTile / kThreads;
    __shared__ double   sums[kWaves * L * 64];
    __shared__ uint32_t count[kWaves * L * 64];
    __shared__ double   edges[L];
    __shared__ uint8_t  codes[kTile];
    __shared__ Range    waves[kWaves];
    const uint32_t row = blockIdx.y, t = threadIdx.x, lane = t & 63u, wave = t / 64;
    const float* v = vals + (int64_t)row * ld_vals;
    float x[kPer];
    auto load_tile = [&](int64_t k0) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int64_t k = k0 + i * kThreads + t;
            x[i] = k < n ? v[k] : 0.0f;
        }
    };
    int64_t k0 = (int64_t)blockIdx.x * kTile;
    load_tile(k0);

    // the row's range
    Range r = {0u, 0xFFFFFFFFu};
    if constexpr (ALONE) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) widen(r, x[i]);
    } else {
        for (uint32_t b = t; b < gridDim.x; b += kThreads) {
            const Range o = ranges[(size_t)row * gridDim.x + b];
            r.vmax = max(r.vmax, o.vmax);
            r.vmin = min(r.vmin, o.vmin);
        }
    }
    r = wave_range(r);
    if (lane == 0) waves[wave] = r;
    for (int i = t; i < kWaves * L * 64; i += kThreads) {
        sums[i] = 0.0;
        count[i] = 0u;
    }
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < kWaves; ++w) {
            r.vmax = max(r.vmax, waves[w].vmax);
            r.vmin = min(r.vmin, waves[w].vmin);
        }
        if (r.vmax == 0) {
            for (int l = 0; l < L; ++l) edges[l] = 0.0;
        } else {
            const double hi = (double)__uint_as_float(r.vmax), lo = (double)__uint_as_float(r.vmin);
            double alpha = hi / lo;
            for (int i = 0; i < q - 1; ++i) alpha = sqrt(alpha);
            double edge = hi;
            edges[0] = edge;
            for (int l = 1; l < L; ++l) {
                edge /= alpha;
                edges[l] = edge;
            }
        }
    }
    __syncthreads();

    uint32_t* out = streams + (int64_t)row * ld_words;
    const int64_t n_words = (n * q + 31) / 32;
    double*   my_sums = sums + wave * (L * 64) + lane;
    uint32_t* my_count = count + wave * (L * 64) + lane;
    for (;;) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (WORK == Work::Row && k0 + i * kThreads >= n) break;            // uniform
            const bool live = k0 + i * kThreads + t < n;
            const double m = (double)fabsf(x[i]);
            uint32_t l = 0;                       // interval - 1 = #{ j in 1 .. L-1 : m <= edges[j] }
#pragma unroll
            for (int s = L / 2; s >= 1; s >>= 1)
                if (m <= edges[l + s]) l += s;
            uint32_t code = 0;
            if (live) {
                code = l | ((__float_as_uint(x[i]) >> 31) << (q - 1));
                my_sums[l * 64] += m;
                my_count[l * 64] += 1u;
            }
            codes[i * kThreads + t] = (uint8_t)code;
        }
        __syncthreads();
        // word w of the tile holds stream bits [32 w, 32 w + 32): the codes that overlap it
        constexpr int kTileWords = kTile * q / 32;
        for (int w = t; w < kTileWords; w += kThreads) {
            const int first = 32 * w / q;
            uint32_t word = 0;
#pragma unroll
            for (int i = 0; i <= (31 + q) / q; ++i) {
                const int at = (first + i) * q - 32 * w;               // the code's first bit, from -q + 1 on
                const uint32_t c = (at < 32 && first + i < kTile) ? codes[first + i] : 0u;
                word |= at >= 0 ? c << (at & 31) : c >> -at;
            }
            const int64_t at = k0 / 32 * q + w;
            if (at < n_words) out[at] = word;
        }
        k0 += (int64_t)gridDim.x * kTile;
        if (ALONE || k0 >= n) break;              // uniform
        load_tile(k0);
        __syncthreads();                          // the codes' bytes are free
    }
    // the loop's barrier has passed since the last addition to the tables

    // per interval: kLanes lanes add up the columns of all wavefronts' tables, each its share in a fixed
    // order, then each other's in a fixed tree.  The columns a wavefront reads together are all different.
    constexpr int kLanes = kThreads / L >= 64 ? 64 : kThreads / L >= 1 ? kThreads / L : 1;
    for (int i = t; i < L * kLanes; i += kThreads) {
        const int l = i / kLanes, p = i % kLanes;
        double   s = 0.0;
        uint32_t c = 0;
        for (int w = 0; w < kWaves; ++w)
#pragma unroll 4
            for (int j = 0; j < 64 / kLanes; ++j) {
                const int col = (j * kLanes + p + l * kLanes) & 63;
                s += sums[(w * L + l) * 64 + col];
                c += count[(w * L + l) * 64 + col];
            }
        for (int o = kLanes / 2; o >= 1; o >>= 1) {
            s += __shfl_xor(s, o, 64);
            c += __shfl_xor(c, o, 64);
        }
        if (p == 0) {
            if constexpr (ALONE) {
                means[(int64_t)row * L + l] = c ? (float)(s / (double)c) : 0.0f;
            } else {
                partial[((size_t)row * gridDim.x + blockIdx.x) * L + l] = s;
                pcount[((size_t)row * gridDim.x + blockIdx.x) * L + l] = c;
            }
        }
    }
}

// Means of a row: one wavefront per interval; lane j adds the sums of blocks j, j + 64, ... and the
// lanes are then added in a fixed tree.
__global__ __launch_bounds__(kMeanThreads) void quant_means_kernel(const double* __restrict__ partial,
                                                                   const uint32_t* __restrict__ pcount,
                                                                   uint32_t n_blocks, int L, float* __restrict__ means)
{
    const size_t row = blockIdx.x;
    const uint32_t lane = threadIdx.x & 63u;
    for (int l = (int)(threadIdx.x / 64); l < L; l += kMeanThreads / 64) {
        double   s = 0.0;
        uint32_t c = 0;
#pragma unroll
        for (int u = 0; u < kMaxBlocks / 64; ++u) {
            const uint32_t b = lane + 64u * u;
            if (b < n_blocks) {
                s += partial[(row * n_blocks + b) * L + l];
                c += pcount[(row * n_blocks + b) * L + l];
            }
        }
        for (int o = 32; o >= 1; o >>= 1) {
            s += __shfl_xor(s, o, 64);
            c += __shfl_xor(c, o, 64);
        }
        if (lane == 0) means[row * L + l] = c ? (float)(s / (double)c) : 0.0f;
    }
}

__global__ __launch_bounds__(256) void quant_decode_kernel(const uint32_t* __restrict__ streams, int64_t ld_words,
                                                           int64_t n, int32_t q, const float* __restrict__ means,
                                                           float* __restrict__ out, int64_t ld_out)
{
    const uint32_t row = blockIdx.y;
    const int L = 1 << (q - 1);
    const uint32_t* w = streams + (int64_t)row * ld_words;
    const float* mu = means + (int64_t)row * L;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) {
        const uint64_t bit = (uint64_t)k * (uint64_t)q;
        uint32_t code = w[bit >> 5] >> (bit & 31);
        if ((bit & 31) + q > 32) code |= w[(bit >> 5) + 1] << (32 - (bit & 31));
        code &= (1u << q) - 1;
        const float m = mu[code & (uint32_t)(L - 1)];
        out[(int64_t)row * ld_out + k] = (code >> (q - 1)) ? -m : m;
    }
}

}  // namespace mvq

extern "C" {

size_t mv_quant_scratch_bytes(int64_t n, int32_t rows, int32_t q)
{
    if (n < 1 || rows < 1 || q < 2 || q > 8) return 0;
    const int64_t groups = (n + mvq::group_size(q) - 1) / mvq::group_size(q);
    return (size_t)rows * (size_t)groups * (size_t)(1 << (q - 1)) * (sizeof(double) + sizeof(uint32_t)) + 256;
}

mv_status mv_quant_encode(const float* vals, int64_t ld_vals, int64_t n, int32_t rows, int32_t q,
                          uint32_t* streams, int64_t ld_words, float* means, void* scratch, size_t scratch_bytes,
                          void* stream)
{
    if (!vals || !streams || !means || !scratch) return MV_ERR_INVALID_ARG;
    if (n < 1 || rows < 1 || rows > 65535 || q < 2 || q > 8 || ld_vals < n) return MV_ERR_INVALID_ARG;
    if (ld_words < (n * q + 31) / 32) return MV_ERR_INVALID_ARG;
    if (scratch_bytes < mv_quant_scratch_bytes(n, rows, q)) return MV_ERR_INVALID_ARG;
    const int L = 1 << (q - 1);
    const int64_t tiles = (n + mvq::kTile - 1) / mvq::kTile;
    const bool row_alone = n > mvq::kTile && n <= mvq::row_most(q);
    const uint32_t blocks = row_alone ? 1u : (uint32_t)(tiles < mvq::kMaxBlocks ? tiles : mvq::kMaxBlocks);
    // Per row and block L sums, L counts and a range, 12 L + 8 bytes: b > 1 blocks have more than
    // 64 (b - 1) >= 2 b packing groups (of at most 32 values), for each of which mv_quant_scratch_bytes counts 12 L.
    static_assert(mvq::kTile >= 64 * 32, "the blocks' records fit the scratch");
    uintptr_t base = (reinterpret_cast<uintptr_t>(scratch) + 255) & ~(uintptr_t)255;
    const size_t records = (size_t)rows * blocks;
    double* partial = reinterpret_cast<double*>(base);
    mvq::Range* ranges = reinterpret_cast<mvq::Range*>(partial + records * L);
    uint32_t* pcount = reinterpret_cast<uint32_t*>(ranges + records);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid(blocks, (uint32_t)rows);
    if (blocks > 1)
        hipLaunchKernelGGL(mvq::quant_range_kernel, grid, dim3(mvq::kRangeThreads), 0, st, vals, ld_vals, n, ranges);
#define MV_QUANT_KERNEL(Q, W, THREADS)                                                                             \
    hipLaunchKernelGGL((mvq::quant_codes_kernel<Q, mvq::Work::W>), grid, dim3(THREADS), 0, st, vals, ld_vals, n,   \
                       streams, ld_words, (const mvq::Range*)ranges, partial, pcount, means)
#define MV_QUANT_LAUNCH(Q)                                                                                         \
    case Q:                                                                                                        \
        if (blocks > 1) MV_QUANT_KERNEL(Q, Tiles, 64 * mvq::code_waves(Q));                                        \
        else MV_QUANT_KERNEL(Q, Alone, 64 * mvq::code_waves(Q));                                                   \
        break;
#define MV_QUANT_LAUNCH_ROW(Q)                                                                                     \
    case Q:                                                                                                        \
        if (row_alone) MV_QUANT_KERNEL(Q, Row, 64 * mvq::kRowWaves);                                               \
        else if (blocks > 1) MV_QUANT_KERNEL(Q, Tiles, 64 * mvq::code_waves(Q));                                   \
        else MV_QUANT_KERNEL(Q, Alone, 64 * mvq::code_waves(Q));                                                   \
        break;
    switch (q) {
        MV_QUANT_LAUNCH_ROW(2) MV_QUANT_LAUNCH_ROW(3) MV_QUANT_LAUNCH_ROW(4) MV_QUANT_LAUNCH(5)
        MV_QUANT_LAUNCH(6) MV_QUANT_LAUNCH(7) MV_QUANT_LAUNCH(8)
        default: return MV_ERR_INVALID_ARG;
    }
#undef MV_QUANT_LAUNCH_ROW
#undef MV_QUANT_LAUNCH
#undef MV_QUANT_KERNEL
    if (blocks > 1)
        hipLaunchKernelGGL(mvq::quant_means_kernel, dim3((uint32_t)rows), dim3(mvq::kMeanThreads), 0, st,
                           (const double*)partial, (const uint32_t*)pcount, blocks, L, means);
    return hipGetLastError() == hipSuccess ? MV_OK : MV_ERR_DEVICE;
}

mv_status mv_quant_decode(const uint32_t* streams, int64_t ld_words, int64_t n, int32_t rows, int32_t q,
                          const float* means, float* out, int64_t ld_out, void* stream)
{
    if (!streams || !means || !out) return MV_ERR_INVALID_ARG;
    if (n < 1 || rows < 1 || rows > 65535 || q < 2 || q > 8 || ld_out < n) return MV_ERR_INVALID_ARG;
    if (ld_words < (n * q + 31) / 32) return MV_ERR_INVALID_ARG;
    int64_t bx = (n + 255) / 256;
    if (bx > 1024) bx = 1024;
    hipLaunchKernelGGL(mvq::quant_decode_kernel, dim3((uint32_t)bx, (uint32_t)rows), dim3(256), 0,
                       static_cast<hipStream_t>(stream), streams, ld_words, n, q, means, out, ld_out);
    return hipGetLastError() == hipSuccess ? MV_OK : MV_ERR_DEVICE;
}

}  // extern "C"
