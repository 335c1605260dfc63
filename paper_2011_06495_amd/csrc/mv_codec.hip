// Sparse position code of the paper's Sec. 4.3.1 on the GPU: encoder and decoder
// for batches of ascending coordinate lists (the workers' votes, the add / drop
// lists, the global mask).
//
// Stream of one list: the vector's d coordinates are cut into blocks of
// block_len = 1/phi; per listed position a 1 bit followed by the position inside
// its block in B = ceil(log2(block_len)) bits, most significant first; a 0 bit
// closes every block.  Bit k of a stream is bit k % 32 of its word k / 32.
// With n positions the stream has n (1 + B) + ceil(d / block_len) bits.
//
// Encoder: position i of the list lies in block b_i = idx[i] / block_len and is
// preceded by i codes and b_i closing bits, so its code starts at bit
// i (1 + B) + b_i -- no prefix sum is needed.  A workgroup owns kTileWords words of a
// stream: two of its wavefronts find the list entries whose codes reach into them, by a
// 64-ary search over that increasing function, all threads put these codes together
// in LDS, and the words are stored once: no atomics in memory, no clearing pass.
//
// Decoder: the receiver's parse is a finite automaton (state = offset bits still
// to skip, 0..B).  Every 64-bit chunk of the stream becomes a map from entry state to
// (exit state, codes begun); composing these maps along the stream gives every chunk
// its true entry state and the number of codes before it; then each chunk is parsed for
// real and writes coordinate = closed blocks * block_len + offset at its place in the
// list.  Closed blocks are not counted: a flag at stream bit p with c codes before it
// has p - c (1 + B) closing bits before it.
#include "../../include/mv.h"

#include <mutex>
#include <utility>

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mvc {

constexpr int kThreads = 256;
constexpr int kMaxB = 31;
constexpr int kChunkBits = 64;
constexpr int kTileChunks = kThreads;          // chunks a workgroup maps at a time, one per thread
constexpr int kGroupChunks = 16;               // chunks composed by one thread
constexpr int kGroups = kTileChunks / kGroupChunks;
constexpr int kMaxTiles = 256;                 // per row: longer streams give every workgroup several runs of kTileChunks
constexpr int kTileGroup = 16;                 // tiles composed by one thread

__host__ __device__ inline int offset_bits(int64_t block_len)
{
    int b = 0;
    while (((int64_t)1 << b) < block_len) ++b;
    return b;
}

// first bit of the code of list entry i
__device__ __forceinline__ uint64_t code_start(const uint32_t* __restrict__ idx, uint32_t i, uint32_t code_len,
                                               uint32_t block_len)
{
    return (uint64_t)i * code_len + idx[i] / block_len;
}

constexpr int kTileWords = kThreads;

// The first i in [0, n) with pred(i), n if there is none; pred is false up to some point and true from there
// on.  64 probes at a time: a list of 11,174 entries takes three loads, one after the other, where a
// bisection takes fourteen.  All lanes of the wavefront must call it.
template <typename Pred>
__device__ __forceinline__ uint32_t wave_lower_bound(uint32_t n, Pred pred)
{
    uint32_t lo = 0, hi = n;
    const uint32_t lane = threadIdx.x & 63u;
    while (lo < hi) {                                    // uniform
        const uint32_t step = (hi - lo + 63) / 64;
        const uint32_t last = (hi - lo - 1) / step;      // lanes 0 .. last probe lo, lo + step, ...
        const uint64_t yes = __ballot(lane <= last && pred(lo + min(lane, last) * step));
        const uint32_t first = yes ? (uint32_t)__builtin_ctzll(yes) : last + 1;
        if (yes) hi = lo + first * step;
        if (first) lo += (first - 1) * step + 1;
    }
    return lo;
}

// Bound by its chain: the search, one load of the entries, LDS (16 lists of 11,174: 4.2 us, 6.5 when every thread
// bisected for its own word; 10 lists of 111,740: 7.1 and 13.7).
__global__ __launch_bounds__(kThreads) void codec_encode_kernel(
    const uint32_t* __restrict__ idx, int64_t ld_idx, const uint32_t* __restrict__ counts, int64_t counts_stride,
    uint32_t n_fixed, int64_t d, uint32_t block_len, uint32_t B, uint32_t* __restrict__ streams, int64_t ld_words,
    unsigned long long* __restrict__ n_bits_out)
{
    __shared__ uint32_t words[kTileWords];
    __shared__ uint32_t range[2];
    const uint32_t row = blockIdx.y, t = threadIdx.x;
    // a length read from device memory is wire-side data: never trusted beyond the row's storage
    const uint32_t n = counts ? min(counts[(int64_t)row * counts_stride], n_fixed) : n_fixed;
    const uint32_t code_len = 1 + B;
    const uint64_t n_blocks = ((uint64_t)d + block_len - 1) / block_len;
    const uint64_t total = (uint64_t)n * code_len + n_blocks;
    const uint64_t n_words = (total + 31) / 32;
    const uint32_t* list = idx + (int64_t)row * ld_idx;
    if (blockIdx.x == 0 && t == 0) n_bits_out[row] = total;
    for (uint64_t w0 = (uint64_t)blockIdx.x * kTileWords; w0 < n_words; w0 += (uint64_t)gridDim.x * kTileWords) {
        const uint64_t lo_bit = w0 * 32, hi_bit = lo_bit + 32 * kTileWords;
        words[t] = 0;
        if (t < 128) {                                   // whole wavefronts
            // the first entry whose code ends beyond the tile's first bit, the first that begins behind its last
            const uint64_t bit = t < 64 ? lo_bit : hi_bit + code_len - 1;
            const uint32_t r = wave_lower_bound(n, [&](uint32_t i) {
                return code_start(list, i, code_len, block_len) + code_len > bit;
            });
            if ((t & 63u) == 0) range[t / 64] = r;
        }
        __syncthreads();
        for (uint32_t i = range[0] + t; i < range[1]; i += kThreads) {
            const uint32_t pos = list[i], off = pos % block_len;
            // where the code begins in the tile; a list that is not ascending may give any place
            const int64_t at = (int64_t)((uint64_t)i * code_len + pos / block_len) - (int64_t)lo_bit;
            if (at <= -(int64_t)code_len || at >= 32 * kTileWords) continue;
            // the code as it lies in the stream, first bit in bit 0: the flag, then the offset MSB first
            uint64_t code = 1ull | ((uint64_t)(B ? (__brev(off) >> (32 - B)) : 0u) << 1);
            uint32_t w = 0, sh = 0;
            if (at < 0) {
                code >>= -at;                            // (at most 31)
            } else {
                w = (uint32_t)at / 32;
                sh = (uint32_t)at % 32;
            }
            code <<= sh;                                 // at most 32 + 31 bits
            if ((uint32_t)code) atomicOr(&words[w], (uint32_t)code);
            if ((code >> 32) != 0 && w + 1 < (uint32_t)kTileWords) atomicOr(&words[w + 1], (uint32_t)(code >> 32));
        }
        __syncthreads();
        if (w0 + t < n_words) streams[(int64_t)row * ld_words + w0 + t] = words[t];
        __syncthreads();                                 // the words are free for the next tile
    }
}

// ---- decoder -----------------------------------------------------------------
// The chain is what costs, not the bytes (10 streams of 1 Mbit are 1.3 MB), so the stream is
// cut finely -- 256 chunks per workgroup -- and composed in levels: chunks to groups of 16,
// groups to a tile, tiles to the row.  Two launches: maps of every level; then every workgroup
// walks the tile maps before its own, its groups and its chunks, and emits.  A stream of one
// tile takes one launch and no scratch.  10 lists of 111,740 positions, B = 7: 140 us when one
// workgroup per row composed all chunks, 15 us so (maps 6.2, emission 9.8).
//
// A map entry is exit state | codes begun << kStateBits: 16 bits for a chunk (at most 64 codes), 32
// for a group or a tile.  27 bits of codes hold a tile of any stream of up to 2^35 bits; more than 2^32
// codes counts_out could not say.

constexpr int kStateBits = 5;
static_assert(kMaxB < 1 << kStateBits, "a state fits its bits");
__device__ __forceinline__ uint32_t map_exit(uint32_t m) { return m & ((1u << kStateBits) - 1u); }
__device__ __forceinline__ uint32_t map_codes(uint32_t m) { return m >> kStateBits; }
// entry `m` (state reached, codes so far) carried on through `next`, the map's value at that state
__device__ __forceinline__ uint32_t carry(uint32_t m, uint32_t next) { return m - map_exit(m) + next; }

// stream words i, i + 1, i + 2 with the bits at or beyond `total` read as zero
struct ChunkBits {
    uint64_t lo;                 // the chunk, first bit in bit 0
    uint32_t hi;                 // the 32 bits behind it (an offset may reach into them)
};
__device__ __forceinline__ ChunkBits load_chunk(const uint32_t* __restrict__ words, uint64_t chunk, uint64_t total)
{
    const uint64_t n_words = (total + 31) / 32, i = chunk * 2;
    uint32_t w[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        w[u] = i + u < n_words ? words[i + u] : 0u;
        if ((i + u + 1) * 32 > total && i + u < n_words) w[u] &= (1u << (total & 31u)) - 1u;
    }
    return ChunkBits{(uint64_t)w[1] << 32 | w[0], w[2]};
}

// The chunk's map for entry states 0..B into tab[state * pitch]: backwards over the bits,
// f(j) = what happens from bit j on when a flag is due there, = f(j + 1) behind a 0 and one
// code more than f(j + 1 + B) behind a 1; entering with s offset bits to skip is f(s).  With B
// known the last B + 1 values stay in registers: three instructions per bit, no divergence.
template <int B>
__device__ __forceinline__ void chunk_map(uint64_t bits, uint16_t* tab, uint32_t pitch)
{
    uint32_t f[kChunkBits + 1 + B];
#pragma unroll
    for (int i = 0; i <= B; ++i) f[kChunkBits + i] = (uint32_t)i;
#pragma unroll
    for (int j = kChunkBits - 1; j >= 0; --j) {
        const uint32_t word = j >= 32 ? (uint32_t)(bits >> 32) : (uint32_t)bits;
        f[j] = (word >> (j & 31)) & 1u ? f[j + 1 + B] + (1u << kStateBits) : f[j + 1];
    }
#pragma unroll
    for (int s = 0; s <= B; ++s) tab[s * pitch] = (uint16_t)f[s];
}

// LDS of the maps of up to kTileChunks chunks
struct TileLds {
    uint16_t chunk[(kMaxB + 1) * kTileChunks];    // [state][chunk], pitch = the chunks there are
    uint32_t group[kGroups][kMaxB + 1];
};

// group maps from the chunk maps; all threads, ends without a barrier
__device__ __forceinline__ void compose_groups(TileLds& lds, uint32_t n_chunks, uint32_t n_states)
{
    for (uint32_t i = threadIdx.x; i < kGroups * n_states; i += kThreads) {
        const uint32_t g = i / n_states, s = i % n_states;
        const uint32_t c1 = min((g + 1) * kGroupChunks, n_chunks);
        uint32_t m = s;
        for (uint32_t c = g * kGroupChunks; c < c1; ++c) m = carry(m, lds.chunk[map_exit(m) * n_chunks + c]);
        lds.group[g][s] = m;
    }
}

struct WalkLds {
    uint32_t group_entry[kGroups + 1];            // as a map's entries: state, codes from the start of the run
    uint32_t chunk_entry[kTileChunks];
};

// Entries of the run's groups and chunks from `state`, the run's entry state; returns (to all) the run's
// exit, as a map's entry.  The maps must be in LDS, a barrier behind them.
__device__ __forceinline__ uint32_t walk_run(const TileLds& lds, WalkLds& walk, uint32_t n_chunks, uint32_t state)
{
    const uint32_t t = threadIdx.x;
    if (t == 0) {
        uint32_t m = state;
        for (uint32_t g = 0; g < (uint32_t)kGroups; ++g) {
            walk.group_entry[g] = m;
            m = carry(m, lds.group[g][map_exit(m)]);
        }
        walk.group_entry[kGroups] = m;
    }
    __syncthreads();
    if (t < (uint32_t)kGroups) {
        uint32_t m = walk.group_entry[t];
        const uint32_t c1 = min((t + 1) * kGroupChunks, n_chunks);
        for (uint32_t c = t * kGroupChunks; c < c1; ++c) {
            walk.chunk_entry[c] = m;
            m = carry(m, lds.chunk[map_exit(m) * n_chunks + c]);
        }
    }
    __syncthreads();
    return walk.group_entry[kGroups];
}

// Parses a chunk for real, entering with `state` offset bits to skip and `codes` codes before it.
__device__ __forceinline__ void emit_chunk(ChunkBits c, uint64_t first_bit, uint32_t state, uint32_t codes, uint32_t B,
                                           int64_t d, uint32_t block_len, uint32_t* __restrict__ out, uint32_t max_n)
{
    uint32_t j = state;
    while (j < (uint32_t)kChunkBits) {
        const uint64_t rest = c.lo >> j;
        if (rest == 0) break;                          // only closing bits are left
        j += (uint32_t)__builtin_ctzll(rest);          // the next code's flag
        // the offset lies MSB first in the stream and may run into the next chunk
        const uint32_t sh = j + 1;
        uint64_t v = sh < 64 ? c.lo >> sh : 0;
        if (sh + B > 64) v |= (uint64_t)c.hi << (64 - sh);               // B <= 31, so 64 - sh < 32
        const uint32_t off = B ? __brev((uint32_t)v) >> (32 - B) : 0u;
        const uint64_t closed = first_bit + j - (uint64_t)codes * (1 + B);
        const uint64_t pos = closed * block_len + off;
        if (codes < max_n && pos < (uint64_t)d) out[codes] = (uint32_t)pos;
        ++codes;
        j += 1 + B;
    }
}

// Scratch of a row: chunk maps (per run of kTileChunks chunks [state][chunk]), group maps
// (per run [group][state]), tile maps ([tile][state]).
struct Scratch {
    uint32_t* base;
    uint64_t  chunk_words, group_words, tile_words;   // 32-bit words of each per row
    __device__ uint32_t* chunks(uint32_t row, uint64_t run, uint32_t n_states) const
    {
        return base + (uint64_t)row * (chunk_words + group_words + tile_words) + run * (kTileChunks / 2) * n_states;
    }
    __device__ uint32_t* groups(uint32_t row, uint64_t run, uint32_t n_states) const
    {
        return chunks(row, 0, n_states) + chunk_words + run * kGroups * n_states;
    }
    __device__ uint32_t* tiles(uint32_t row, uint32_t n_states) const
    {
        return chunks(row, 0, n_states) + chunk_words + group_words;
    }
};

// Workgroup (tile, row): the maps of the tile's `runs` runs of kTileChunks chunks, and the tile's.
// `alone` (the row is one run): emits as well, nothing goes to scratch.
template <int B>
__global__ __launch_bounds__(kThreads) void codec_maps_kernel(
    const uint32_t* __restrict__ streams, int64_t ld_words, const unsigned long long* __restrict__ n_bits,
    uint64_t max_bits, uint64_t runs, Scratch scratch, int alone, int64_t d, uint32_t block_len,
    uint32_t* __restrict__ idx_out, int64_t ld_idx, uint32_t max_n, uint32_t* __restrict__ counts_out)
{
    __shared__ TileLds lds;
    __shared__ WalkLds walk;
    constexpr uint32_t n_states = B + 1;
    const uint32_t row = blockIdx.y, t = threadIdx.x;
    // the received length is wire-side data: clamped to what the scratch was sized for
    const uint64_t total = min((uint64_t)n_bits[row], max_bits);
    const uint64_t n_chunks = (total + kChunkBits - 1) / kChunkBits;
    const uint32_t* words = streams + (int64_t)row * ld_words;
    uint32_t tile_map = t;                        // thread t < n_states: the tile's map at entry state t so far
    for (uint64_t run = blockIdx.x * runs; run < (blockIdx.x + 1) * runs; ++run) {
        const uint64_t c0 = run * kTileChunks;
        if (c0 >= n_chunks && !alone) break;      // uniform
        const uint32_t n = (uint32_t)min((uint64_t)kTileChunks, n_chunks - c0);
        ChunkBits bits = {0, 0};
        if (t < n) {
            bits = load_chunk(words, c0 + t, total);
            chunk_map<B>(bits.lo, lds.chunk + t, n);
        }
        __syncthreads();
        compose_groups(lds, n, n_states);
        if (!alone) {
            uint32_t* to = scratch.chunks(row, run, n_states);
            const uint32_t* from = reinterpret_cast<const uint32_t*>(lds.chunk);
            for (uint32_t i = t; i < (n * n_states + 1) / 2; i += kThreads) to[i] = from[i];
        }
        __syncthreads();
        if (alone) {
            const uint32_t end = walk_run(lds, walk, n, 0);
            if (t < n) {
                const uint32_t m = walk.chunk_entry[t];
                emit_chunk(bits, (uint64_t)t * kChunkBits, map_exit(m), map_codes(m), B, d, block_len,
                           idx_out + (int64_t)row * ld_idx, max_n);
            }
            if (t == 0) counts_out[row] = map_codes(end);
            return;
        }
        uint32_t* to = scratch.groups(row, run, n_states);
        for (uint32_t i = t; i < kGroups * n_states; i += kThreads) to[i] = lds.group[i / n_states][i % n_states];
        if (t < n_states)
            for (uint32_t g = 0; g < (uint32_t)kGroups; ++g) tile_map = carry(tile_map, lds.group[g][map_exit(tile_map)]);
        __syncthreads();                          // the tables are free for the next run
    }
    if (t < n_states) scratch.tiles(row, n_states)[(uint64_t)blockIdx.x * n_states + t] = tile_map;
}

struct EmitLds {
    TileLds  tile;
    WalkLds  walk;
    // 16 tiles composed: exit states, codes (which need not fit the bits of a map entry)
    uint8_t  tg_exit[kMaxTiles / kTileGroup][kMaxB + 1];
    uint32_t tg_codes[kMaxTiles / kTileGroup][kMaxB + 1];
    uint32_t entry_state, entry_codes;
};

// Workgroup (tile, row): the tile's entry from the maps of the tiles before it, then its chunks' entries
// and their codes.  The row's last tile also knows how many codes there are.
__global__ __launch_bounds__(kThreads) void codec_emit_kernel(
    const uint32_t* __restrict__ streams, int64_t ld_words, const unsigned long long* __restrict__ n_bits,
    uint64_t max_bits, uint64_t runs, Scratch scratch, uint32_t B, int64_t d, uint32_t block_len,
    uint32_t* __restrict__ idx_out, int64_t ld_idx, uint32_t max_n, uint32_t* __restrict__ counts_out)
{
    __shared__ EmitLds lds;
    extern __shared__ uint32_t tile_maps[];       // gridDim.x * n_states
    const uint32_t row = blockIdx.y, t = threadIdx.x, n_states = B + 1, tile = blockIdx.x;
    const uint64_t total = min((uint64_t)n_bits[row], max_bits);
    const uint64_t n_chunks = (total + kChunkBits - 1) / kChunkBits;
    const uint64_t n_runs = (n_chunks + kTileChunks - 1) / kTileChunks;
    if (n_runs == 0 && tile == 0 && t == 0) counts_out[row] = 0;
    if (tile * runs >= n_runs) return;            // whole workgroup
    const uint32_t* words = streams + (int64_t)row * ld_words;

    // what the first run needs is fetched beside the tile maps
    ChunkBits bits = {0, 0};
    uint32_t  n = 0;
    auto fetch_run = [&](uint64_t run) {
        n = (uint32_t)min((uint64_t)kTileChunks, n_chunks - run * kTileChunks);
        bits = t < n ? load_chunk(words, run * kTileChunks + t, total) : ChunkBits{0, 0};
        const uint32_t* from = scratch.chunks(row, run, n_states);
        uint32_t* to = reinterpret_cast<uint32_t*>(lds.tile.chunk);
#pragma unroll 4
        for (uint32_t i = t; i < (n * n_states + 1) / 2; i += kThreads) to[i] = from[i];
        const uint32_t* groups = scratch.groups(row, run, n_states);
        for (uint32_t i = t; i < kGroups * n_states; i += kThreads) lds.tile.group[i / n_states][i % n_states] = groups[i];
    };
    const uint32_t* maps = scratch.tiles(row, n_states);
#pragma unroll 4
    for (uint32_t i = t; i < tile * n_states; i += kThreads) tile_maps[i] = maps[i];
    fetch_run(tile * runs);
    __syncthreads();
    const uint32_t n_tile_groups = tile / kTileGroup;
    for (uint32_t i = t; i < n_tile_groups * n_states; i += kThreads) {
        const uint32_t g = i / n_states, s = i % n_states;
        uint32_t st = s, sum = 0;
        for (uint32_t k = g * kTileGroup; k < (g + 1) * kTileGroup; ++k) {
            const uint32_t m = tile_maps[k * n_states + st];
            sum += map_codes(m);
            st = map_exit(m);
        }
        lds.tg_exit[g][s] = (uint8_t)st;
        lds.tg_codes[g][s] = sum;
    }
    __syncthreads();
    if (t == 0) {
        uint32_t st = 0, sum = 0;
        for (uint32_t g = 0; g < n_tile_groups; ++g) {
            sum += lds.tg_codes[g][st];
            st = lds.tg_exit[g][st];
        }
        for (uint32_t k = n_tile_groups * kTileGroup; k < tile; ++k) {
            const uint32_t m = tile_maps[k * n_states + st];
            sum += map_codes(m);
            st = map_exit(m);
        }
        lds.entry_state = st;
        lds.entry_codes = sum;
    }
    __syncthreads();
    uint32_t state = lds.entry_state, codes = lds.entry_codes;
    for (uint64_t run = tile * runs;;) {
        const uint32_t end = walk_run(lds.tile, lds.walk, n, state);
        if (t < n) {
            const uint32_t m = lds.walk.chunk_entry[t];
            emit_chunk(bits, (run * kTileChunks + t) * kChunkBits, map_exit(m), codes + map_codes(m), B, d, block_len,
                       idx_out + (int64_t)row * ld_idx, max_n);
        }
        state = map_exit(end);
        codes += map_codes(end);
        if (++run >= n_runs) {
            if (t == 0) counts_out[row] = codes;
            return;
        }
        if (run == (tile + 1) * runs) return;
        __syncthreads();                          // the tables are free for the next run
        fetch_run(run);
        __syncthreads();
    }
}

// Host side of the scratch: 108 bytes per chunk is what mv_codec_scratch_bytes counts.  Used are, with
// S <= 32 states: 2 S bytes per chunk, and 4 (kGroups + 1) S bytes per run of 256 chunks (rounded up),
// at most 64 c + 2176 (c / 256 + 1) < 108 c for the c > 256 chunks of a stream that needs scratch.
constexpr uint64_t kScratchPerChunk = 108;

// the instance of codec_maps_kernel for this B, 0 .. kMaxB
template <int... Bs, typename... Args>
void launch_maps(uint32_t B, std::integer_sequence<int, Bs...>, dim3 grid, hipStream_t st, Args... args)
{
    (void)((B == (uint32_t)Bs
                ? (codec_maps_kernel<Bs><<<grid, dim3(kThreads), 0, st>>>(args...), true)
                : false) || ...);
}

}  // namespace mvc

extern "C" {

uint64_t mv_codec_stream_bits(int64_t n, int64_t d, int64_t block_len)
{
    if (n < 0 || d < 1 || block_len < 1 || block_len > 0x7FFFFFFFll || d > 0x7FFFFFFFll || n > d) return 0;
    return (uint64_t)n * (uint64_t)(1 + mvc::offset_bits(block_len)) + (uint64_t)((d + block_len - 1) / block_len);
}

size_t mv_codec_scratch_bytes(uint64_t max_bits, int32_t rows)
{
    if (rows < 1) return 0;
    const uint64_t chunks = (max_bits + mvc::kChunkBits - 1) / mvc::kChunkBits;
    return (size_t)rows * chunks * mvc::kScratchPerChunk + 512;
}

mv_status mv_codec_encode(const uint32_t* idx, int64_t ld_idx, const uint32_t* counts, int64_t counts_stride,
                          int64_t n, int32_t rows, int64_t d, int64_t block_len, uint32_t* streams,
                          int64_t ld_words, uint64_t* n_bits, void* stream)
{
    if (!idx || !streams || !n_bits || rows < 1 || rows > 65535) return MV_ERR_INVALID_ARG;
    if (d < 1 || d > 0x7FFFFFFFll || block_len < 1 || block_len > d || n < 0 || n > d || ld_idx < n)
        return MV_ERR_INVALID_ARG;
    if (counts && counts_stride < 1) return MV_ERR_INVALID_ARG;
    const uint64_t max_bits = mv_codec_stream_bits(n, d, block_len);
    const uint64_t max_words = (max_bits + 31) / 32;
    if ((uint64_t)ld_words < max_words) return MV_ERR_INVALID_ARG;
    uint64_t bx = (max_words + mvc::kThreads - 1) / mvc::kThreads;
    if (bx > 4096) bx = 4096;
    if (bx < 1) bx = 1;
    hipLaunchKernelGGL(mvc::codec_encode_kernel, dim3((uint32_t)bx, (uint32_t)rows), dim3(mvc::kThreads), 0,
                       static_cast<hipStream_t>(stream), idx, ld_idx, counts, counts_stride, (uint32_t)n, d,
                       (uint32_t)block_len, (uint32_t)mvc::offset_bits(block_len), streams, ld_words,
                       reinterpret_cast<unsigned long long*>(n_bits));
    return hipGetLastError() == hipSuccess ? MV_OK : MV_ERR_DEVICE;
}

// ---- the decoder's scratch for callers that cannot allocate -----------------
// One array per GPU, there from the moment the library's code is loaded on that GPU
// until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; what kernels and copies are given is the address that call
// returns for the device that is current, kept per device below.
static __device__ __align__(256) unsigned char scratch[MV_CODEC_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void*      g_scratch_ptr[kMaxDevices];      // the array's address on each device, once asked for

// The address of `scratch` on the current device; asked for once per device.
mv_status static_scratch_of_current_device(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return MV_ERR_DEVICE;
    if (dev >= kMaxDevices) return MV_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return MV_ERR_DEVICE;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return MV_OK;
}
}  // namespace

static mv_status decode_with_scratch(const uint32_t* streams, int64_t ld_words, const uint64_t* n_bits,
                                     uint64_t max_bits, int32_t rows, int64_t d, int64_t block_len,
                                     uint32_t* idx_out, int64_t ld_idx, int64_t max_n, uint32_t* counts_out,
                                     void* scratch, void* stream)
{
    const uint64_t max_chunks = (max_bits + mvc::kChunkBits - 1) / mvc::kChunkBits;
    const uint64_t max_runs = (max_chunks + mvc::kTileChunks - 1) / mvc::kTileChunks;
    const uint64_t runs = (max_runs + mvc::kMaxTiles - 1) / mvc::kMaxTiles;      // per tile
    const uint32_t tiles = (uint32_t)((max_runs + runs - 1) / runs);
    const uint32_t B = (uint32_t)mvc::offset_bits(block_len), n_states = B + 1;
    uintptr_t base = (reinterpret_cast<uintptr_t>(scratch) + 255) & ~(uintptr_t)255;
    mvc::Scratch sc;
    sc.base = reinterpret_cast<uint32_t*>(base);
    sc.chunk_words = (max_chunks * n_states + 1) / 2;
    sc.group_words = max_runs * mvc::kGroups * n_states;
    sc.tile_words = (uint64_t)tiles * n_states;
    const int alone = max_runs == 1;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const unsigned long long* nb = reinterpret_cast<const unsigned long long*>(n_bits);
    const dim3 grid(tiles, (uint32_t)rows);
    mvc::launch_maps(B, std::make_integer_sequence<int, mvc::kMaxB + 1>(), grid, st, streams, ld_words, nb, max_bits,
                     runs, sc, alone, d, (uint32_t)block_len, idx_out, ld_idx, (uint32_t)max_n, counts_out);
    if (!alone)
        hipLaunchKernelGGL(mvc::codec_emit_kernel, grid, dim3(mvc::kThreads), tiles * n_states * 4, st, streams,
                           ld_words, nb, max_bits, runs, sc, B, d, (uint32_t)block_len, idx_out, ld_idx,
                           (uint32_t)max_n, counts_out);
    return hipGetLastError() == hipSuccess ? MV_OK : MV_ERR_DEVICE;
}

static bool decode_args_valid(const uint32_t* streams, int64_t ld_words, const uint64_t* n_bits, uint64_t max_bits,
                              int32_t rows, int64_t d, int64_t block_len, const uint32_t* idx_out, int64_t ld_idx,
                              int64_t max_n, const uint32_t* counts_out)
{
    if (!streams || !n_bits || !idx_out || !counts_out || rows < 1 || rows > 65535) return false;
    if (d < 1 || d > 0x7FFFFFFFll || block_len < 1 || block_len > d || max_n < 0 || ld_idx < max_n ||
        max_n > 0xFFFFFFFFll)
        return false;
    if (ld_words < 0 || (uint64_t)ld_words * 32 < max_bits) return false;
    return max_bits != 0;
}

mv_status mv_codec_decode(const uint32_t* streams, int64_t ld_words, const uint64_t* n_bits, uint64_t max_bits,
                          int32_t rows, int64_t d, int64_t block_len, uint32_t* idx_out, int64_t ld_idx,
                          int64_t max_n, uint32_t* counts_out, void* scratch, size_t scratch_bytes, void* stream)
{
    if (!scratch || !decode_args_valid(streams, ld_words, n_bits, max_bits, rows, d, block_len, idx_out, ld_idx,
                                       max_n, counts_out))
        return MV_ERR_INVALID_ARG;
    if (scratch_bytes < mv_codec_scratch_bytes(max_bits, rows)) return MV_ERR_INVALID_ARG;
    return decode_with_scratch(streams, ld_words, n_bits, max_bits, rows, d, block_len, idx_out, ld_idx, max_n,
                               counts_out, scratch, stream);
}

mv_status mv_codec_decode_static(const uint32_t* streams, int64_t ld_words, const uint64_t* n_bits,
                                 uint64_t max_bits, int32_t rows, int64_t d, int64_t block_len, uint32_t* idx_out,
                                 int64_t ld_idx, int64_t max_n, uint32_t* counts_out, void* stream)
{
    if (!decode_args_valid(streams, ld_words, n_bits, max_bits, rows, d, block_len, idx_out, ld_idx, max_n,
                           counts_out))
        return MV_ERR_INVALID_ARG;
    if (mv_codec_scratch_bytes(max_bits, rows) > (size_t)MV_CODEC_STATIC_SCRATCH_BYTES) return MV_ERR_UNSUPPORTED;
    void* ptr = nullptr;
    const mv_status got = static_scratch_of_current_device(&ptr);
    if (got != MV_OK) return got;
    // the kernels write every scratch entry they later read: nothing of the last call's contents matters
    return decode_with_scratch(streams, ld_words, n_bits, max_bits, rows, d, block_len, idx_out, ld_idx, max_n,
                               counts_out, ptr, stream);
}

}  // extern "C"
