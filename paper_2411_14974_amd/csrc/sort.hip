// Tile binning and ordering (gfx950): the pair-offset scan, a stable LSD
// radix sort of (u32 key, u32 value) pairs, (cell, convex) pair emission and
// per-cell list ranges.
//
// The front-to-back order within a tile (paper Sec. 3.2: convexes sorted by
// increasing distance) comes from a two-stage LSD sort of the (cell | depth)
// key: the depth digits are sorted once over the N convexes, the convexes are
// expanded into (cell, convex) pairs in that order, and a stable sort of the
// pairs on the cell digits alone completes the lexicographic order.  This moves
// the depth passes from the pairs to the N convexes, and a pair carries the
// mask of the cell's tiles (see FrameHeader), so that the pairs are a quarter
// of the (tile, convex) pairs.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.hpp"

namespace cs {

// ----------------------------------------------------------------- scan ----

constexpr int SCAN_BLOCK = 256;
// Instances per thread: few enough that the chip has a few hundred workgroups
// (a thread's gathers are one latency each), many enough that the tiles' claims
// and look-back chain stay short.  us with 4 / 8 / 16: 20k 8 / 10 / 14, 100k 9.4 /
// 10.7 / 14.6, 317k 16 / 14 / 16, 1M 40 / 32 / 29.
inline int scan_items(uint32_t n) { return n <= 160u * 1024 ? 4 : n <= 640u * 1024 ? 8 : 16; }
inline size_t scan_tiles(uint32_t n, int items) { return ((size_t)n + SCAN_BLOCK * items - 1) / (SCAN_BLOCK * items); }

__device__ __forceinline__ int lds_pad(int i) { return i + (i >> 5); }

// Sum of two counts of cell pairs that are at most MAX_CELL_PAIRS, saturating
// there.  A call that goes beyond is refused, but its count must arrive: one
// convex can make 2^20 pairs (16384 x 16384 in tiles of 8), 4096 of them 2^32.
__device__ __forceinline__ uint32_t add_cells(uint32_t a, uint32_t b) { return min(a + b, MAX_CELL_PAIRS); }
// Sum of two counts of tile pairs, saturating at 2^32 - 1 (a call's cell pairs
// can stand for 2^34).
__device__ __forceinline__ uint32_t add_tiles(uint32_t a, uint32_t b) { return a + b < a ? 0xFFFFFFFFu : a + b; }

// Exclusive scan of the block's SCAN_ITEMS values per thread held in LDS
// (padded layout); returns the block total.  The sum of a wavefront's values is
// at most 2^30 and a little; sums over wavefronts saturate at MAX_CELL_PAIRS.
template <int SCAN_ITEMS>
__device__ uint32_t block_scan_lds(uint32_t *s, uint32_t *s_wave)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t v[SCAN_ITEMS], sum = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        v[k] = s[lds_pad(tid * SCAN_ITEMS + k)];
        sum += v[k];
    }
    // inclusive wave scan of the per-thread sums
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t wbase = 0, total = 0;
    for (int w = 0; w < SCAN_BLOCK / 64; ++w) {
        const uint32_t c = min(s_wave[w], MAX_CELL_PAIRS);
        if (w < wave) wbase = add_cells(wbase, c);
        total = add_cells(total, c);
    }
    uint32_t run = wbase + incl - sum; // (below 2^32)
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        s[lds_pad(tid * SCAN_ITEMS + k)] = run;
        run += v[k];
    }
    __syncthreads();
    return total;
}

// (cell, convex) pair counts in depth order and their exclusive scan (the pair offsets), in
// one pass: each workgroup claims the next tile of ranks, gathers
// the binning records bins[sorted_ids[r]] (copied out in depth order for the
// pair emission) and their pair counts, scans the counts in LDS, publishes the tile's sum and
// finds its prefix by a decoupled look-back in which one wave reads 64
// predecessors' 64-bit status words at a time.  The last tile stores the total.
// A status word: state in bits 62-63, cell pairs in bits 32-61, tile pairs below
// (both saturating).
constexpr uint64_t SS_AGG = 1ull << 62, SS_INC = 2ull << 62, SS_VAL = SS_AGG - 1ull;
__device__ __forceinline__ uint64_t ss_pack(uint32_t cells, uint32_t tiles) { return ((uint64_t)cells << 32) | tiles; }
constexpr uint32_t SS_SPIN_LIMIT = 1u << 22;

__device__ __forceinline__ uint64_t ss_load(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ss_store(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The counts of cell pairs m and of tile pairs, where the host and the pair pass
// look for them.
__device__ __forceinline__ void store_pair_counts(uint32_t *counters, uint32_t m, uint32_t tiles, unsigned long long *host_word,
                                                  uint32_t tag, uint32_t capacity)
{
    counters[CNT_PAIRS] = m;
    counters[CNT_TILE_PAIRS] = tiles;
    if (capacity) { // the pair pass's count, clamped to the buffers, and the overflow flag
        counters[CNT_PAIRS_EFF] = m < capacity ? m : capacity;
        counters[CNT_OVERFLOW] = m > capacity ? 1u : 0u;
    }
    if (host_word) {
        const unsigned long long tg = (unsigned long long)tag << 32;
        __hip_atomic_store(host_word + 1, tg | tiles, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(host_word, tg | m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// host_word (nullable): two words of coherent pinned host memory that also
// receive the counts of cell and tile pairs, each as tag << 32 | count: the
// host waits for its tag there, with no copy or event in the stream.
template <int SCAN_ITEMS>
__global__ __launch_bounds__(SCAN_BLOCK) void gather_scan_kernel(
    uint32_t n, const uint32_t *__restrict__ sorted_ids, const uint4 *__restrict__ bins,
    uint4 *__restrict__ bins_sorted, uint32_t *__restrict__ counts_sorted, uint32_t *__restrict__ offsets,
    uint32_t *__restrict__ counters, uint64_t *__restrict__ status, unsigned long long *__restrict__ host_word,
    uint32_t tag, uint32_t capacity, ZeroSpans zero)
{
    zero_share(zero); // the cell ranges, when this scan also prepares the pair pass
    constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;
    __shared__ uint32_t s[SCAN_TILE + SCAN_TILE / 32];
    __shared__ uint32_t s_wave[SCAN_BLOCK / 64];
    __shared__ uint32_t s_tile;
    __shared__ uint32_t s_excl;
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid == 0) s_tile = atomicAdd(&counters[CNT_SCAN_TILE], 1u);
    __syncthreads();
    const uint32_t t = s_tile;
    const size_t base = (size_t)t * SCAN_TILE;
    if (base >= n) return;
    uint32_t tile_pairs = 0, id[SCAN_ITEMS];
    uint4 b[SCAN_ITEMS];
    // (all the loads before the first use, at clamped places: one latency for
    // each of the two chains instead of one per item)
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) id[k] = sorted_ids[min(base + (size_t)k * SCAN_BLOCK + tid, (size_t)n - 1)];
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) b[k] = bins[id[k]]; // the one random read per instance
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        const size_t i = base + (size_t)k * SCAN_BLOCK + tid;
        uint32_t c = 0;
        if (i < n) {
            c = bin_cells(b[k]);
            tile_pairs += bin_count(b[k]);
            bins_sorted[i] = b[k];
            counts_sorted[i] = c;
        }
        s[lds_pad(k * SCAN_BLOCK + tid)] = c;
    }
    __syncthreads();
    const uint32_t tile_total = block_scan_lds<SCAN_ITEMS>(s, s_wave);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) tile_pairs = add_tiles(tile_pairs, __shfl_xor(tile_pairs, o, 64));
    if (lane == 0) s_wave[tid >> 6] = tile_pairs; // (the scan above ended with a barrier)
    __syncthreads();
    if (tid < 64) {
        uint32_t block_tiles = 0;
        for (int w = 0; w < SCAN_BLOCK / 64; ++w) block_tiles = add_tiles(block_tiles, s_wave[w]);
        if (tid == 0) ss_store(&status[t], (t == 0 ? SS_INC : SS_AGG) | ss_pack(tile_total, block_tiles));
        uint32_t excl = 0, excl_tiles = 0;
        if (t > 0) {
            int64_t j = (int64_t)t - 1; // the window's newest tile
            uint32_t spins = 0;
            for (;;) {
                const int64_t idx = j - lane;
                const uint64_t sv = idx >= 0 ? ss_load(&status[idx]) : SS_INC; // before tile 0: inclusive 0
                const uint64_t flag = sv & ~SS_VAL;
                const uint64_t notready = __ballot(flag == 0ull), inc = __ballot(flag == SS_INC);
                const int fi = inc ? __builtin_ctzll(inc) : 64; // nearest inclusive prefix in the window
                const uint64_t need = (fi >= 63) ? ~0ull : ((2ull << fi) - 1ull);
                if (notready & need) {
                    if (++spins > SS_SPIN_LIMIT) {
                        if (lane == 0) atomicOr(&counters[CNT_SORT_ERR], 2u);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                    continue;
                }
                uint32_t v = (lane <= fi) ? (uint32_t)((sv & SS_VAL) >> 32) : 0u;
                uint32_t vt = (lane <= fi) ? (uint32_t)sv : 0u;
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) {
                    v = add_cells(v, __shfl_xor(v, o, 64));
                    vt = add_tiles(vt, __shfl_xor(vt, o, 64));
                }
                excl = add_cells(excl, v);
                excl_tiles = add_tiles(excl_tiles, vt);
                if (fi < 64) break;
                j -= 64;
            }
            if (tid == 0) ss_store(&status[t], SS_INC | ss_pack(add_cells(excl, tile_total), add_tiles(excl_tiles, block_tiles)));
        }
        if (tid == 0) {
            s_excl = excl;
            if (base + SCAN_TILE >= n) {
                store_pair_counts(counters, add_cells(excl, tile_total), add_tiles(excl_tiles, block_tiles), host_word, tag, capacity);
            }
        }
    }
    __syncthreads();
    const uint32_t ex = s_excl;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        const size_t i = base + (size_t)k * SCAN_BLOCK + tid;
        if (i < n) offsets[i] = min(s[lds_pad(k * SCAN_BLOCK + tid)] + ex, MAX_CELL_PAIRS); // (the sum below 2^32)
    }
}

// 32-bit words of the scan's look-back status (u64 per tile) for up to n
// instances: the most tiles that any count up to n is split into.
size_t scan_status_words(uint32_t n)
{
    const size_t few = scan_tiles(std::min(n, 160u * 1024), 4), more = scan_tiles(std::min(n, 640u * 1024), 8);
    return 2 * (std::max({few, more, scan_tiles(n, 16)}) + 1);
}

// bins_sorted[r] = bins[sorted_ids[r]], counts_sorted[r] its pair count,
// offsets = their exclusive scan, counters[CNT_PAIRS] = the total,
// counters[CNT_TILE_PAIRS] = the (tile, convex) pairs.  counters
// must hold CNT_WORDS words, zeroed, followed by scan_status_words(n) zeroed words.
void launch_gather_scan(hipStream_t st, uint32_t n, const uint32_t *sorted_ids, const uint4 *bins,
                        uint4 *bins_sorted, uint32_t *counts_sorted, uint32_t *offsets, uint32_t *counters,
                        unsigned long long *host_word, uint32_t tag, uint32_t capacity, uint32_t *ranges,
                        uint32_t range_words)
{
    if (n == 0) return;
    const int items = scan_items(n);
    const ZeroSpans z{{capacity ? ranges : nullptr}, {capacity ? range_words : 0u}};
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)scan_tiles(n, items)), dim3(SCAN_BLOCK), 0, st, n, sorted_ids, bins, bins_sorted,
                           counts_sorted, offsets, counters, reinterpret_cast<uint64_t *>(counters + CNT_STATUS),
                           host_word, tag, capacity, z);
    };
    if (items == 4) launch(gather_scan_kernel<4>);
    else if (items == 8) launch(gather_scan_kernel<8>);
    else launch(gather_scan_kernel<16>);
}

// ----------------------------------------------------------- radix sort ----
//
// Stable LSD radix sort of (u32 key, u32 value) pairs with one kernel per
// digit (single-pass scatter with decoupled look-back, after Merrill and
// Garland's single-pass prefix scan as used by the "Onesweep" radix sort):
//  1. one kernel reads the keys once and builds the global digit histograms of
//     every pass;
//  2. per pass, each workgroup claims the next tile of elements from an
//     atomic counter (tiles are claimed in order by running workgroups), ranks
//     its elements per digit (wave ballots), publishes its per-digit counts,
//     then walks back over its predecessors' published counts until it meets an
//     inclusive prefix, publishes its own inclusive prefix, and writes its
//     elements digit-sorted to their global positions.
// A predecessor publishes its counts before it waits on anything, so every
// wait ends; it is still bounded (OS_SPIN_LIMIT), and a wait that runs out
// sets the caller's error word instead of spinning on.

constexpr int OS_BLOCK = 512;
constexpr int OS_WAVES = OS_BLOCK / 64;
// Keys per thread: small tiles for few keys (more workgroups in flight), large
// ones for many (a shorter look-back chain).  us a pass of 8 bits with 4 / 8: 20k 7.7 /
// 9.4, 100k 9.3 / 10.1, 317k 13.2 / 12.8, 1M 22.5 / 17.9.
constexpr uint32_t OS_FEW = 128u * 1024, OS_MANY = 1u << 22;
inline int os_items(size_t n) { return n <= OS_FEW ? 4 : n <= OS_MANY ? 8 : 16; }
inline size_t os_tiles(size_t n, int items) { return (n + OS_BLOCK * items - 1) / (OS_BLOCK * items); }
constexpr int OS_RADIX = 256; // digits of up to 8 bits (one pass of 9 bits: os_radix)
constexpr int OS_MAX_PASSES = 8;
constexpr uint32_t OS_AGG = 1u << 30, OS_INC = 2u << 30, OS_VAL = OS_AGG - 1u;
constexpr uint32_t OS_SPIN_LIMIT = 1u << 22;
constexpr int OS_WINDOW = 8; // predecessors read per look-back round trip
// temporary layout (words): histograms [P][256] | tile counters [64] | status [P][tiles][256]
constexpr size_t OS_CTR = (size_t)OS_MAX_PASSES * OS_RADIX, OS_STATUS = OS_CTR + 64;

__host__ __device__ constexpr int os_passes(int end_bit, int digit_bits) { return (end_bit + digit_bits - 1) / digit_bits; }
// The end_bit bits are split over the passes as evenly as possible (13 bits in
// two passes: 7 + 6); pass p covers bits [os_shift, os_shift + os_width).
__host__ __device__ constexpr int os_width(int end_bit, int passes, int p)
{
    return end_bit / passes + (p < end_bit % passes ? 1 : 0);
}
__host__ __device__ constexpr int os_shift(int end_bit, int passes, int p)
{
    return p * (end_bit / passes) + (p < end_bit % passes ? p : end_bit % passes);
}

// Status words per tile of a pass.  Only a sort of one pass has digits of 9 bits
// (its histogram takes the room of two).
__host__ __device__ constexpr int os_radix(int width) { return width > 8 ? 1 << width : OS_RADIX; }

__device__ __forceinline__ uint32_t os_load(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void os_store(uint32_t *p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Lanes of the wave holding the same BITS-bit digit (ballot per bit).
template <int BITS> __device__ __forceinline__ uint64_t digit_peers(uint32_t dg, bool valid)
{
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const uint64_t bal = __ballot((dg >> b) & 1u);
        peers &= ((dg >> b) & 1u) ? bal : ~bal;
    }
    return peers;
}

// Exclusive scan of one value per thread over the workgroup (OS_BLOCK threads).
__device__ __forceinline__ uint32_t os_block_excl(uint32_t x, uint32_t *s_wsum)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) s_wsum[wave] = incl;
    __syncthreads();
    uint32_t wb = 0;
    for (int w = 0; w < wave; ++w) wb += s_wsum[w];
    __syncthreads();
    return wb + incl - x;
}

// Global histograms of every pass: hist[p * 256 + digit].  A workgroup takes
// tiles of OS_BLOCK x ITEMS keys (grid-stride), loads a tile's keys at
// once and counts them into per-wave LDS histograms (fewer same-address
// collisions), then adds its nonzero bins to the global histogram.
template <int BITS, int ITEMS>
__global__ __launch_bounds__(OS_BLOCK) void os_hist_kernel(const uint32_t *__restrict__ keys,
                                                           const uint32_t *__restrict__ n_dev, uint32_t n_host,
                                                           int end_bit, int P, uint32_t *__restrict__ hist)
{
    constexpr int TILE = OS_BLOCK * ITEMS;
    constexpr int R = 1 << BITS; // bins per pass (BITS: the widest pass)
    constexpr int HW = 1024;     // bins per wave: P * R <= 1024 for keys of up to 32 bits
    __shared__ uint32_t h[OS_WAVES][HW];
    const uint32_t n = n_dev ? *n_dev : n_host;
    const int wave = threadIdx.x >> 6;
    for (int d = threadIdx.x; d < OS_WAVES * HW; d += OS_BLOCK) (&h[0][0])[d] = 0;
    __syncthreads();
    const uint32_t ntiles = (n + TILE - 1) / TILE;
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        // each thread counts a contiguous run of ITEMS keys (16-byte loads), so
        // the lanes of a wave hold keys ITEMS apart: runs of equal digits (pairs
        // of one convex in neighbouring tiles) fall to one thread instead of
        // colliding on one LDS counter across the wave
        const size_t base = (size_t)t * TILE + (size_t)threadIdx.x * ITEMS;
        uint32_t k[ITEMS];
        int cnt;
        if (base + ITEMS <= n) {
            const uint4 *src = reinterpret_cast<const uint4 *>(keys + base);
#pragma unroll
            for (int q = 0; q < ITEMS / 4; ++q) {
                const uint4 w = src[q];
                k[4 * q] = w.x; k[4 * q + 1] = w.y; k[4 * q + 2] = w.z; k[4 * q + 3] = w.w;
            }
            cnt = ITEMS;
        } else {
            cnt = base < n ? (int)(n - base) : 0;
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) k[i] = i < cnt ? keys[base + i] : 0u;
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (i < cnt)
                for (int p = 0; p < P; ++p)
                    atomicAdd(&h[wave][p * R + ((k[i] >> os_shift(end_bit, P, p)) & ((1u << os_width(end_bit, P, p)) - 1u))],
                              1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < P * R; d += OS_BLOCK) {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < OS_WAVES; ++w) c += h[w][d];
        if (c) atomicAdd(&hist[(d / R) * OS_RADIX + d % R], c);
    }
}

template <int BITS, int ITEMS>
__global__ __launch_bounds__(OS_BLOCK) void os_scatter_kernel(
    const uint32_t *__restrict__ keys_in, const uint32_t *__restrict__ vals_in, uint32_t *__restrict__ keys_out,
    uint32_t *__restrict__ vals_out, const uint32_t *__restrict__ n_dev, uint32_t n_host, int shift,
    const uint32_t *__restrict__ hist, uint32_t *__restrict__ tile_counter, uint32_t *__restrict__ status,
    uint32_t *__restrict__ err, uint2 *__restrict__ ranges, uint32_t nranges)
{
    static_assert((1 << BITS) <= OS_BLOCK, "one digit per thread");
    constexpr int TILE = OS_BLOCK * ITEMS;
    constexpr int R = 1 << BITS;
    __shared__ uint32_t s_keys[TILE];
    __shared__ uint32_t s_vals[TILE];
    __shared__ uint32_t s_wcnt[OS_WAVES][R];
    __shared__ uint32_t s_dstart[R];
    __shared__ uint32_t s_gofs[R];
    __shared__ uint32_t s_wsum[OS_WAVES];
    __shared__ uint32_t s_tile;

    const uint32_t n = n_dev ? *n_dev : n_host;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // a grid sized for a capacity: as many workgroups as there are tiles claim
    // one each, the others leave without a claim (the claims are same-address
    // atomics, about 18 ns each)
    if ((size_t)blockIdx.x * TILE >= n) return;
    if (tid == 0) s_tile = atomicAdd(tile_counter, 1u);
    for (int d = tid; d < OS_WAVES * R; d += OS_BLOCK) (&s_wcnt[0][0])[d] = 0;
    __syncthreads();
    const uint32_t t = s_tile;
    const size_t tbase = (size_t)t * TILE;

    // rank: element order within the tile is (wave, item, lane)
    uint32_t k[ITEMS], v[ITEMS], off[ITEMS];
    const size_t wbase = tbase + (size_t)wave * 64 * ITEMS;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const size_t idx = wbase + i * 64 + lane;
        k[i] = keys_in[min(idx, (size_t)n - 1)]; // (clamped: no branch between the loads)
        v[i] = vals_in[min(idx, (size_t)n - 1)];
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const size_t idx = wbase + i * 64 + lane;
        const bool valid = idx < n;
        const uint32_t dg = (k[i] >> shift) & (R - 1);
        const uint64_t peers = digit_peers<BITS>(dg, valid);
        const uint32_t rank = __popcll(peers & lt_mask);
        const uint32_t before = valid ? s_wcnt[wave][dg] : 0u;
        off[i] = before + rank;
        if (valid && rank == 0) s_wcnt[wave][dg] = before + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    // per digit: exclusive over waves and the tile's count, published at once
    uint32_t total = 0;
    if (tid < R) {
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < OS_WAVES; ++w) {
            const uint32_t c = s_wcnt[w][tid];
            s_wcnt[w][tid] = run;
            run += c;
        }
        total = run;
        os_store(&status[(size_t)t * R + tid], (t == 0 ? OS_INC : OS_AGG) | total);
    }
    const uint32_t dstart = os_block_excl(tid < R ? total : 0u, s_wsum);
    // (a sort of one tile has its histogram here)
    const uint32_t all = tid < R ? (hist ? hist[tid] : total) : 0u;
    const uint32_t dbase = hist ? os_block_excl(all, s_wsum) : dstart;
    // a sort of one pass: the digits are the keys, their runs the histogram's scan
    if (ranges && t == 0 && tid < R && tid < (int)nranges) ranges[tid] = make_uint2(dbase, dbase + all);
    if (tid < R) {
        s_dstart[tid] = dstart;
        uint32_t excl = 0;
        if (t > 0) {
            // look back to the nearest inclusive prefix, OS_WINDOW predecessors
            // per round trip (entries before tile 0 read as inclusive zero)
            int64_t j = (int64_t)t - 1; // newest predecessor not yet consumed
            uint32_t spins = 0;
            for (;;) {
                uint32_t sv[OS_WINDOW];
#pragma unroll
                for (int w = 0; w < OS_WINDOW; ++w)
                    sv[w] = (j - w >= 0) ? os_load(&status[(size_t)(j - w) * R + tid]) : OS_INC;
                int used = 0;
                bool found = false, pending = false;
#pragma unroll
                for (int w = 0; w < OS_WINDOW; ++w) {
                    if (found || pending) continue;
                    const uint32_t f = sv[w] & ~OS_VAL;
                    if (f == 0u) { pending = true; continue; } // not published yet: re-read from here
                    excl += sv[w] & OS_VAL;
                    ++used;
                    found = (f == OS_INC);
                }
                if (found) break;
                j -= used;
                if (pending) {
                    if (++spins > OS_SPIN_LIMIT) { atomicOr(err, 1u); break; }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            os_store(&status[(size_t)t * R + tid], OS_INC | (excl + total));
        }
        s_gofs[tid] = dbase + excl;
    }
    __syncthreads();
    // digit-sorted tile in LDS, then each digit's run to its global position
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const size_t idx = wbase + i * 64 + lane;
        if (idx < n) {
            const uint32_t dg = (k[i] >> shift) & (R - 1);
            const uint32_t lp = s_dstart[dg] + s_wcnt[wave][dg] + off[i];
            s_keys[lp] = k[i];
            s_vals[lp] = v[i];
        }
    }
    __syncthreads();
    const uint32_t nvalid = (uint32_t)min((size_t)TILE, (size_t)n - tbase);
    for (uint32_t j = tid; j < nvalid; j += OS_BLOCK) {
        const uint32_t kk = s_keys[j];
        const uint32_t dg = (kk >> shift) & (R - 1);
        const uint32_t pos = s_gofs[dg] + (j - s_dstart[dg]);
        keys_out[pos] = kk;
        vals_out[pos] = s_vals[j];
    }
}

__global__ void fill_u32_kernel(uint32_t *__restrict__ p, size_t n, uint32_t v);

size_t sort_temp_words(uint32_t n_capacity, int end_bit, int digit_bits)
{
    digit_bits = std::min(8, std::max(4, digit_bits));
    // (the most tiles that any count up to the capacity is split into)
    const size_t tiles = std::max(os_tiles(std::min(n_capacity, OS_FEW), 4), os_tiles(n_capacity, 8));
    return OS_STATUS + (size_t)os_passes(end_bit, digit_bits) * std::max<size_t>(tiles, 1) * OS_RADIX;
}

template <int B, int I>
static void os_launch_hist(hipStream_t st, const uint32_t *keys, uint32_t n_host, const uint32_t *n_dev, int blocks,
                           int end_bit, int P, uint32_t *hist)
{
    hipLaunchKernelGGL((os_hist_kernel<B, I>), dim3(blocks), dim3(OS_BLOCK), 0, st, keys, n_dev, n_host, end_bit, P, hist);
}

template <int B, int I>
static void os_launch_scatter(hipStream_t st, const uint32_t *keys, const uint32_t *vals, uint32_t *keys_out,
                              uint32_t *vals_out, uint32_t n_host, const uint32_t *n_dev, int tiles, int shift,
                              const uint32_t *hist, uint32_t *ctr, uint32_t *status, uint32_t *err, uint2 *ranges,
                              uint32_t nranges)
{
    hipLaunchKernelGGL((os_scatter_kernel<B, I>), dim3(tiles), dim3(OS_BLOCK), 0, st, keys, vals, keys_out, vals_out, n_dev,
                       n_host, shift, hist, ctr, status, err, ranges, nranges);
}

#define OS_DISPATCH(BITS, CALL)                                                                                    \
    switch (BITS) {                                                                                                \
    case 1: { constexpr int BB = 1; CALL; } break;                                                                 \
    case 2: { constexpr int BB = 2; CALL; } break;                                                                 \
    case 3: { constexpr int BB = 3; CALL; } break;                                                                 \
    case 4: { constexpr int BB = 4; CALL; } break;                                                                 \
    case 5: { constexpr int BB = 5; CALL; } break;                                                                 \
    case 6: { constexpr int BB = 6; CALL; } break;                                                                 \
    case 7: { constexpr int BB = 7; CALL; } break;                                                                 \
    case 9: { constexpr int BB = 9; CALL; } break;                                                                 \
    default: { constexpr int BB = 8; CALL; } break;                                                                \
    }

#define OS_ITEMS_DISPATCH(ITEMS, CALL)                                                                             \
    do {                                                                                                           \
        if (ITEMS == 4) CALL(std::integral_constant<int, 4>{});                                                    \
        else if (ITEMS == 8) CALL(std::integral_constant<int, 8>{});                                               \
        else CALL(std::integral_constant<int, 16>{});                                                              \
    } while (0)

// Sorts bits [0, end_bit) of the keys in ceil(end_bit / digit_bits) passes
// (digit_bits in 4..8; the bits are split evenly over the passes).  On
// return *keys/*vals point at the sorted arrays (one of the two buffer pairs).
// n_dev may be NULL (n_host used); with n_dev the element count is read on the
// device (graph capture needs no host read-back) and n_capacity bounds it.
// temp: sort_temp_words(n_capacity, end_bit, digit_bits) words.  *err (device)
// gets bit 0 set if a look-back wait ran out of its bound.  The key arrays must
// be 16-byte aligned (the histogram pass reads them in 16-byte loads).
// Nine bits go in one pass of 512 digits where the caller allows 8-bit digits
// (the widest that it can ask for): the 510 cells of 1920x1080 then take one
// pass over their pairs instead of two.
static int sort_digits(int end_bit, int digit_bits)
{
    digit_bits = std::min(8, std::max(4, digit_bits));
    return digit_bits == 8 && end_bit == 9 ? 9 : digit_bits;
}

// Words of temp that radix_sort uses (and clears first, unless told that they
// are clear) for these arguments.
size_t radix_sort_words(uint32_t n_host, bool n_on_device, uint32_t n_capacity, int end_bit, int digit_bits)
{
    digit_bits = sort_digits(end_bit, digit_bits);
    const uint32_t n_grid = n_on_device ? n_capacity : n_host;
    if (n_grid == 0 || end_bit <= 0) return 0;
    const int P = os_passes(end_bit, digit_bits);
    const size_t tiles = os_tiles(n_grid, os_items(n_grid));
    return OS_STATUS + (size_t)P * tiles * os_radix(os_width(end_bit, P, 0));
}

// ranges (nullable, nranges entries): a sort of one pass also stores the
// [start, end) of every key below nranges there, and returns true.
bool radix_sort(hipStream_t st, uint32_t **keys, uint32_t **vals, uint32_t **keys_alt, uint32_t **vals_alt,
                uint32_t n_host, const uint32_t *n_dev, uint32_t n_capacity, int end_bit, uint32_t *temp,
                int digit_bits, uint32_t *err, bool temp_clear, uint2 *ranges, uint32_t nranges)
{
    digit_bits = sort_digits(end_bit, digit_bits);
    const uint32_t n_grid = n_dev ? n_capacity : n_host;
    if (n_grid == 0 || end_bit <= 0) return false;
    const int P = os_passes(end_bit, digit_bits);
    const int items = os_items(n_grid), tiles = (int)os_tiles(n_grid, items);
    const size_t words = radix_sort_words(n_host, n_dev != nullptr, n_capacity, end_bit, digit_bits);
    if (!temp_clear) {
        const size_t fb = std::min<size_t>((words + 255) / 256, 4096);
        hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)fb), dim3(256), 0, st, temp, words, 0u);
    }
    const int hb = std::max(1, std::min(tiles, 256)); // one workgroup per CU: fewer same-address global adds
    const int widest = os_width(end_bit, P, 0);
    const bool one_tile = tiles == 1; // (of n_grid, so for any count on the device)
    auto hist = [&](auto I) {
        OS_DISPATCH(widest, (os_launch_hist<BB, I.value>(st, *keys, n_host, n_dev, hb, end_bit, P, temp)));
    };
    if (!one_tile) OS_ITEMS_DISPATCH(items, hist);
    for (int p = 0; p < P; ++p) {
        const int shift = os_shift(end_bit, P, p);
        const int b = os_width(end_bit, P, p);
        uint32_t *status = temp + OS_STATUS + (size_t)p * tiles * os_radix(widest);
        uint2 *rg = P == 1 ? ranges : nullptr;
        auto scatter = [&](auto I) {
            OS_DISPATCH(b, (os_launch_scatter<BB, I.value>(st, *keys, *vals, *keys_alt, *vals_alt, n_host, n_dev, tiles, shift,
                                                           one_tile ? nullptr : temp + (size_t)p * OS_RADIX,
                                                           temp + OS_CTR + p, status, err, rg, nranges)));
        };
        OS_ITEMS_DISPATCH(items, scatter);
        std::swap(*keys, *keys_alt);
        std::swap(*vals, *vals_alt);
    }
    return P == 1 && ranges != nullptr;
}

// --------------------------------------------- small scenes in one kernel ----

// The depth sort, the gather of the binning records and the pair-offset scan of
// up to SMALL_ORDER_MAX instances by one workgroup: the radix sort's four passes
// in LDS (ranks by wavefront ballots, as above), then one scan.  Latency-bound,
// in place of six launches that take 4 to 8 us each however few their keys: a
// render of 1000 convexes at 128 x 128 97 -> 66 us; 8000 instances 41 us against
// the launches' 57.  A thread holds ITEMS instances; element order is (wavefront,
// item, lane).
constexpr int SM_BLOCK = 1024, SM_WAVES = SM_BLOCK / 64;
template <int ITEMS>
__global__ __launch_bounds__(SM_BLOCK) void small_order_kernel(
    uint32_t n, const uint32_t *__restrict__ keys, const uint4 *__restrict__ bins, uint32_t *__restrict__ sorted_ids,
    uint4 *__restrict__ bins_sorted, uint32_t *__restrict__ counts_sorted, uint32_t *__restrict__ offsets,
    uint32_t *__restrict__ counters, unsigned long long *__restrict__ host_word, uint32_t tag, uint32_t capacity, ZeroSpans zero)
{
    zero_share(zero); // the cell ranges, when this also prepares the pair pass
    constexpr int R = 256;
    __shared__ uint32_t s_key[SM_BLOCK * ITEMS], s_val[SM_BLOCK * ITEMS];
    __shared__ uint32_t s_cnt[SM_WAVES][R], s_start[R], s_wsum[2][SM_WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const uint32_t first = (uint32_t)(wave * 64 * ITEMS + lane);
    uint32_t k[ITEMS], v[ITEMS], off[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) { // places past n: the largest key, behind every instance
        v[i] = first + 64u * i;
        k[i] = v[i] < n ? keys[v[i]] : 0xFFFFFFFFu;
    }
    for (int shift = 0; shift < 32; shift += 8) {
        for (int d = tid; d < SM_WAVES * R; d += SM_BLOCK) (&s_cnt[0][0])[d] = 0u;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t dg = (k[i] >> shift) & (R - 1);
            const uint64_t peers = digit_peers<8>(dg, true);
            const uint32_t rank = __popcll(peers & lt_mask), before = s_cnt[wave][dg];
            off[i] = before + rank;
            if (rank == 0) s_cnt[wave][dg] = before + (uint32_t)__popcll(peers);
        }
        __syncthreads();
        // per digit: exclusive over the wavefronts, then over the digits
        uint32_t total = 0;
        if (tid < R) {
#pragma unroll
            for (int w = 0; w < SM_WAVES; ++w) {
                const uint32_t c = s_cnt[w][tid];
                s_cnt[w][tid] = total;
                total += c;
            }
        }
        uint32_t incl = total;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        if (lane == 63) s_wsum[0][wave] = incl;
        __syncthreads();
        if (tid < R) {
            for (int w = 0; w < wave; ++w) incl += s_wsum[0][w];
            s_start[tid] = incl - total;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t dg = (k[i] >> shift) & (R - 1), at = s_start[dg] + s_cnt[wave][dg] + off[i];
            s_key[at] = k[i];
            s_val[at] = v[i];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            k[i] = s_key[first + 64u * i];
            v[i] = s_val[first + 64u * i];
        }
    }
    uint32_t c[ITEMS], run = 0, tile_pairs = 0;
    uint4 b[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) b[i] = bins[min(v[i], n - 1u)];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t r = first + 64u * i;
        const uint32_t cells = r < n ? bin_cells(b[i]) : 0u;
        tile_pairs += r < n ? bin_count(b[i]) : 0u;
        uint32_t incl = cells;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        c[i] = run + incl - cells; // before this one in the wavefront
        run += __shfl(incl, 63, 64);
        if (r < n) {
            sorted_ids[r] = v[i];
            bins_sorted[r] = b[i];
            counts_sorted[r] = cells;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) tile_pairs = add_tiles(tile_pairs, __shfl_xor(tile_pairs, o, 64));
    if (lane == 0) {
        s_wsum[0][wave] = run;
        s_wsum[1][wave] = tile_pairs;
    }
    __syncthreads();
    uint32_t before = 0, m = 0, tiles = 0; // (a wavefront's 512 instances at most: some 2^29 pairs)
    for (int w = 0; w < SM_WAVES; ++w) {
        if (w < wave) before = add_cells(before, s_wsum[0][w]);
        m = add_cells(m, s_wsum[0][w]);
        tiles = add_tiles(tiles, s_wsum[1][w]);
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (first + 64u * i < n) offsets[first + 64u * i] = min(before + c[i], MAX_CELL_PAIRS);
    if (tid == 0) store_pair_counts(counters, m, tiles, host_word, tag, capacity);
}

// Whether the order of n instances is made by small_order_kernel; then it is
// (arguments as launch_gather_scan's, keys in instance order).  The line is where
// the keys still fit LDS: one workgroup is faster up to there (above).
constexpr uint32_t SMALL_ORDER_MAX = 8 * SM_BLOCK;
bool launch_small_order(hipStream_t st, uint32_t n, const uint32_t *keys, const uint4 *bins, uint32_t *sorted_ids,
                        uint4 *bins_sorted, uint32_t *counts_sorted, uint32_t *offsets, uint32_t *counters,
                        unsigned long long *host_word, uint32_t tag, uint32_t capacity, uint32_t *ranges, uint32_t range_words)
{
    if (n == 0 || n > SMALL_ORDER_MAX) return false;
    const ZeroSpans z{{capacity ? ranges : nullptr}, {capacity ? range_words : 0u}};
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(1), dim3(SM_BLOCK), 0, st, n, keys, bins, sorted_ids, bins_sorted, counts_sorted, offsets,
                           counters, host_word, tag, capacity, z);
    };
    if (n <= SM_BLOCK) launch(small_order_kernel<1>);
    else if (n <= 2 * SM_BLOCK) launch(small_order_kernel<2>);
    else if (n <= 4 * SM_BLOCK) launch(small_order_kernel<4>);
    else launch(small_order_kernel<8>);
    return true;
}

// ------------------------------------------------------------- binning ----

// (cell, convex) pairs of 256 consecutive instances in depth order, written
// cooperatively: their pair ranges are contiguous ([offsets[r], offsets[r] +
// counts[r]) in rank order), so the workgroup strides over the whole run with
// one pair per thread (coalesced stores).  Within an instance the pairs run
// row-major over its cells, band by band in a large rectangle (see rect_cells); a
// pair's key is the cell with the mask of its kept tiles above (see FrameHeader).
// Instance id = view * n_convex + convex.
constexpr int EMIT_BLOCK = 256;
constexpr int EMIT_ITEMS = 8;
constexpr int EMIT_CHUNK = EMIT_BLOCK * EMIT_ITEMS; // pairs whose owners are found per round

// Position of the q-th set bit of m (q < popcount(m)).
__device__ __forceinline__ uint32_t nth_set_bit(uint64_t m, uint32_t q)
{
    uint32_t pos = 0;
    uint32_t w = (uint32_t)m;
    const uint32_t c32 = __popc(w);
    if (q >= c32) { q -= c32; w = (uint32_t)(m >> 32); pos = 32; }
#pragma unroll
    for (int half = 16; half >= 1; half >>= 1) {
        const uint32_t c = __popc(w & ((1u << half) - 1u));
        if (q >= c) { q -= c; w >>= half; pos += half; }
    }
    return pos;
}
// q / d for q < 2^24, through the reciprocal, corrected by one step.
__device__ __forceinline__ uint32_t small_div(uint32_t q, uint32_t d)
{
    uint32_t r = (uint32_t)((float)q * __builtin_amdgcn_rcpf((float)d));
    if (r * d > q) --r;
    else if ((r + 1u) * d <= q) ++r;
    return r;
}
// The kept tiles of the cell whose first tile is (ctx, cty), one bit per tile
// row-major over the cell, of a rectangle of at most 64 tiles.
__device__ __forceinline__ uint32_t cell_mask(uint64_t mask, int tx0, int ty0, int w, int th, int ctx, int cty,
                                              int shift)
{
    const int side = 1 << shift;
    const uint32_t sidemask = (1u << side) - 1u;
    const int c0 = ctx - tx0; // the cell's first column, rectangle-relative (may be negative)
    const uint64_t rowmask = w < 64 ? (1ull << w) - 1ull : ~0ull;
    uint32_t m = 0;
    for (int sy = 0; sy < side; ++sy) {
        const int r = cty + sy - ty0;
        if (r < 0 || r >= th) continue;
        const uint64_t row = (mask >> (r * w)) & rowmask;
        const uint32_t nib = (uint32_t)(c0 >= 0 ? row >> c0 : row << -c0) & sidemask;
        m |= nib << (sy * side);
    }
    return m;
}
// The tiles of the cell whose first tile is (ctx, cty) in band r of a larger one.
__device__ __forceinline__ uint32_t band_mask(uint64_t mask, int tx0, int ty0, int w, int th, int r, int ctx, int cty, int shift)
{
    int row0, nrow, col0, ncol;
    big_band(mask, w, th, r, &row0, &nrow, &col0, &ncol);
    const int last = (1 << shift) - 1;
    const int x0 = max(tx0 + col0 - ctx, 0), x1 = min(tx0 + col0 + ncol - 1 - ctx, last);
    const int y0 = max(ty0 + row0 - cty, 0), y1 = min(ty0 + row0 + nrow - 1 - cty, last);
    uint32_t m = 0;
    for (int y = y0; y <= y1; ++y) m |= (((2u << x1) - 1u) & ~((1u << x0) - 1u)) << (y << shift);
    return m;
}

__global__ __launch_bounds__(EMIT_BLOCK) void emit_pairs_kernel(
    uint32_t n, uint32_t n_convex, const uint32_t *__restrict__ sorted_ids, const uint32_t *__restrict__ offsets,
    const uint32_t *__restrict__ counts_sorted, const uint4 *__restrict__ bins_sorted,
    const FrameHeader *__restrict__ frame, uint32_t capacity, uint32_t *__restrict__ pair_keys,
    uint32_t *__restrict__ pair_ids, ZeroSpans zero)
{
    zero_share(zero); // the cell sort's temporaries
    __shared__ uint32_t s_off[EMIT_BLOCK];
    __shared__ uint32_t s_id[EMIT_BLOCK];
    __shared__ uint4 s_bin[EMIT_BLOCK];
    __shared__ uint32_t s_base[EMIT_BLOCK]; // the view's cell_off
    __shared__ uint32_t s_cx[EMIT_BLOCK];   // the view's cells per row
    // a rectangle of at most 64 tiles: its cell marks (low, high word) and whether every
    // cell that it meets makes a pair (then there are no marks); a larger one: the pairs up to the
    // end of its first bands
    __shared__ uint32_t s_in[3][EMIT_BLOCK];
    static_assert(BIG_BANDS == 4, "a word for every band but the last");
    __shared__ uint32_t s_own[EMIT_CHUNK];  // owner (block-local convex) of each pair of the chunk
    __shared__ uint32_t s_wmax[EMIT_BLOCK / 64];
    __shared__ uint32_t s_end;
    const uint32_t r0 = blockIdx.x * EMIT_BLOCK;
    const int cnt = (int)min((uint32_t)EMIT_BLOCK, n - r0);
    const int tid = threadIdx.x;
    const ViewDesc *views = reinterpret_cast<const ViewDesc *>(frame + 1);
    const uint32_t kbits = frame->key_bits;
    if (tid < cnt) {
        const uint32_t r = r0 + tid;
        const uint32_t id = sorted_ids[r];
        const uint32_t off = offsets[r], count = counts_sorted[r];
        s_off[tid] = off;
        s_id[tid] = id;
        if (count > 0) {
            const uint4 b = bins_sorted[r];
            const ViewDesc &vd = views[id / n_convex];
            s_bin[tid] = b;
            s_base[tid] = (uint32_t)vd.cell_off;
            const uint32_t shift = bin_shift(b);
            s_cx[tid] = ((uint32_t)vd.tiles_x + (1u << shift) - 1u) >> shift;
            const uint32_t tx0 = bin_tx0(b), ty0 = bin_ty0(b), tx1 = bin_tx1(b), ty1 = bin_ty1(b);
            const uint32_t tw = tx1 - tx0 + 1u, th = ty1 - ty0 + 1u;
            const uint64_t mask = (uint64_t)b.z | ((uint64_t)b.w << 32);
            if (tw * th <= 64u) {
                const bool all = count == cells_met((int)tx0, (int)tx1, shift) * cells_met((int)ty0, (int)ty1, shift);
                s_in[2][tid] = all ? 1u : 0u;
                if (!all) {
                    const uint64_t marks = cell_marks(mask, tx0, ty0, tw, th, shift);
                    s_in[0][tid] = (uint32_t)marks;
                    s_in[1][tid] = (uint32_t)(marks >> 32);
                }
            } else {
                uint32_t end = 0;
#pragma unroll
                for (int k = 0; k < BIG_BANDS - 1; ++k) {
                    const CellBlock c = band_cells(mask, (int)tx0, (int)ty0, (int)tw, (int)th, k, shift);
                    s_in[k][tid] = end += c.nx * c.ny;
                }
            }
        }
        if (tid == cnt - 1) s_end = off + count;
    }
    __syncthreads();
    const uint32_t p0 = s_off[0], p1 = min(s_end, capacity);
    const int lane = tid & 63, wave = tid >> 6;
    // The pairs' owners, EMIT_CHUNK pairs at a time: each convex marks the first
    // pair of its run (entries with no pairs share the next one's offset: the
    // larger index, the owner, wins), the chunk's first pair gets its owner by
    // one binary search, and a running maximum carries the marks along the runs.
    for (uint32_t c0 = p0; c0 < p1; c0 += EMIT_CHUNK) {
        const uint32_t cn = min((uint32_t)EMIT_CHUNK, p1 - c0);
        for (int j = tid; j < EMIT_CHUNK; j += EMIT_BLOCK) s_own[j] = 0u;
        __syncthreads();
        if (tid == 0) { // last entry with s_off <= c0
            int lo = 0, hi = cnt - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_off[mid] <= c0) lo = mid;
                else hi = mid - 1;
            }
            atomicMax(&s_own[0], (uint32_t)lo);
        }
        if (tid < cnt) {
            const uint32_t o = s_off[tid];
            if (o >= c0 && o < c0 + cn) atomicMax(&s_own[o - c0], (uint32_t)tid);
        }
        __syncthreads();
        // inclusive running maximum over the chunk: EMIT_ITEMS consecutive entries per thread
        uint32_t v[EMIT_ITEMS], m = 0u;
#pragma unroll
        for (int k = 0; k < EMIT_ITEMS; ++k) {
            m = max(m, s_own[tid * EMIT_ITEMS + k]);
            v[k] = m;
        }
        uint32_t incl = m;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl = max(incl, y);
        }
        if (lane == 63) s_wmax[wave] = incl;
        __syncthreads();
        uint32_t before = __shfl_up(incl, 1, 64);
        if (lane == 0) before = 0u;
        for (int w = 0; w < wave; ++w) before = max(before, s_wmax[w]);
#pragma unroll
        for (int k = 0; k < EMIT_ITEMS; ++k) s_own[tid * EMIT_ITEMS + k] = max(before, v[k]);
        __syncthreads();
        for (uint32_t j = tid; j < cn; j += EMIT_BLOCK) {
            const uint32_t p = c0 + j;
            const int lo = (int)s_own[j];
            const uint32_t q = p - s_off[lo];
            const uint4 b = s_bin[lo];
            const uint32_t tx0 = bin_tx0(b), ty0 = bin_ty0(b), tx1 = bin_tx1(b), ty1 = bin_ty1(b), shift = bin_shift(b);
            const uint32_t tw = tx1 - tx0 + 1u, th = ty1 - ty0 + 1u;
            const uint64_t kept = (uint64_t)b.z | ((uint64_t)b.w << 32);
            const uint32_t in0 = s_in[0][lo], in1 = s_in[1][lo], in2 = s_in[2][lo];
            uint32_t cx, cy, mask;
            if (tw * th <= 64u) {
                if (in2) { // the q-th cell, row-major
                    const uint32_t cw = cells_met((int)tx0, (int)tx1, shift), row = small_div(q, cw);
                    cx = (tx0 >> shift) + q - row * cw;
                    cy = (ty0 >> shift) + row;
                } else { // the q-th marked one
                    const uint32_t at = nth_set_bit((uint64_t)in0 | ((uint64_t)in1 << 32), q), row = small_div(at, tw);
                    cx = (tx0 + at - row * tw) >> shift;
                    cy = (ty0 + row) >> shift;
                }
                mask = cell_mask(kept, (int)tx0, (int)ty0, (int)tw, (int)th, (int)(cx << shift), (int)(cy << shift), (int)shift);
            } else { // the q-th cell of the bands, band by band
                const int r = (q >= in0) + (q >= in1) + (q >= in2);
                const uint32_t before = r == 0 ? 0u : r == 1 ? in0 : r == 2 ? in1 : in2;
                const CellBlock c = band_cells(kept, (int)tx0, (int)ty0, (int)tw, (int)th, r, shift);
                const uint32_t qb = q - before, nx = max(c.nx, 1u), row = small_div(qb, nx);
                cx = c.x + qb - row * nx;
                cy = c.y + row;
                mask = band_mask(kept, (int)tx0, (int)ty0, (int)tw, (int)th, r, (int)(cx << shift), (int)(cy << shift), (int)shift);
            }
            pair_keys[p] = (s_base[lo] + cy * s_cx[lo] + cx) | (mask << kbits);
            pair_ids[p] = s_id[lo];
        }
        __syncthreads();
    }
}

// Sort keys that put the tiles of long cell lists first: key = 0xFFFF -
// min(length, 0xFFFF); slots past the frame's tiles sort behind them.
__global__ void tile_length_keys_kernel(uint32_t ntiles, const FrameHeader *__restrict__ frame,
                                        const uint2 *__restrict__ ranges, uint32_t *__restrict__ keys,
                                        uint32_t *__restrict__ vals)
{
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntiles) return;
    uint32_t len = 0;
    if (t < frame->total_tiles) {
        const ViewDesc *views = reinterpret_cast<const ViewDesc *>(frame + 1);
        const ViewDesc &vd = views[find_view(views, (int)frame->nviews, (int)t)];
        const uint32_t lt = t - (uint32_t)vd.tile_off, tx = lt % (uint32_t)vd.tiles_x, ty = lt / (uint32_t)vd.tiles_x;
        const uint2 r = ranges[tile_cell(vd, tx, ty)];
        len = r.y - r.x;
    }
    keys[t] = 0xFFFFu - (len < 0xFFFFu ? len : 0xFFFFu);
    vals[t] = t;
}

// Zero up to four ranges of words in one launch.
struct FillRanges {
    uint32_t *p[4];
    size_t n[4];
};
__global__ void zero_ranges_kernel(FillRanges r)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < r.n[k]; i += stride) r.p[k][i] = 0u;
}

// The pair count that fits the buffers and the overflow flag, and the tile
// ranges cleared, in one launch.
__global__ void prepare_tail_kernel(uint32_t *__restrict__ counters, uint32_t capacity, uint32_t *__restrict__ ranges,
                                    size_t nwords)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const uint32_t m = counters[CNT_PAIRS];
        counters[CNT_PAIRS_EFF] = m < capacity ? m : capacity;
        counters[CNT_OVERFLOW] = m > capacity ? 1u : 0u;
    }
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nwords; i += (size_t)gridDim.x * blockDim.x)
        ranges[i] = 0u;
}

__global__ void fill_u32_kernel(uint32_t *__restrict__ p, size_t n, uint32_t v)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// [start, end) of every cell's run in the sorted keys (the cell is a key's low
// bits).  Each thread takes RANGE_ITEMS consecutive keys in 16-byte loads (the
// sorted keys are 16-byte aligned) plus the key before them, and marks the run
// boundaries among them.
constexpr int RANGE_ITEMS = 8;

// ncells bounds the cells written (every cell of a pair is below it; the
// bound keeps a wrong count from writing past the ranges).
__global__ __launch_bounds__(256) void cell_ranges_kernel(const uint32_t *__restrict__ keys,
                                                          const uint32_t *__restrict__ n_dev, uint32_t n_host,
                                                          uint2 *__restrict__ ranges, uint32_t ncells, uint32_t cmask)
{
    const uint32_t n = n_dev ? *n_dev : n_host;
    const size_t i0 = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * RANGE_ITEMS;
    if (i0 >= n) return;
    uint32_t t[RANGE_ITEMS];
    if (i0 + RANGE_ITEMS <= n) {
        const uint4 *src = reinterpret_cast<const uint4 *>(keys + i0);
#pragma unroll
        for (int q = 0; q < RANGE_ITEMS / 4; ++q) {
            const uint4 w = src[q];
            t[4 * q] = w.x; t[4 * q + 1] = w.y; t[4 * q + 2] = w.z; t[4 * q + 3] = w.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < RANGE_ITEMS; ++k) t[k] = i0 + k < n ? keys[i0 + k] : 0u;
    }
#pragma unroll
    for (int k = 0; k < RANGE_ITEMS; ++k) t[k] &= cmask;
    uint32_t prev = i0 > 0 ? (keys[i0 - 1] & cmask) : 0xFFFFFFFFu;
#pragma unroll
    for (int k = 0; k < RANGE_ITEMS; ++k) {
        const size_t i = i0 + k;
        if (i >= n) break;
        if (t[k] != prev) { // a run starts at i and the previous one ends there
            if (t[k] < ncells) ranges[t[k]].x = (uint32_t)i;
            if (i > 0 && prev < ncells) ranges[prev].y = (uint32_t)i;
        }
        prev = t[k];
    }
    if (i0 + RANGE_ITEMS >= n && prev < ncells) ranges[prev].y = n; // the last run
}

void launch_fill_u32(hipStream_t st, uint32_t *p, size_t n, uint32_t v)
{
    if (n == 0) return;
    const size_t blocks = std::min<size_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
}

void launch_emit_pairs(hipStream_t st, uint32_t n, uint32_t n_convex, const uint32_t *sorted_ids,
                       const uint32_t *offsets, const uint32_t *counts_sorted, const uint4 *bins_sorted,
                       const FrameHeader *views, uint32_t capacity, uint32_t *pair_tiles, uint32_t *pair_ids,
                       uint32_t *zero, uint32_t zero_words)
{
    if (n == 0) return;
    const ZeroSpans z{{zero}, {zero ? zero_words : 0u}};
    hipLaunchKernelGGL(emit_pairs_kernel, dim3((n + EMIT_BLOCK - 1) / EMIT_BLOCK), dim3(EMIT_BLOCK), 0, st, n,
                       n_convex, sorted_ids, offsets, counts_sorted, bins_sorted, views, capacity, pair_tiles,
                       pair_ids, z);
}

void launch_prepare_tail(hipStream_t st, uint32_t *counters, uint32_t capacity, uint32_t *ranges, size_t nwords)
{
    const size_t blocks = std::max<size_t>(1, std::min<size_t>((nwords + 255) / 256, 1024));
    hipLaunchKernelGGL(prepare_tail_kernel, dim3((unsigned)blocks), dim3(256), 0, st, counters, capacity, ranges,
                       nwords);
}

void launch_zero_ranges(hipStream_t st, uint32_t *p0, size_t n0, uint32_t *p1, size_t n1, uint32_t *p2, size_t n2)
{
    FillRanges r = {{p0, p1, p2, p0}, {n0, n1, n2, 0}};
    const size_t most = std::max(std::max(n0, n1), n2);
    if (most == 0) return;
    const size_t blocks = std::min<size_t>((most + 255) / 256, 4096);
    hipLaunchKernelGGL(zero_ranges_kernel, dim3((unsigned)blocks), dim3(256), 0, st, r);
}

void launch_tile_length_keys(hipStream_t st, uint32_t ntiles, const FrameHeader *frame, const uint2 *ranges,
                             uint32_t *keys, uint32_t *vals)
{
    if (ntiles == 0) return;
    hipLaunchKernelGGL(tile_length_keys_kernel, dim3((ntiles + 255) / 256), dim3(256), 0, st, ntiles, frame, ranges,
                       keys, vals);
}

void launch_cell_ranges(hipStream_t st, const uint32_t *keys, uint32_t n_host, const uint32_t *n_dev,
                        uint32_t n_capacity, uint2 *ranges, uint32_t ncells, uint32_t cmask)
{
    if (n_capacity == 0) return;
    const size_t threads = ((size_t)n_capacity + RANGE_ITEMS - 1) / RANGE_ITEMS;
    hipLaunchKernelGGL(cell_ranges_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, keys, n_dev,
                       n_host, ranges, ncells, cmask);
}

} // namespace cs
