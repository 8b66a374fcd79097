// Per-tile compositing, forward and backward (gfx950).
//
// One workgroup per tile (8x8, 16x16 or 32x32 pixels), one pixel per thread,
// in a persistent grid that pulls tiles of all views from per-XCD work queues.
// The tile's depth-ordered convex list (its cell's list, filtered by the tile's
// mask bit) is streamed through LDS in batches of records; every thread walks the batch front to back and evaluates, for its pixel,
//   x2_j = log2(e) delta' L_j(q)           (FP64: hull lines, Supp. B scaling)
//   phi  = LogSumExp of the x_j            (Sec. 3.1 Eq. smoothness, base 2)
//   I    = Sigmoid(-sigma' phi)            (Sec. 3.1 Eq. sharpness)
//   alpha = o I,  C += T alpha c,  T *= 1 - alpha   (Sec. 3.2 compositing eq.)
// skipping pairs with alpha < eps_alpha and stopping after the convex that
// brings T below t_min.  Only x2_j is FP64: at the configured sharpness the
// indicator moves by sigma' delta' / 4 per pixel of line offset, so the line
// must be exact to ~1e-9 px; everything after it runs in FP32 on the hardware
// exp2 / log2 / reciprocal.
//
// The backward kernel walks the same lists back to front from each pixel's
// last contributor, recomputing alpha with the same function (bit-identical
// decisions), recovering T_n = T_{n+1} / (1 - alpha_n); the per-pair gradients
// are reduced over the wavefront (lane swaps + DPP), summed over the
// workgroup's waves in LDS, and leave as one float atomic add per
// (convex, value) and workgroup.
#include <algorithm>
#include <cstddef>
#include <mutex>
#include <unordered_map>
#include <utility>

#include "common.hpp"

namespace cs {

namespace {

// A pixel's (u, y) lies in a record's box (box_u, box_v), outside of which alpha < eps.
__device__ __forceinline__ bool in_box(uint32_t box_u, uint32_t box_v, int u, int y)
{
    return u >= (int)(box_u & 0xFFFFu) && u <= (int)(box_u >> 16) && y >= (int)(box_v & 0xFFFFu) &&
           y <= (int)(box_v >> 16);
}

template <int K> struct PairEval {
    float I, omI, alpha, oma, phi2, inv_sum;
    float e[K];  // 2^(x2_j - max)
    float x2[K]; // x2_j rounded to float
};

// Runs the statements with the compile-time constant NLL equal to the wave-
// uniform hull size TV (3..K; records in tile lists always have T >= 3).
#define CS_NL_CASE(n, K, ...) \
    case n:                   \
        if constexpr (n <= K) { \
            constexpr int NLL = n; \
            __VA_ARGS__;      \
        }                     \
        break;
#define CS_DISPATCH_NL(K, TV, ...)                                                                               \
    switch (TV) {                                                                                                \
        CS_NL_CASE(3, K, __VA_ARGS__) CS_NL_CASE(4, K, __VA_ARGS__) CS_NL_CASE(5, K, __VA_ARGS__)                \
        CS_NL_CASE(6, K, __VA_ARGS__) CS_NL_CASE(7, K, __VA_ARGS__) CS_NL_CASE(8, K, __VA_ARGS__) default: break; \
    }

// The FP32 part of a pair evaluation from the line values x (m: their
// maximum, full: the pair passed the max-line test): softmax weights,
// LogSumExp, indicator and alpha.  Returns whether the pair contributes.
template <int K, int NL>
__device__ __forceinline__ bool finish_pair(const RecHeader &h, const double *x, double m, bool full, float eps,
                                            PairEval<K> &pe)
{
    const float mf = (float)m;
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const float xf = (float)x[j];
        const float e = __builtin_amdgcn_exp2f(xf - mf);
        pe.e[j] = e;
        pe.x2[j] = xf;
        s += e;
    }
    pe.inv_sum = __builtin_amdgcn_rcpf(s);
    const float phi2 = mf + __builtin_amdgcn_logf(s);
    const float z = h.sigma_p * phi2; // I = 1 / (1 + 2^z)
    const float ez = __builtin_amdgcn_exp2f(-fabsf(z));
    const float r = __builtin_amdgcn_rcpf(1.0f + ez);
    pe.I = z > 0.0f ? ez * r : r;
    pe.omI = z > 0.0f ? r : ez * r;
    pe.alpha = h.opacity * pe.I;
    pe.oma = (1.0f - h.opacity) + h.opacity * pe.omI;
    pe.phi2 = phi2;
    return full && !(pe.alpha < eps);
}

// The one evaluation of a (pixel, convex) pair shared by both passes, called
// by every lane of the wavefront (live: the pixel still takes convexes).
// Returns whether the pair contributes: the pixel lies in the record's pixel
// box (tested), the largest line value passes the skip threshold (full), and
// alpha >= eps_alpha.  When some lane passes the threshold, every field of pe
// is computed, and finite, for every lane, so that callers can use them
// without branches; otherwise the wavefront leaves early.
//
// The record (header and all K line slots) is read from LDS in one burst of
// 16-byte reads with a single wait (a branch per line would serialise the LDS
// round trips; slots past T hold null lines).  The lines are evaluated in FP64; the exponents are taken
// as differences of the FP32-rounded values (phi already starts from the
// rounded maximum, and where the sigmoid is sensitive |x2| is small).
// NL: the record's hull size T (its line count), a compile-time constant of
// the caller's dispatch on the wave-uniform T, so that only the hull's lines
// are read and evaluated.
template <int K, int NL>
__device__ __forceinline__ bool eval_pair(const uint8_t *rec, bool live, int u, int y, float pxf, float pyf,
                                          float eps, PairEval<K> &pe, bool &tested, bool &full)
{
    static_assert(NL >= 3 && NL <= K, "hull size out of range");
    // the pixel box first: its test then waits for it alone, with the line
    // reads still in flight
    const uint2 box = *reinterpret_cast<const uint2 *>(rec + offsetof(RecHeader, box_u));
    const RecHeader h = *reinterpret_cast<const RecHeader *>(rec);
    double L[3 * NL + 1]; // one spare slot: odd 3 NL reads one double past the last line (still in the record)
    const double2 *l2 = reinterpret_cast<const double2 *>(rec + REC_HEADER);
#pragma unroll
    for (int q = 0; q < (3 * NL + 1) / 2; ++q) {
        const double2 w = l2[q];
        L[2 * q] = w.x;
        L[2 * q + 1] = w.y;
    }
    tested = live & in_box(box.x, box.y, u, y); // no short circuit: no branch around the box test
    const double dx = (double)(pxf - h.ox), dy = (double)(pyf - h.oy);
    double x[NL];
    double m = -INFINITY;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        x[j] = fma(L[3 * j], dx, fma(L[3 * j + 1], dy, L[3 * j + 2]));
        m = fmax(m, x[j]);
    }
    // LogSumExp >= its largest term: past thr2 alpha < eps for certain
    full = tested && (m <= (double)h.thr2);
    if (!__any(full)) return false;
    return finish_pair<K, NL>(h, x, m, full, eps, pe);
}

// First half of a whole-wavefront sum of NP values (NP a multiple of 4), by
// transposition: a 32-lane swap (v_permlane32_swap) pairs value j with value
// j + NP/2 so that one add leaves the two half-wave sums of j in the lower
// half and of j + NP/2 in the upper half; a 16-lane swap (v_permlane16_swap)
// does the same between rows.  On return lane l of row r holds in v[j],
// j < NP/4, a partial sum of value j + r NP/4 (the row reduction finishes it).
template <int NP> __device__ __forceinline__ void wave_to_rows(float *v)
{
    static_assert(NP % 4 == 0, "pad the values to a multiple of 4");
    constexpr int H = NP / 2, Q = NP / 4;
#pragma unroll
    for (int j = 0; j < H; ++j) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[j]), __float_as_uint(v[j + H]), false, false);
        v[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[j]), __float_as_uint(v[j + Q]), false, false);
        v[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
}

// Row totals of Q values over the 16 lanes of each row, transposed like the
// swaps above: four DPP stages pair every lane with a partner (row mirror,
// half-row mirror, quad swap of 2, of 1), and at each stage the registers are
// taken in pairs: both values of a pair are added to the partner's, and the
// lanes on one side of the stage keep the first sum, the others the second
// (an unpaired last register is summed in place).  The register count halves
// per stage, so Q values cost about 1.5 (Q + Q/2 + Q/4 + Q/8) instructions
// where plain row sums take 4 Q; at the end lane i of a row holds the row
// total of value rr_value(Q, i).
__host__ __device__ constexpr bool rr_keeps_first(int stage, int i)
{
    return stage == 0 ? (i < 8) : stage == 1 ? ((i & 7) < 4) : stage == 2 ? ((i & 2) == 0) : ((i & 1) == 0);
}
__host__ __device__ constexpr int rr_value(int Q, int lane)
{
    int reg[16] = {};
    int m = Q;
    for (int k = 0; k < Q; ++k) reg[k] = k;
    for (int s = 0; s < 4; ++s) {
        const bool first = rr_keeps_first(s, lane);
        int nm = 0;
        for (int p = 0; p + 1 < m; p += 2) reg[nm++] = first ? reg[p] : reg[p + 1];
        if (m & 1) reg[nm++] = reg[m - 1];
        m = nm;
    }
    return reg[0];
}
// 4 bits per lane: the value whose total the lane holds
__host__ __device__ constexpr uint64_t rr_map(int Q)
{
    uint64_t t = 0;
    for (int i = 0; i < 16; ++i) t |= (uint64_t)rr_value(Q, i) << (4 * i);
    return t;
}
// the lanes that hold a value no lower lane of the row holds
__host__ __device__ constexpr uint32_t rr_first_lanes(int Q)
{
    uint32_t f = 0;
    for (int i = 0; i < 16; ++i) {
        bool first = true;
        for (int j = 0; j < i; ++j) first = first && rr_value(Q, j) != rr_value(Q, i);
        if (first) f |= 1u << i;
    }
    return f;
}
// every value's total reaches exactly one first lane
__host__ __device__ constexpr bool rr_covers(int Q)
{
    const uint32_t f = rr_first_lanes(Q);
    int holders[16] = {};
    for (int i = 0; i < 16; ++i)
        if ((f >> i) & 1u) ++holders[rr_value(Q, i)];
    bool ok = true;
    for (int q = 0; q < 16; ++q) ok = ok && holders[q] == (q < Q ? 1 : 0);
    return ok;
}
static_assert(rr_covers(4) && rr_covers(5) && rr_covers(6) && rr_covers(7) && rr_covers(8),
              "row reduction lane map");
template <int S, int M> __device__ __forceinline__ void rr_stage(float *v, int li)
{
    constexpr int CTRL = S == 0 ? 0x140 : S == 1 ? 0x141 : S == 2 ? 0x4E : 0xB1; // DPP partner of the stage
    const bool first = rr_keeps_first(S, li);
#pragma unroll
    for (int p = 0; p + 1 < M; p += 2) {
        // the sums first, then the choice: a choice between the two array
        // elements would become a per-lane index into the array
        const float a = v[p], b = v[p + 1];
        const float sa = a + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a), CTRL, 0xF, 0xF, true));
        const float sb = b + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(b), CTRL, 0xF, 0xF, true));
        v[p / 2] = first ? sa : sb;
    }
    if constexpr ((M & 1) != 0) {
        const float a = v[M - 1];
        v[M / 2] = a + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a), CTRL, 0xF, 0xF, true));
    }
}
template <int Q> __device__ __forceinline__ float row_reduce(float *v)
{
    static_assert(Q >= 1 && Q <= 16, "at most 16 values per row");
    const int li = threadIdx.x & 15;
    constexpr int M1 = (Q + 1) / 2, M2 = (M1 + 1) / 2, M3 = (M2 + 1) / 2;
    rr_stage<0, Q>(v, li);
    rr_stage<1, M1>(v, li);
    rr_stage<2, M2>(v, li);
    rr_stage<3, M3>(v, li);
    return v[0];
}

// Pixel of a thread within its tile: each wavefront covers an 8x8 square
// (a compact patch: more of its lanes fall inside the same convex than in a
// 16x4 strip), wavefronts tile the TILE x TILE tile row-major.
template <int TILE> __device__ __forceinline__ void tile_pixel(int &dx, int &dy)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    dx = (w % (TILE / 8)) * 8 + (l & 7);
    dy = (w / (TILE / 8)) * 8 + (l >> 3);
}


// The bounding rectangle, in the square, of the pixels whose lanes are in the
// (nonempty) mask: x0 | x1 << 4 | y0 << 8 | y1 << 12.
__device__ __forceinline__ uint32_t lanes_box(uint64_t mask)
{
    const uint32_t y0 = (uint32_t)__builtin_ctzll(mask) >> 3, y1 = (63u - (uint32_t)__builtin_clzll(mask)) >> 3;
    uint32_t c = (uint32_t)mask | (uint32_t)(mask >> 32);
    c |= c >> 16;
    c = (c | (c >> 8)) & 0xFFu;
    const uint32_t x0 = (uint32_t)__builtin_ctz(c), x1 = 31u - (uint32_t)__builtin_clz(c);
    return x0 | (x1 << 4) | (y0 << 8) | (y1 << 12);
}

// Can a record reach alpha >= eps_alpha at a pixel centre of the rectangle `lb`
// (lanes_box: of the pixels that still take convexes) of the square at (su,
// sv)?  Its pixel box must meet the rectangle, and no
// hull line may keep x2 above the skip threshold over all pixel centres of
// the rectangle's part of the box (then the pair evaluation skips every one of
// them).  A line's minimum over a rectangle is at a corner; the margin covers
// the rounding of this test and of the pair evaluation.
template <int K> __device__ __forceinline__ bool square_meets(const uint8_t *rec, int su, int sv, uint32_t lb)
{
    const RecHeader h = *reinterpret_cast<const RecHeader *>(rec);
    double L[3 * K + 1];
    const double2 *l2 = reinterpret_cast<const double2 *>(rec + REC_HEADER);
#pragma unroll
    for (int q = 0; q < (3 * K + 1) / 2; ++q) {
        const double2 w = l2[q];
        L[2 * q] = w.x;
        L[2 * q + 1] = w.y;
    }
    const int u0 = max(su + (int)(lb & 15u), (int)(h.box_u & 0xFFFFu));
    const int u1 = min(su + (int)((lb >> 4) & 15u), (int)(h.box_u >> 16));
    const int v0 = max(sv + (int)((lb >> 8) & 15u), (int)(h.box_v & 0xFFFFu));
    const int v1 = min(sv + (int)(lb >> 12), (int)(h.box_v >> 16));
    if (u0 > u1 || v0 > v1) return false;
    const double a0 = (double)u0 + 0.5 - (double)h.ox, a1 = (double)u1 + 0.5 - (double)h.ox;
    const double c0 = (double)v0 + 0.5 - (double)h.oy, c1 = (double)v1 + 0.5 - (double)h.oy;
    const double lim = (double)h.thr2 + 1e-3;
    bool ok = true;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const double mn = L[3 * j + 2] + fmin(L[3 * j] * a0, L[3 * j] * a1) + fmin(L[3 * j + 1] * c0, L[3 * j + 1] * c1);
        ok = ok && !(mn > lim); // null lines never reject
    }
    return ok;
}

// Software pipeline of the LDS record batches.  While a batch is composited
// from LDS, the records of the next batch are in flight into registers, and
// the list is kept queued a batch further ahead (TileFeed), so a record load
// seldom waits on its id load and one LDS record buffer suffices.
template <int K, int NT, int BATCH> constexpr int pipe_regs() { return (BATCH * (rec_stride(K) / 16) + NT - 1) / NT; }

// The thread index, opaque to the compiler: what a step between the record
// loops derives from it (addresses, quotients, lane masks) is computed there
// instead of being kept in registers across those loops.
__device__ __forceinline__ int opaque_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// native 16-byte vector (HIP's uint4 is a struct with a union, which keeps a
// register array of it in scratch)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int K, int NT, int NL>
__device__ __forceinline__ void pipe_load_records(u32x4 (&pre)[NL], const uint2 *s_ring, uint32_t head, uint32_t ringmask,
                                                  const uint8_t *__restrict__ records, int cnt)
{
    constexpr int CH = rec_stride(K) / 16;
    const int last = cnt * CH - 1; // chunks past the batch reload its last chunk (never stored)
#pragma clang loop unroll(full)
    for (int r = 0; r < NL; ++r) {
        const int c = min((int)threadIdx.x + r * NT, last);
        const int e = c / CH, part = c - e * CH;
        pre[r] = reinterpret_cast<const u32x4 *>(records + (size_t)s_ring[(head + e) & ringmask].x * rec_stride(K))[part];
    }
}

template <int K, int NT>
__device__ __forceinline__ void load_records_direct(uint4 *lds, const uint2 *s_ring, uint32_t head, uint32_t ringmask,
                                                    const uint8_t *__restrict__ records, int cnt)
{
    constexpr int CH = rec_stride(K) / 16;
    for (int c = opaque_tid(); c < cnt * CH; c += NT) {
        const int e = c / CH, part = c - e * CH;
        reinterpret_cast<u32x4 *>(lds)[c] =
            reinterpret_cast<const u32x4 *>(records + (size_t)s_ring[(head + e) & ringmask].x * rec_stride(K))[part];
    }
}

template <int K, int NT, int NL>
__device__ __forceinline__ void pipe_store_records(const u32x4 (&pre)[NL], uint4 *lds, int cnt)
{
    constexpr int CH = rec_stride(K) / 16;
#pragma clang loop unroll(full)
    for (int r = 0; r < NL; ++r) {
        const int c = (int)threadIdx.x + r * NT;
        if (c < cnt * CH) reinterpret_cast<u32x4 *>(lds)[c] = pre[r];
    }
}

// Work distribution of the persistent compositing grid.  Items (tiles of all
// views, in the order given by `order`, or natural order) are split into one
// contiguous band per XCD; a workgroup takes items from the band of its own XCD
// (workgroups are dealt to the 8 XCDs round-robin), so neighbouring tiles, which
// share convex records, meet in one L2, and steals from the other bands when
// its own runs dry.  Every workgroup exits once all bands are through.
// Items are claimed one at a time: tiles differ by a factor of four and a
// workgroup takes only a few (1.7 tiles each at 979 x 546), so runs of two cost
// more in balance than they save in claims (forward, 317k convexes there 98 -> 78 us,
// 1M at 1920 x 1080 176 -> 167).  A claim's round trip is a microsecond or two: a workgroup's
// first items are its own by its index, without a claim, and a band whose items
// are all given out that way is not claimed from (a 128 x 128 view of one convex:
// 20 -> 11 us).  A claim made ahead, while the last item is worked on, is no gain: it ties an
// item to a workgroup that may be long busy (100k convexes at 1297 x 840: 0.102
// -> 0.139 ms).
struct Claims {
    uint32_t *queues;
    uint32_t total;
    int q, tried;         // the band that items are taken from, bands found dry
    bool first;
    uint32_t item;

    __device__ __forceinline__ Claims(uint32_t *queues_, uint32_t total_)
        : queues(queues_), total(total_), q(blockIdx.x % NUM_QUEUES), tried(0), first(true), item(0)
    {
    }
    __device__ __forceinline__ uint32_t per() const { return (total + NUM_QUEUES - 1) / NUM_QUEUES; }
    __device__ __forceinline__ uint32_t lo(int b) const { return min(total, (uint32_t)b * per()); }
    __device__ __forceinline__ uint32_t size(int b) const { return min(total, ((uint32_t)b + 1u) * per()) - lo(b); }
    // items of a band that belong to workgroups by their index
    __device__ __forceinline__ uint32_t given(int b) const
    {
        return (gridDim.x + (uint32_t)(NUM_QUEUES - 1 - b)) / NUM_QUEUES;
    }
    __device__ __forceinline__ bool take(uint32_t k) // item k of band q
    {
        if (k >= size(q)) return false;
        item = lo(q) + k;
        return true;
    }
    // thread 0 only
    __device__ __forceinline__ uint32_t one()
    {
        bool got = first && take(blockIdx.x / NUM_QUEUES);
        first = false;
        while (!got && tried < NUM_QUEUES) {
            if (given(q) < size(q)) got = take(given(q) + atomicAdd(&queues[QUEUE_STRIDE * q], 1u));
            if (!got) {
                q = (q + 1) % NUM_QUEUES;
                ++tried;
            }
        }
        return got ? item : 0xFFFFFFFFu;
    }
    // The next item, for the whole workgroup (0xFFFFFFFF: none left).
    __device__ __forceinline__ uint32_t next(uint32_t *s_item)
    {
        if (threadIdx.x == 0) *s_item = one();
        __syncthreads();
        // a scalar: what hangs on the item (view, cell, list, image size) then stays
        // in scalar registers
        const uint32_t i = (uint32_t)__builtin_amdgcn_readfirstlane((int)*s_item);
        __syncthreads();
        return i;
    }
};

// A tile's depth-ordered convex list, streamed out of its cell's list into a
// ring in LDS that the batches of records are taken from.  A round reads the
// keys of FEED_SUB * NT consecutive entries, front to back or (REVERSE) back
// to front, and counts those with the tile's mask bit per wavefront; after a
// barrier whole sub-rounds of NT entries are appended in order, as (id,
// position in the cell's list), until enough are queued (the rest is read
// again by the next round).  Only the entries that a round appends have their
// ids read.  About a quarter of a cell's entries are a given tile's at 1M
// convexes and 1080p, but a twelfth where convexes are smaller than a tile
// (200k convexes, 256 x 256), hence rounds of 4 NT: with rounds of NT that
// view's compositing took twice as long.
// While a batch is composited one sub-round is in flight, every entry's key and id
// (request), which the kernels count before and append after the barrier of the
// next batch (publish, append): where the hits are dense enough, the list is then
// read on without a wait.
constexpr int FEED_SUB = 4;
template <int NT, int RING, bool REVERSE> struct TileFeed {
    static constexpr int NW = NT / 64;
    const uint32_t *keys, *ids;  // the cell's list
    int next, count;     // entries gone through / to go through
    uint32_t hitmask;    // the tile's bit in a key
    uint32_t head, tail; // ring positions: first queued entry, end
    uint32_t k0, v0;     // the sub-round in flight: this thread's entry

    __device__ __forceinline__ void request()
    {
        const int i = next + opaque_tid();
        const uint32_t pos = (uint32_t)(REVERSE ? count - 1 - i : i);
        k0 = i < count ? keys[pos] : 0u;
        v0 = i < count ? ids[pos] : 0u;
    }
    __device__ __forceinline__ void publish(uint32_t (*s_cnt)[NW])
    {
        const uint32_t c = (uint32_t)__popcll(__ballot((k0 & hitmask) != 0u));
        const int t = opaque_tid();
        if ((t & 63) == 0) s_cnt[0][t >> 6] = c;
    }
    __device__ __forceinline__ void append(uint32_t k, uint32_t v, bool have_v, int t, const uint32_t *cnt, uint2 *s_ring)
    {
        const int wave = t >> 6;
        uint32_t at = tail, end = tail;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const uint32_t c = cnt[w];
            if (w < wave) at += c;
            end += c;
        }
        tail = (uint32_t)__builtin_amdgcn_readfirstlane((int)end);
        const bool hit = (k & hitmask) != 0u;
        const uint64_t m = __ballot(hit);
        if (hit) {
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            const int i = next + t, pos = REVERSE ? count - 1 - i : i;
            s_ring[(at + rank) & (RING - 1)] = make_uint2(have_v ? v : ids[(uint32_t)pos], (uint32_t)pos);
        }
        next += NT;
    }
    __device__ __forceinline__ void start(const uint32_t *keys_, const uint32_t *ids_, int count_, uint32_t hitmask_)
    {
        keys = keys_; ids = ids_; count = count_; hitmask = hitmask_;
        next = 0;
        head = tail = 0;
    }
    __device__ __forceinline__ bool more() const { return next < count; }
    __device__ __forceinline__ int queued() const { return (int)(tail - head); }
    // Rounds until `want` entries are queued or the list is through (want <=
    // RING - NT - the entries before head that are still in use).  Every thread
    // calls it; returns with the ring readable.
    __device__ __forceinline__ void fill(int want, uint32_t (*s_cnt)[NW], uint2 *s_ring)
    {
        while (queued() < want && more()) {
            const int t = opaque_tid();
            uint32_t k[FEED_SUB];
#pragma unroll
            for (int j = 0; j < FEED_SUB; ++j) {
                const int i = next + j * NT + t;
                k[j] = i < count ? keys[(uint32_t)(REVERSE ? count - 1 - i : i)] : 0u;
            }
#pragma unroll
            for (int j = 0; j < FEED_SUB; ++j) {
                const uint32_t c = (uint32_t)__popcll(__ballot((k[j] & hitmask) != 0u));
                if ((t & 63) == 0) s_cnt[j][t >> 6] = c;
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < FEED_SUB; ++j)
                if (queued() < want && more()) append(k[j], 0u, false, t, s_cnt[j], s_ring);
            __syncthreads();
        }
    }
};
// Entries of the ring: a sub-round, two batches queued and one in use (batches
// of 64, of 32 at 64 threads).
template <int NT> constexpr int feed_ring() { return NT >= 1024 ? 2048 : NT == 256 ? 512 : 256; }

// The workgroup's work counters (per-lane tested / full / hull-size sums and
// the wavefront's evaluation count, which every lane of a wavefront holds),
// stored in the workgroup's own slot of EVAL_FIELDS words.
__device__ __forceinline__ void store_work_counts(unsigned long long *evalcount, unsigned long long *s_ev,
                                                  uint32_t nevals, uint32_t nfull, uint32_t nsumT, uint32_t nwave)
{
    unsigned long long c = nevals, f = nfull, t = nsumT;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        c += __shfl_xor(c, o, 64);
        f += __shfl_xor(f, o, 64);
        t += __shfl_xor(t, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&s_ev[EV_TESTED], c);
        atomicAdd(&s_ev[EV_FULL], f);
        atomicAdd(&s_ev[EV_SUM_T], t);
        atomicAdd(&s_ev[EV_WAVES], (unsigned long long)nwave);
    }
    __syncthreads();
    if (threadIdx.x < EVAL_FIELDS) evalcount[EVAL_FIELDS * blockIdx.x + threadIdx.x] = s_ev[threadIdx.x];
}

} // namespace

// 5 wavefronts per SIMD (at most 96 VGPRs): the compiler keeps a few values
// of the batch loop (one record prefetch register among them) in scratch,
// outside the record loop, and the extra wavefront hides more of the LDS and
// transcendental latency (0.183 -> 0.169 ms at 1M convexes, 1080p, against 4
// wavefronts and 106 VGPRs without spills).  K = 7 and 8 hold more and would
// spill 75 to 79 values: 4 wavefronts.
constexpr int fwd_waves(int K, int TILE) { return K <= (TILE == 8 ? 4 : 6) ? 5 : 4; }
template <int K, int TILE, int BATCH>
__global__ __launch_bounds__(TILE *TILE) __attribute__((amdgpu_waves_per_eu(fwd_waves(K, TILE)))) void render_fwd_kernel(
    const FrameHeader *__restrict__ frame, const uint32_t *__restrict__ order, uint32_t *__restrict__ queues,
    const uint2 *__restrict__ ranges, const uint32_t *__restrict__ keys, const uint32_t *__restrict__ ids,
    const uint8_t *__restrict__ records, RenderArgs ra, uint2 *__restrict__ pixstate,
    unsigned long long *__restrict__ evalcount, u32x4 *__restrict__ zero_acc, uint32_t zero_n4)
{
    constexpr int NT = TILE * TILE;
    constexpr int CH = rec_stride(K) / 16;
    constexpr int RING = feed_ring<NT>();
    static_assert(BATCH <= 64, "one ballot bit per batch entry");
    constexpr int WANT = RING - NT - BATCH; // queued entries to go for: a batch may be in use, a sub-round may overshoot
    static_assert(WANT >= 2 * BATCH, "the ring holds less than two batches");
    __shared__ uint4 lds[BATCH * CH];
    __shared__ uint2 s_ring[RING];
    __shared__ uint32_t s_cnt[FEED_SUB][NT / 64];
    __shared__ uint32_t s_item;
    __shared__ unsigned long long s_ev[EVAL_FIELDS];
    const int lane = threadIdx.x & 63, wbit = threadIdx.x >> 6;
    if (threadIdx.x < EVAL_FIELDS) s_ev[threadIdx.x] = 0ull;
    constexpr int NL = pipe_regs<K, NT, BATCH>();
    u32x4 pre[NL];
    TileFeed<NT, RING, false> feed;
    const ViewDesc *views = reinterpret_cast<const ViewDesc *>(frame + 1);
    const int nviews = (int)frame->nviews;
    const uint32_t total_tiles = frame->total_tiles;
    Claims claims(queues, total_tiles);
    // work counters: pairs tested / pairs past the max-line test (the hull
    // sizes and wavefront evaluations of the same pairs are counted by the
    // backward walk, where they cost less)
    uint32_t nevals = 0, nfull = 0;
    // the backward's accumulators (zero_n4 16-byte words, or none) are cleared
    // here, one slice per tile item, by stores that overlap the compositing
    const uint32_t zper = total_tiles ? (zero_n4 + total_tiles - 1) / total_tiles : 0u;
    for (;;) {
        const uint32_t item = claims.next(&s_item);
        if (item == 0xFFFFFFFFu) break;
        if (zper) {
            const uint32_t z0 = min(item * zper, zero_n4), z1 = min(z0 + zper, zero_n4);
            for (uint32_t z = z0 + threadIdx.x; z < z1; z += NT) zero_acc[z] = u32x4{0u, 0u, 0u, 0u};
        }
        const int gt = order ? (int)order[item] : (int)item;
        const int v = find_view(views, nviews, gt);
        const ViewDesc &vd = views[v];
        const int lt = gt - vd.tile_off;
        const int tx = lt % vd.tiles_x, ty = lt / vd.tiles_x;
        const int W = vd.cam.W, H = vd.cam.H;
        int pdx, pdy;
        tile_pixel<TILE>(pdx, pdy);
        const int u = tx * TILE + pdx, y = ty * TILE + pdy;
        const int su = tx * TILE + (wbit % (TILE / 8)) * 8, sv = ty * TILE + (wbit / (TILE / 8)) * 8; // wave's square
        const bool inside = u < W && y < H;
        const float pxf = (float)u + 0.5f, pyf = (float)y + 0.5f;
        // the tile's cell and its bit in the cell's keys
        const uint2 rg = ranges[tile_cell(vd, (uint32_t)tx, (uint32_t)ty)];
        const uint32_t hitmask = tile_bit(vd, frame->key_bits, (uint32_t)tx, (uint32_t)ty);

        float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, Tlast = 1.0f;
        uint32_t nend = 0; // position after the last contributor in the cell's list
        bool done = !inside;
        int cnt = 0;
        if (rg.y > rg.x) { // prologue: the first batch's ids, then its records
            feed.start(keys + rg.x, ids + rg.x, (int)(rg.y - rg.x), hitmask);
            feed.fill(2 * BATCH, s_cnt, s_ring); // most tiles need no more
            feed.request();
            cnt = min(BATCH, feed.queued());
            if (cnt > 0) pipe_load_records<K, NT, NL>(pre, s_ring, feed.head, RING - 1, records, cnt);
        }
        while (cnt > 0) {
            pipe_store_records<K, NT, NL>(pre, lds, cnt);
            const bool refill = feed.queued() <= RING - NT && feed.more();
            if (refill) feed.publish(s_cnt);
            __syncthreads();
            const uint32_t head = feed.head;
            feed.head += (uint32_t)cnt;
            // the next batch, of what the ring held before this refill (unless
            // that is little: then the list is read on first)
            const int ncnt = feed.queued() >= BATCH / 2 || !feed.more() ? min(BATCH, feed.queued()) : 0;
            if (refill) {
                feed.append(feed.k0, feed.v0, true, opaque_tid(), s_cnt[0], s_ring);
                feed.request();
            }
            if (ncnt > 0) pipe_load_records<K, NT, NL>(pre, s_ring, feed.head, RING - 1, records, ncnt);
            // the wave's records of this batch (lane e tests entry e against
            // the wave's square), front to back in a wave-uniform walk
            uint64_t M = 0;
            int last = -1; // the pixel's last contributor of this batch
            if (const uint64_t live = __ballot(!done)) {
                const bool meets = lane < cnt && square_meets<K>(reinterpret_cast<const uint8_t *>(&lds[min(lane, BATCH - 1) * CH]),
                                                                 su, sv, lanes_box(live));
                M = __ballot(meets);
            }
            while (M) {
                const int e = __builtin_ctzll(M);
                M &= M - 1;
                const uint8_t *rec = reinterpret_cast<const uint8_t *>(&lds[e * CH]);
                PairEval<K> pe;
                bool tested, full;
                // all K line slots (slots past T hold null lines): a dispatch on
                // T costs the forward more than the null lines it saves
                const bool hit = eval_pair<K, K>(rec, !done, u, y, pxf, pyf, ra.eps_alpha, pe, tested, full);
                nevals += tested;
                nfull += full;
                if (hit) {
                    const RecHeader &h = *reinterpret_cast<const RecHeader *>(rec);
                    const float w = T * pe.alpha;
                    C0 = fmaf(w, h.rgb[0], C0);
                    C1 = fmaf(w, h.rgb[1], C1);
                    C2 = fmaf(w, h.rgb[2], C2);
                    Tlast = T;
                    T = T * pe.oma;
                    last = e;
                    done = T < ra.t_min;
                }
                if (__all(done)) break;
            }
            if (last >= 0) nend = s_ring[(head + (uint32_t)last) & (RING - 1)].y + 1u;
            if (__syncthreads_and(done)) break;
            cnt = ncnt;
            if (cnt == 0 && feed.queued() < BATCH && feed.more()) {
                feed.fill(WANT, s_cnt, s_ring);
                feed.request();
            }
            if (cnt == 0) {
                cnt = min(BATCH, feed.queued());
                if (cnt > 0) pipe_load_records<K, NT, NL>(pre, s_ring, feed.head, RING - 1, records, cnt);
            }
        }
        if (inside) {
            const size_t pix = (size_t)y * W + u;
            float *o = vd.out_rgb + 3 * pix;
            o[0] = fmaf(T, ra.bg[0], C0);
            o[1] = fmaf(T, ra.bg[1], C1);
            o[2] = fmaf(T, ra.bg[2], C2);
            pixstate[vd.pix_off + pix] = make_uint2(nend, __float_as_uint(Tlast));
        }
    }
    if (evalcount) store_work_counts(evalcount, s_ev, nevals, nfull, 0u, 0u);
}

// Compact per-pair gradient values of a record with NL hull lines: a[NL]
// b[NL] c[NL] (base-2 line coefficients), sigma', opacity, rgb[3], and
// sum_j dL/dx2_j x2_j, padded with zeros to a multiple of 4 for the wave sums.
template <int NL> constexpr int bwd_values() { return 3 * NL + 6; }
template <int NL> constexpr int bwd_padded() { return (bwd_values<NL>() + 3) & ~3; }

// Slot of compact value qv of a record with T lines in the accumulator row
// a[K] b[K] c[K] sigma' opacity rgb[3] x2sum.
template <int K> __device__ __forceinline__ int acc_slot(int qv, int T)
{
    return qv < T ? qv : qv < 2 * T ? K + (qv - T) : qv < 3 * T ? 2 * K + (qv - 2 * T) : 3 * K + (qv - 3 * T);
}

// A pixel's state in the back-to-front walk: dL/dC, the transmittance after
// its last contributor, the transmittance before the pair being walked (T_n,
// recovered by division), and the colour composited behind it.
struct BwdPixel {
    float g0, g1, g2, Tlast, Tcur, B0, B1, B2;
    bool first;
};

// The pixel's transmittance before a contributing record (0 for a lane that does
// not contribute: it zeroes all of its values) and dL/dalpha.
__device__ __forceinline__ float pixel_before(const BwdPixel &P, bool contrib, float oma)
{
    return contrib ? (P.first ? P.Tlast : P.Tcur * __builtin_amdgcn_rcpf(oma)) : 0.0f;
}
__device__ __forceinline__ float pixel_dalpha(const BwdPixel &P, const float *rgb, float Tn)
{
    return Tn * (P.g0 * (rgb[0] - P.B0) + P.g1 * (rgb[1] - P.B1) + P.g2 * (rgb[2] - P.B2));
}
// The pixel's walk advanced past a contributing record.
__device__ __forceinline__ void pixel_pass(BwdPixel &P, const float *rgb, float Tn, float alpha, float oma)
{
    P.first = false;
    P.Tcur = Tn;
    P.B0 = fmaf(alpha, rgb[0], oma * P.B0);
    P.B1 = fmaf(alpha, rgb[1], oma * P.B1);
    P.B2 = fmaf(alpha, rgb[2], oma * P.B2);
}
// A pixel's compact gradient values of one record (see bwd_values), stored into v.
template <int K, int NL>
__device__ __forceinline__ void pair_values(const RecHeader &h, const PairEval<K> &pe, const BwdPixel &P, float Tn, float dLda,
                                            float pxf, float pyf, float *v)
{
    const float ta = Tn * pe.alpha;
    v[3 * NL + 2] = P.g0 * ta;
    v[3 * NL + 3] = P.g1 * ta;
    v[3 * NL + 4] = P.g2 * ta;
    v[3 * NL + 1] = dLda * pe.I;
    const float dLdz = -dLda * h.opacity * pe.I * pe.omI; // I = Sigmoid(-z), z = sigma' phi
    v[3 * NL] = dLdz * pe.phi2 * (float)LN2;
    const float dLdphi2 = dLdz * h.sigma_p * (float)LN2;
    const float gs = dLdphi2 * pe.inv_sum; // dL/dx2_j = gs e_j (softmax weights)
    const float dxf = pxf - h.ox, dyf = pyf - h.oy;
    float gdl = 0.0f;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const float gx = gs * pe.e[j];
        v[j] = gx * dxf;
        v[NL + j] = gx * dyf;
        v[2 * NL + j] = gx;
        gdl = fmaf(gx, pe.x2[j], gdl);
    }
    v[3 * NL + 5] = gdl;
#pragma unroll
    for (int qv = bwd_values<NL>(); qv < bwd_padded<NL>(); ++qv) v[qv] = 0.0f;
}
// The wavefront's sums of a record's values, added to its LDS slot: whole-wave
// sums even when few lanes contribute (lane-by-lane LDS atomics serialise badly
// when a record covers the square).
template <int NP> __device__ __forceinline__ void add_wave_sums(float *val, float *slot)
{
    constexpr int Q = NP / 4;
    wave_to_rows<NP>(val);
    const float total = row_reduce<Q>(val);
    const int li = threadIdx.x & 15;
    if ((rr_first_lanes(Q) >> li) & 1u) { // one lane per (row, value) adds the wave's sum
        const int qv = (int)((rr_map(Q) >> (4 * li)) & 15u);
        atomicAdd(slot + ((threadIdx.x & 63) >> 4) * Q + qv, total);
    }
}

// Backward of one record for the wavefront's pixels: recompute the pair (the
// forward's decisions, bit for bit), recover T_n, form the pixel's gradient
// values, sum them over the wavefront and add the four row sums into the
// record's LDS slot (compact layout, bwd_padded<K>() floats).
template <int K, int NL>
__device__ __forceinline__ void bwd_record(const uint8_t *rec, bool live, int u, int y, float pxf, float pyf,
                                           float eps, BwdPixel &P, float *slot, bool &full)
{
    PairEval<K> pe;
    bool tested;
    const bool contrib = eval_pair<K, NL>(rec, live, u, y, pxf, pyf, eps, pe, tested, full);
    if (__ballot(contrib) == 0ull) return; // wave-uniform
    const RecHeader &h = *reinterpret_cast<const RecHeader *>(rec);
    // branch-free: every pe field is finite
    const float Tn = pixel_before(P, contrib, pe.oma);
    float val[bwd_padded<NL>()];
    pair_values<K, NL>(h, pe, P, Tn, pixel_dalpha(P, h.rgb, Tn), pxf, pyf, val);
    if (contrib) pixel_pass(P, h.rgb, Tn, pe.alpha, pe.oma);
    add_wave_sums<bwd_padded<NL>()>(val, slot);
}

template <int K, int TILE, int BATCH>
__global__ __launch_bounds__(TILE *TILE) __attribute__((amdgpu_waves_per_eu(K <= 6 ? 5 : 1))) void render_bwd_kernel(
    const FrameHeader *__restrict__ frame, const uint32_t *__restrict__ order, uint32_t *__restrict__ queues,
    const uint2 *__restrict__ ranges, const uint32_t *__restrict__ keys, const uint32_t *__restrict__ ids,
    const uint8_t *__restrict__ records, RenderArgs ra, const uint2 *__restrict__ pixstate,
    float *__restrict__ acc, unsigned long long *__restrict__ evalcount)
{
    constexpr int NT = TILE * TILE;
    constexpr int CH = rec_stride(K) / 16;
    constexpr int AS = acc_stride(K);
    constexpr int NP = bwd_padded<K>(); // LDS slot per batch entry (compact values of the largest hull)
    constexpr int RING = feed_ring<NT>();
    static_assert(BATCH <= 64, "one ballot bit per batch entry");
    constexpr int WANT = RING - NT - BATCH; // queued entries to go for: a batch may be in use, a sub-round may overshoot
    static_assert(WANT >= 2 * BATCH, "the ring holds less than two batches");
    __shared__ uint4 lds[BATCH * CH];
    __shared__ uint2 s_ring[RING];
    __shared__ uint32_t s_cnt[FEED_SUB][NT / 64];
    // per entry sums of the block's waves, flushed after each batch
    __shared__ float s_acc[BATCH * NP];
    __shared__ int s_maxn;
    __shared__ uint32_t s_item;
    __shared__ unsigned long long s_ev[EVAL_FIELDS];
    for (int c = threadIdx.x; c < BATCH * NP; c += NT) s_acc[c] = 0.0f;
    if (threadIdx.x < EVAL_FIELDS) s_ev[threadIdx.x] = 0ull;
    const ViewDesc *views = reinterpret_cast<const ViewDesc *>(frame + 1);
    const int nviews = (int)frame->nviews;
    const uint32_t total_tiles = frame->total_tiles;
    const int lane = threadIdx.x & 63, wbit = threadIdx.x >> 6;
    Claims claims(queues, total_tiles);
    uint32_t nfull = 0, nsumT = 0, nwave = 0;
    TileFeed<NT, RING, true> feed;
    for (;;) {
        const uint32_t item = claims.next(&s_item);
        if (item == 0xFFFFFFFFu) break;
        const int gt = order ? (int)order[item] : (int)item;
        const int v = find_view(views, nviews, gt);
        const ViewDesc &vd = views[v];
        const int lt = gt - vd.tile_off;
        const int tx = lt % vd.tiles_x, ty = lt / vd.tiles_x;
        const int W = vd.cam.W, H = vd.cam.H;
        int pdx, pdy;
        tile_pixel<TILE>(pdx, pdy);
        const int u = tx * TILE + pdx, y = ty * TILE + pdy;
        const int su = tx * TILE + (wbit % (TILE / 8)) * 8, sv = ty * TILE + (wbit / (TILE / 8)) * 8; // wave's square
        const bool inside = u < W && y < H;
        const float pxf = (float)u + 0.5f, pyf = (float)y + 0.5f;
        // the tile's cell and its bit in the cell's keys
        const uint2 rg = ranges[tile_cell(vd, (uint32_t)tx, (uint32_t)ty)];
        const uint32_t hitmask = tile_bit(vd, frame->key_bits, (uint32_t)tx, (uint32_t)ty);

        BwdPixel P{0.f, 0.f, 0.f, 1.f, 1.f, ra.bg[0], ra.bg[1], ra.bg[2], true};
        int nend = 0;
        if (inside) {
            const size_t pix = (size_t)y * W + u;
            const float *g = vd.dl_drgb + 3 * pix;
            P.g0 = g[0];
            P.g1 = g[1];
            P.g2 = g[2];
            const uint2 ps = pixstate[vd.pix_off + pix];
            nend = (int)ps.x;
            P.Tlast = __uint_as_float(ps.y);
            P.Tcur = P.Tlast;
        }
        if (threadIdx.x == 0) s_maxn = 0;
        __syncthreads();
        if (nend > 0) atomicMax(&s_maxn, nend);
        __syncthreads();
        const int maxn = min(__builtin_amdgcn_readfirstlane(s_maxn), (int)(rg.y - rg.x));
        int wmaxn = nend; // the wave's last contributor
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) wmaxn = max(wmaxn, __shfl_xor(wmaxn, o, 64));
        wmaxn = __builtin_amdgcn_readfirstlane(wmaxn);

        // batches walk the list back to front from the tile's last contributor
        // (the walk is VALU-bound: plain loads, no prefetch registers)
        if (maxn > 0) {
            feed.start(keys + rg.x, ids + rg.x, maxn, hitmask);
            feed.request();
        }
        while (maxn > 0) {
            __syncthreads(); // the previous batch's records are flushed
            if (feed.queued() < BATCH && feed.more()) {
                feed.fill(2 * BATCH, s_cnt, s_ring);
                feed.request();
            }
            const int cnt = min(BATCH, feed.queued());
            if (cnt == 0) break;
            load_records_direct<K, NT>(lds, s_ring, feed.head, RING - 1, records, cnt);
            const bool refill = feed.queued() <= RING - NT && feed.more();
            if (refill) feed.publish(s_cnt);
            __syncthreads();
            const uint32_t head = feed.head;
            feed.head += (uint32_t)cnt;
            if (refill) {
                feed.append(feed.k0, feed.v0, true, opaque_tid(), s_cnt[0], s_ring);
                feed.request();
            }
            // the wave's records of this batch before its last contributor, back to front
            const int mine_e = min(lane, cnt - 1);
            const uint8_t *mine = reinterpret_cast<const uint8_t *>(&lds[mine_e * CH]);
            const int mypos = (int)s_ring[(head + (uint32_t)mine_e) & (RING - 1)].y; // lane e: list position of entry e
            // (of the pixels whose last contributor is not before the batch's last entry)
            const uint64_t live = __ballot(nend > __builtin_amdgcn_readlane(mypos, cnt - 1));
            const bool meets = live != 0ull && lane < cnt && mypos < wmaxn && square_meets<K>(mine, su, sv, lanes_box(live));
            const int myT = reinterpret_cast<const RecHeader *>(mine)->T; // lane e: hull size of entry e
            uint64_t M = __ballot(meets);
            while (M) {
                const int e = __builtin_ctzll(M);
                M &= M - 1;
                const uint8_t *rec = reinterpret_cast<const uint8_t *>(&lds[e * CH]);
                const int Tr = __builtin_amdgcn_readlane(myT, e);
                const bool live = __builtin_amdgcn_readlane(mypos, e) < nend;
                bool full = false;
                CS_DISPATCH_NL(K, Tr, bwd_record<K, NLL>(rec, live, u, y, pxf, pyf, ra.eps_alpha, P, &s_acc[e * NP], full));
                nfull += full;
                nsumT += full ? (uint32_t)Tr : 0u;
                nwave += __any(full) ? 1u : 0u;
            }
            // one global atomic per (entry, value) for the whole workgroup; the
            // compact values of entry e go to the slots of its hull size
            __syncthreads();
            for (int c = opaque_tid(); c < cnt * NP; c += NT) {
                const int e = c / NP, qv = c - e * NP;
                float *src = &s_acc[c];
                const float a = *src;
                if (a != 0.0f) {
                    const int T = reinterpret_cast<const RecHeader *>(&lds[e * CH])->T;
                    unsafeAtomicAdd(&acc[(size_t)s_ring[(head + (uint32_t)e) & (RING - 1)].x * AS + acc_slot<K>(qv, T)], a);
                    *src = 0.0f;
                }
            }
        }
    }
    if (evalcount) store_work_counts(evalcount, s_ev, 0u, nfull, nsumT, nwave);
}

// ---------------------------------------------- compositing, split by record
//
// A wavefront walks its square's records one after another, 0.4 us each in the
// forward when it has a SIMD to itself, so a small view takes as long as its
// longest walk however many CUs are idle.  What takes the time, evaluating a
// record's alpha at the pixels, does not depend on the records before it: here a
// workgroup of four wavefronts takes one 8 x 8 square, each evaluates two of the
// next SPLIT records (both at once, one's latencies behind the other's), passes
// alpha and 1 - alpha through LDS, and all four composite the SPLIT records in
// order, each for itself (the same operations on the same values: the image and
// the walk's decisions are the other kernels' bit for bit).  The backward does
// the same: alphas by record, T_n and the colour behind in order by every
// wavefront, then each forms and sums the gradient values of its two records.
// All four wavefronts composite every record, and a record is loaded and tested
// for every square instead of every tile: where the chip is full it takes 2.3
// times as long (1M convexes, 1920 x 1080: forward 175 -> 412 us, backward 313 ->
// 782), so it is for views whose squares do not fill the chip (split_by_record).
constexpr int SPLIT = 8;
constexpr float NOT_FULL = -1.0f, NOT_TESTED = -2.0f; // in place of alpha

// The square of a work item: tile gt, square (sx, sy) of it.
struct SquareItem { int gt, sx, sy; };
__device__ __forceinline__ SquareItem square_item(uint32_t item, const uint32_t *order, uint32_t side)
{
    const uint32_t per = side * side, t = item / per, s = item - t * per;
    return {order ? __builtin_amdgcn_readfirstlane((int)order[t]) : (int)t, (int)(s % side), (int)(s / side)};
}
// The set of M without its i lowest members.
__device__ __forceinline__ uint64_t drop_lowest(uint64_t M, int i)
{
    for (; i > 0; --i) M &= M - 1;
    return M;
}

template <int K>
__global__ __launch_bounds__(256) void render_fwd_split_kernel(
    const FrameHeader *__restrict__ frame, const uint32_t *__restrict__ order, uint32_t *__restrict__ queues,
    const uint2 *__restrict__ ranges, const uint32_t *__restrict__ keys, const uint32_t *__restrict__ ids,
    const uint8_t *__restrict__ records, RenderArgs ra, uint2 *__restrict__ pixstate,
    unsigned long long *__restrict__ evalcount, u32x4 *__restrict__ zero_acc, uint32_t zero_n4)
{
    constexpr int NT = 256, BATCH = 64, RING = feed_ring<NT>(), WANT = RING - NT - BATCH;
    constexpr int CH = rec_stride(K) / 16, NL = pipe_regs<K, NT, BATCH>();
    __shared__ uint4 lds[BATCH * CH];
    __shared__ uint2 s_ring[RING];
    __shared__ uint32_t s_cnt[FEED_SUB][NT / 64];
    __shared__ float2 s_ab[2][SPLIT][64]; // alpha (or why there is none) and 1 - alpha by record and pixel
    __shared__ uint32_t s_item;
    __shared__ unsigned long long s_ev[EVAL_FIELDS];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (threadIdx.x < EVAL_FIELDS) s_ev[threadIdx.x] = 0ull;
    u32x4 pre[NL];
    TileFeed<NT, RING, false> feed;
    const ViewDesc *views = reinterpret_cast<const ViewDesc *>(frame + 1);
    const int nviews = (int)frame->nviews;
    const uint32_t side = (uint32_t)ra.tile / 8u, total = frame->total_tiles * side * side;
    Claims claims(queues, total);
    uint32_t nevals = 0, nfull = 0;
    const uint32_t zper = total ? (zero_n4 + total - 1) / total : 0u;
    int buf = 0;
    for (;;) {
        const uint32_t item = claims.next(&s_item);
        if (item == 0xFFFFFFFFu) break;
        if (zper) {
            const uint32_t z0 = min(item * zper, zero_n4), z1 = min(z0 + zper, zero_n4);
            for (uint32_t z = z0 + threadIdx.x; z < z1; z += NT) zero_acc[z] = u32x4{0u, 0u, 0u, 0u};
        }
        const SquareItem it = square_item(item, order, side);
        const ViewDesc &vd = views[find_view(views, nviews, it.gt)];
        const int lt = it.gt - vd.tile_off, tx = lt % vd.tiles_x, ty = lt / vd.tiles_x;
        const int W = vd.cam.W, H = vd.cam.H;
        const int su = tx * ra.tile + 8 * it.sx, sv = ty * ra.tile + 8 * it.sy;
        if (su >= W || sv >= H) continue; // a square past the image's edge
        const int u = su + (lane & 7), y = sv + (lane >> 3);
        const bool inside = u < W && y < H;
        const float pxf = (float)u + 0.5f, pyf = (float)y + 0.5f;
        const uint2 rg = ranges[tile_cell(vd, (uint32_t)tx, (uint32_t)ty)];
        const uint32_t hitmask = tile_bit(vd, frame->key_bits, (uint32_t)tx, (uint32_t)ty);

        float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, Tlast = 1.0f;
        uint32_t nend = 0;
        bool done = !inside;
        int cnt = 0;
        if (rg.y > rg.x) {
            feed.start(keys + rg.x, ids + rg.x, (int)(rg.y - rg.x), hitmask);
            feed.fill(2 * BATCH, s_cnt, s_ring);
            feed.request();
            cnt = min(BATCH, feed.queued());
            if (cnt > 0) pipe_load_records<K, NT, NL>(pre, s_ring, feed.head, RING - 1, records, cnt);
        }
        while (cnt > 0) {
            pipe_store_records<K, NT, NL>(pre, lds, cnt);
            const bool refill = feed.queued() <= RING - NT && feed.more();
            if (refill) feed.publish(s_cnt);
            __syncthreads();
            const uint32_t head = feed.head;
            feed.head += (uint32_t)cnt;
            const int ncnt = feed.queued() >= BATCH / 2 || !feed.more() ? min(BATCH, feed.queued()) : 0;
            if (refill) {
                feed.append(feed.k0, feed.v0, true, opaque_tid(), s_cnt[0], s_ring);
                feed.request();
            }
            if (ncnt > 0) pipe_load_records<K, NT, NL>(pre, s_ring, feed.head, RING - 1, records, ncnt);
            uint64_t M = 0;
            if (const uint64_t live = __ballot(!done))
                M = __ballot(lane < cnt && square_meets<K>(reinterpret_cast<const uint8_t *>(&lds[min(lane, BATCH - 1) * CH]), su, sv,
                                                           lanes_box(live)));
            int last = -1;
            while (M && !__all(done)) {
                // the next SPLIT records: this wavefront's two, evaluated together
                uint64_t mine = drop_lowest(M, 2 * wave);
                if (mine) {
                    const int e0 = __builtin_ctzll(mine);
                    mine &= mine - 1;
                    const int e1 = mine ? __builtin_ctzll(mine) : e0;
                    PairEval<K> p0, p1;
                    bool t0, f0, t1, f1;
                    p0.alpha = p0.oma = p1.alpha = p1.oma = 0.0f;
                    eval_pair<K, K>(reinterpret_cast<const uint8_t *>(&lds[e0 * CH]), !done, u, y, pxf, pyf, ra.eps_alpha, p0, t0, f0);
                    eval_pair<K, K>(reinterpret_cast<const uint8_t *>(&lds[e1 * CH]), !done, u, y, pxf, pyf, ra.eps_alpha, p1, t1, f1);
                    s_ab[buf][2 * wave][lane] = make_float2(f0 ? p0.alpha : t0 ? NOT_FULL : NOT_TESTED, p0.oma);
                    s_ab[buf][2 * wave + 1][lane] = make_float2(f1 ? p1.alpha : t1 ? NOT_FULL : NOT_TESTED, p1.oma);
                }
                __syncthreads();
#pragma unroll
                for (int j = 0; j < SPLIT; ++j) {
                    if (M == 0) break;
                    const int e = __builtin_ctzll(M);
                    M &= M - 1;
                    const float2 ab = s_ab[buf][j][lane];
                    const RecHeader &h = *reinterpret_cast<const RecHeader *>(&lds[e * CH]);
                    const float c0 = h.rgb[0], c1 = h.rgb[1], c2 = h.rgb[2];
                    const bool tested = !done && ab.x != NOT_TESTED, full = tested && ab.x != NOT_FULL;
                    nevals += tested;
                    nfull += full;
                    if (full && !(ab.x < ra.eps_alpha)) {
                        const float w = T * ab.x;
                        C0 = fmaf(w, c0, C0);
                        C1 = fmaf(w, c1, C1);
                        C2 = fmaf(w, c2, C2);
                        Tlast = T;
                        T = T * ab.y;
                        last = e;
                        done = T < ra.t_min;
                    }
                }
                buf ^= 1; // (a wavefront two steps ahead would wait at the barrier between)
            }
            if (last >= 0) nend = s_ring[(head + (uint32_t)last) & (RING - 1)].y + 1u;
            if (__syncthreads_and(done)) break;
            cnt = ncnt;
            if (cnt == 0 && feed.queued() < BATCH && feed.more()) {
                feed.fill(WANT, s_cnt, s_ring);
                feed.request();
            }
            if (cnt == 0) {
                cnt = min(BATCH, feed.queued());
                if (cnt > 0) pipe_load_records<K, NT, NL>(pre, s_ring, feed.head, RING - 1, records, cnt);
            }
        }
        if (inside && wave == 0) {
            const size_t pix = (size_t)y * W + u;
            float *o = vd.out_rgb + 3 * pix;
            o[0] = fmaf(T, ra.bg[0], C0);
            o[1] = fmaf(T, ra.bg[1], C1);
            o[2] = fmaf(T, ra.bg[2], C2);
            pixstate[vd.pix_off + pix] = make_uint2(nend, __float_as_uint(Tlast));
        }
    }
    // every wavefront walked the same pairs: one counts them
    if (wave != 0) nevals = nfull = 0;
    if (evalcount) store_work_counts(evalcount, s_ev, nevals, nfull, 0u, 0u);
}

template <int K>
__global__ __launch_bounds__(256) void render_bwd_split_kernel(
    const FrameHeader *__restrict__ frame, const uint32_t *__restrict__ order, uint32_t *__restrict__ queues,
    const uint2 *__restrict__ ranges, const uint32_t *__restrict__ keys, const uint32_t *__restrict__ ids,
    const uint8_t *__restrict__ records, RenderArgs ra, const uint2 *__restrict__ pixstate,
    float *__restrict__ acc, unsigned long long *__restrict__ evalcount)
{
    constexpr int NT = 256, BATCH = 64, RING = feed_ring<NT>(), WANT = RING - NT - BATCH;
    constexpr int CH = rec_stride(K) / 16, AS = acc_stride(K), NP = bwd_padded<K>();
    __shared__ uint4 lds[BATCH * CH];
    __shared__ uint2 s_ring[RING];
    __shared__ uint32_t s_cnt[FEED_SUB][NT / 64];
    __shared__ float s_acc[BATCH * NP];
    __shared__ float2 s_ab[2][SPLIT][64]; // alpha (NOT_FULL: no contribution) and 1 - alpha
    __shared__ uint32_t s_item;
    __shared__ unsigned long long s_ev[EVAL_FIELDS];
    for (int c = threadIdx.x; c < BATCH * NP; c += NT) s_acc[c] = 0.0f;
    if (threadIdx.x < EVAL_FIELDS) s_ev[threadIdx.x] = 0ull;
    const ViewDesc *views = reinterpret_cast<const ViewDesc *>(frame + 1);
    const int nviews = (int)frame->nviews;
    const uint32_t side = (uint32_t)ra.tile / 8u, total = frame->total_tiles * side * side;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    Claims claims(queues, total);
    uint32_t nfull = 0, nsumT = 0, nwave = 0;
    TileFeed<NT, RING, true> feed;
    int buf = 0;
    for (;;) {
        const uint32_t item = claims.next(&s_item);
        if (item == 0xFFFFFFFFu) break;
        const SquareItem it = square_item(item, order, side);
        const ViewDesc &vd = views[find_view(views, nviews, it.gt)];
        const int lt = it.gt - vd.tile_off, tx = lt % vd.tiles_x, ty = lt / vd.tiles_x;
        const int W = vd.cam.W, H = vd.cam.H;
        const int su = tx * ra.tile + 8 * it.sx, sv = ty * ra.tile + 8 * it.sy;
        if (su >= W || sv >= H) continue;
        const int u = su + (lane & 7), y = sv + (lane >> 3);
        const bool inside = u < W && y < H;
        const float pxf = (float)u + 0.5f, pyf = (float)y + 0.5f;
        const uint2 rg = ranges[tile_cell(vd, (uint32_t)tx, (uint32_t)ty)];
        const uint32_t hitmask = tile_bit(vd, frame->key_bits, (uint32_t)tx, (uint32_t)ty);

        BwdPixel P{0.f, 0.f, 0.f, 1.f, 1.f, ra.bg[0], ra.bg[1], ra.bg[2], true};
        int nend = 0;
        if (inside) {
            const size_t pix = (size_t)y * W + u;
            const float *g = vd.dl_drgb + 3 * pix;
            P.g0 = g[0];
            P.g1 = g[1];
            P.g2 = g[2];
            const uint2 ps = pixstate[vd.pix_off + pix];
            nend = (int)ps.x;
            P.Tlast = __uint_as_float(ps.y);
            P.Tcur = P.Tlast;
        }
        int wmaxn = nend; // the square's last contributor
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) wmaxn = max(wmaxn, __shfl_xor(wmaxn, o, 64));
        const int maxn = min(__builtin_amdgcn_readfirstlane(wmaxn), (int)(rg.y - rg.x));
        if (maxn > 0) {
            feed.start(keys + rg.x, ids + rg.x, maxn, hitmask);
            feed.request();
        }
        while (maxn > 0) {
            __syncthreads(); // the previous batch's records are flushed
            if (feed.queued() < BATCH && feed.more()) {
                feed.fill(2 * BATCH, s_cnt, s_ring);
                feed.request();
            }
            const int cnt = min(BATCH, feed.queued());
            if (cnt == 0) break;
            load_records_direct<K, NT>(lds, s_ring, feed.head, RING - 1, records, cnt);
            const bool refill = feed.queued() <= RING - NT && feed.more();
            if (refill) feed.publish(s_cnt);
            __syncthreads();
            const uint32_t head = feed.head;
            feed.head += (uint32_t)cnt;
            if (refill) {
                feed.append(feed.k0, feed.v0, true, opaque_tid(), s_cnt[0], s_ring);
                feed.request();
            }
            const int mine_e = min(lane, cnt - 1);
            const uint8_t *mine_r = reinterpret_cast<const uint8_t *>(&lds[mine_e * CH]);
            const int mypos = (int)s_ring[(head + (uint32_t)mine_e) & (RING - 1)].y; // lane e: list position of entry e
            const int myT = reinterpret_cast<const RecHeader *>(mine_r)->T;
            const uint64_t live = __ballot(nend > __builtin_amdgcn_readlane(mypos, cnt - 1));
            uint64_t M = 0;
            if (live) M = __ballot(lane < cnt && square_meets<K>(mine_r, su, sv, lanes_box(live)));
            while (M) {
                uint64_t mine = drop_lowest(M, 2 * wave);
                const bool some = mine != 0ull, both = (mine & (mine - 1)) != 0ull;
                int e0 = 0, e1 = 0;
                PairEval<K> p0, p1;
                bool c0 = false, c1 = false;
                if (some) {
                    e0 = __builtin_ctzll(mine);
                    mine &= mine - 1;
                    e1 = both ? __builtin_ctzll(mine) : e0;
                    bool tested, f0, f1;
                    c0 = eval_pair<K, K>(reinterpret_cast<const uint8_t *>(&lds[e0 * CH]),
                                         __builtin_amdgcn_readlane(mypos, e0) < nend, u, y, pxf, pyf, ra.eps_alpha, p0, tested, f0);
                    c1 = eval_pair<K, K>(reinterpret_cast<const uint8_t *>(&lds[e1 * CH]),
                                         both && __builtin_amdgcn_readlane(mypos, e1) < nend, u, y, pxf, pyf, ra.eps_alpha, p1, tested, f1);
                    s_ab[buf][2 * wave][lane] = c0 ? make_float2(p0.alpha, p0.oma) : make_float2(NOT_FULL, 1.0f);
                    s_ab[buf][2 * wave + 1][lane] = c1 ? make_float2(p1.alpha, p1.oma) : make_float2(NOT_FULL, 1.0f);
                    const uint32_t T0 = (uint32_t)__builtin_amdgcn_readlane(myT, e0), T1 = (uint32_t)__builtin_amdgcn_readlane(myT, e1);
                    nfull += (f0 ? 1u : 0u) + (f1 ? 1u : 0u);
                    nsumT += (f0 ? T0 : 0u) + (f1 ? T1 : 0u);
                    nwave += (__any(f0) ? 1u : 0u) + (__any(f1) ? 1u : 0u);
                }
                __syncthreads();
                // in order: T_n and dL/dalpha of this wavefront's records
                float Tn0 = 0.0f, Tn1 = 0.0f, da0 = 0.0f, da1 = 0.0f;
#pragma unroll
                for (int j = 0; j < SPLIT; ++j) {
                    if (M == 0) break;
                    const int e = __builtin_ctzll(M);
                    M &= M - 1;
                    const float2 ab = s_ab[buf][j][lane];
                    const RecHeader &h = *reinterpret_cast<const RecHeader *>(&lds[e * CH]);
                    const float rgb[3] = {h.rgb[0], h.rgb[1], h.rgb[2]};
                    const bool contrib = ab.x != NOT_FULL;
                    const float Tn = pixel_before(P, contrib, ab.y);
                    if (j / 2 == wave) {
                        const float da = pixel_dalpha(P, rgb, Tn);
                        if (j % 2) { Tn1 = Tn; da1 = da; }
                        else { Tn0 = Tn; da0 = da; }
                    }
                    if (contrib) pixel_pass(P, rgb, Tn, ab.x, ab.y);
                }
                buf ^= 1;
                // their gradient values (null lines past T give zeros)
                float val[NP];
                if (__any(c0)) {
                    pair_values<K, K>(*reinterpret_cast<const RecHeader *>(&lds[e0 * CH]), p0, P, Tn0, da0, pxf, pyf, val);
                    add_wave_sums<NP>(val, &s_acc[e0 * NP]);
                }
                if (__any(c1)) {
                    pair_values<K, K>(*reinterpret_cast<const RecHeader *>(&lds[e1 * CH]), p1, P, Tn1, da1, pxf, pyf, val);
                    add_wave_sums<NP>(val, &s_acc[e1 * NP]);
                }
            }
            __syncthreads();
            for (int c = opaque_tid(); c < cnt * NP; c += NT) {
                const int e = c / NP, qv = c - e * NP;
                const float a = s_acc[c];
                if (a != 0.0f) {
                    unsafeAtomicAdd(&acc[(size_t)s_ring[(head + (uint32_t)e) & (RING - 1)].x * AS + acc_slot<K>(qv, K)], a);
                    s_acc[c] = 0.0f;
                }
            }
        }
    }
    if (evalcount) store_work_counts(evalcount, s_ev, 0u, nfull, nsumT, nwave);
}

// ------------------------------------------------------------- launchers ---


#define CS_DISPATCH_K(K, ...)                                                                                      \
    switch (K) {                                                                                                   \
    case 3: { constexpr int KK = 3; __VA_ARGS__; } break;                                                          \
    case 4: { constexpr int KK = 4; __VA_ARGS__; } break;                                                          \
    case 5: { constexpr int KK = 5; __VA_ARGS__; } break;                                                          \
    case 6: { constexpr int KK = 6; __VA_ARGS__; } break;                                                          \
    case 7: { constexpr int KK = 7; __VA_ARGS__; } break;                                                          \
    case 8: { constexpr int KK = 8; __VA_ARGS__; } break;                                                          \
    default: break;                                                                                                \
    }

#define CS_DISPATCH_TILE(TILEV, ...)                                                                               \
    switch (TILEV) {                                                                                               \
    case 8: { constexpr int TT = 8, BF = 32, BBW = 32; __VA_ARGS__; } break;                                       \
    case 16: { constexpr int TT = 16, BF = 64, BBW = 64; __VA_ARGS__; } break;                                     \
    case 32: { constexpr int TT = 32, BF = 64, BBW = 64; __VA_ARGS__; } break;                                     \
    default: break;                                                                                                \
    }

namespace {
// Resident workgroups of a kernel on the whole device, cached per kernel.
template <class F> int persistent_grid(F kernel, int threads)
{
    static std::mutex mu;
    static std::unordered_map<const void *, int> cache;
    std::lock_guard<std::mutex> lock(mu);
    const void *key = reinterpret_cast<const void *>(kernel);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int dev = 0, cus = 0, per = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, 0);
    const int g = std::max(1, cus) * std::max(1, per);
    cache[key] = g;
    return g;
}
int split_grid(int resident, uint32_t max_items, int tile)
{
    const uint64_t squares = (uint64_t)max_items * (uint64_t)(tile / 8) * (uint64_t)(tile / 8);
    return (int)std::min<uint64_t>({(uint64_t)resident, squares, (uint64_t)EVAL_SLOTS});
}
} // namespace

// max_items bounds the grid (a persistent grid larger than the work only idles);
// split: by squares with the records split over wavefronts.  Returns the grid
// size (the number of evalcount slots written).
int launch_render_fwd(hipStream_t st, int K, int tile, const FrameHeader *frame, const uint32_t *order,
                      uint32_t max_items, uint32_t *queues, const uint2 *ranges, const uint32_t *keys,
                      const uint32_t *ids, const uint8_t *records, const RenderArgs &ra, uint2 *pixstate,
                      unsigned long long *evalcount, float *zero_acc, size_t zero_floats, bool split)
{
    // the accumulator rows are whole 16-byte words (acc_stride is a multiple of 4)
    u32x4 *z4 = reinterpret_cast<u32x4 *>(zero_acc);
    const uint32_t n4 = zero_acc ? (uint32_t)(zero_floats / 4) : 0u;
    if (max_items == 0) return 0;
    int used = 0;
    if (split) {
        CS_DISPATCH_K(K, {
            auto kern = render_fwd_split_kernel<KK>;
            used = split_grid(persistent_grid(kern, 256), max_items, tile);
            hipLaunchKernelGGL(kern, dim3(used), dim3(256), 0, st, frame, order, queues, ranges, keys, ids, records, ra,
                               pixstate, evalcount, z4, n4);
        });
    } else {
        CS_DISPATCH_K(K, CS_DISPATCH_TILE(tile, {
            auto kern = render_fwd_kernel<KK, TT, BF>;
            used = std::min({persistent_grid(kern, TT * TT), (int)max_items, EVAL_SLOTS});
            hipLaunchKernelGGL(kern, dim3(used), dim3(TT * TT), 0, st, frame, order, queues, ranges, keys, ids, records, ra,
                               pixstate, evalcount, z4, n4);
        }));
    }
    return used;
}

int launch_render_bwd(hipStream_t st, int K, int tile, const FrameHeader *frame, const uint32_t *order,
                      uint32_t max_items, uint32_t *queues, const uint2 *ranges, const uint32_t *keys,
                      const uint32_t *ids, const uint8_t *records, const RenderArgs &ra, const uint2 *pixstate, float *acc,
                      unsigned long long *evalcount, bool split)
{
    if (max_items == 0) return 0;
    int used = 0;
    if (split) {
        CS_DISPATCH_K(K, {
            auto kern = render_bwd_split_kernel<KK>;
            used = split_grid(persistent_grid(kern, 256), max_items, tile);
            hipLaunchKernelGGL(kern, dim3(used), dim3(256), 0, st, frame, order, queues, ranges, keys, ids, records, ra,
                               pixstate, acc, evalcount);
        });
    } else {
        CS_DISPATCH_K(K, CS_DISPATCH_TILE(tile, {
            auto kern = render_bwd_kernel<KK, TT, BBW>;
            used = std::min({persistent_grid(kern, TT * TT), (int)max_items, EVAL_SLOTS});
            hipLaunchKernelGGL(kern, dim3(used), dim3(TT * TT), 0, st, frame, order, queues, ranges, keys, ids, records, ra,
                               pixstate, acc, evalcount);
        }));
    }
    return used;
}

// ------------------------------------------------------------ L1 loss ----

// block_sum (nullable): each block stores its sum of |rgb - target| in its
// own slot (same-address atomics from every block would serialise)
__global__ __launch_bounds__(256) void l1_grad_kernel(const float *__restrict__ rgb, const float *__restrict__ target,
                                                      size_t n, float scale, float *__restrict__ grad,
                                                      float *__restrict__ block_sum)
{
    __shared__ float s_w[4];
    float part = 0.0f;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const float d = rgb[i] - target[i];
        grad[i] = d > 0.0f ? scale : (d < 0.0f ? -scale : 0.0f);
        part += fabsf(d);
    }
    if (block_sum) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
        if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = part;
        __syncthreads();
        if (threadIdx.x == 0) block_sum[blockIdx.x] = (s_w[0] + s_w[1]) + (s_w[2] + s_w[3]);
    }
}

// *loss += scale * (sum of the nb block sums): one workgroup
__global__ __launch_bounds__(1024) void sum_slots_kernel(const float *__restrict__ slots, int nb, float scale,
                                                         float *__restrict__ loss)
{
    __shared__ float s_w[16];
    float t = 0.0f;
    for (int b = threadIdx.x; b < nb; b += 1024) t += slots[b];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        float u = 0.0f;
        for (int w = 0; w < 16; ++w) u += s_w[w];
        *loss += u * scale;
    }
}

// Returns hipSuccess, or the error of the scratch allocation (loss only).
hipError_t launch_l1_grad(hipStream_t st, const float *rgb, const float *target, size_t n, float *grad, float *loss)
{
    if (n == 0) return hipSuccess;
    const size_t blocks = std::min<size_t>((n + 255) / 256, 2048);
    float *slots = nullptr;
    if (loss) {
        const hipError_t e = hipMallocAsync((void **)&slots, blocks * sizeof(float), st);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(l1_grad_kernel, dim3((unsigned)blocks), dim3(256), 0, st, rgb, target, n, 1.0f / (float)n,
                       grad, slots);
    if (loss) {
        hipLaunchKernelGGL(sum_slots_kernel, dim3(1), dim3(1024), 0, st, slots, (int)blocks, 1.0f / (float)n, loss);
        (void)hipFreeAsync(slots, st);
    }
    return hipSuccess;
}

} // namespace cs
