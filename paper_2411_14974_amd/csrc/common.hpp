// Shared definitions of the convex rasterizer's HIP kernels (gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace cs {

constexpr int MAXK = 8;
constexpr int WAVE = 64;
constexpr double LOG2E = 1.4426950408889634;
constexpr double LN2 = 0.6931471805599453;
constexpr uint32_t KEY_CULLED = 0xFFFFFFFFu;

// Convex status codes (also reported by the debug dump).
enum : int32_t { ST_VISIBLE = 0, ST_NEAR = 1, ST_HULL = 2, ST_FAINT = 3 };

// Per-convex record read by the compositing kernels: a 64-byte header then
// one 24-byte line (a, b, c as double) per hull edge.  A line evaluates
//   x2 = a*dx + b*dy + c = log2(e) * delta' * L_j(q),   dx = qx - ox, dy = qy - oy,
// so the LogSumExp runs in base 2 on the hardware exp2/log2.
struct RecHeader {
    float ox, oy;     // integer pixel origin of the line coefficients
    float sigma_p;    // sigma' = d * sigma
    float thr2;       // a pair is skipped when max_j x2_j > thr2 (alpha < eps certain)
    float opacity;
    float rgb[3];
    int32_t T;        // number of hull lines
    int32_t id;       // convex index
    uint32_t box_u;   // pixel columns u0 | u1 << 16 (inclusive) where alpha can reach eps
    uint32_t box_v;   // pixel rows    v0 | v1 << 16
};
// the K lines (three doubles each) follow the header; slots past the hull's
// T lines hold the null line (0, 0, NULL_LINE_C): its value is so negative
// that it never sets the maximum, its exponential is 0 and its gradient
// terms vanish, so consumers need no per-slot test against T
constexpr int REC_HEADER = 48;
constexpr double NULL_LINE_C = -1e30;
static_assert(sizeof(RecHeader) == REC_HEADER, "record header is 48 bytes");

__host__ __device__ constexpr int rec_stride(int K) { return (REC_HEADER + 24 * K + 15) & ~15; }
// accumulator slots per convex for the backward pass:
//   a[K] b[K] c[K]  (base-2 line coefficients), sigma', opacity, rgb[3], and
//   sum_j dL/dx2_j * x2_j  (= delta' dL/ddelta', accumulated per pair because
//   the same quantity rebuilt from the line slots cancels badly)
constexpr int acc_values(int K) { return 3 * K + 6; }
__host__ __device__ constexpr int acc_stride(int K) { return (acc_values(K) + 3) & ~3; }

// Camera as the kernels take it (by value).
struct CamArgs {
    int32_t W, H;
    float fx, fy, cx, cy;
    float R[9];
    float t[3];
    float znear;
    double campos[3]; // -R^T t
};

struct RenderArgs {
    float eps_alpha, t_min;
    float bg[3];
    int32_t tile;
};

// One view of a (possibly batched) render, as the kernels read it from device
// memory.  Tiles of all views share one global index space: view v owns
// [tile_off, tile_off + tiles_x * tiles_y); its per-pixel state starts at pix_off;
// its cells, blocks of 2^cell_shift x 2^cell_shift tiles, start at cell_off.
struct ViewDesc {
    CamArgs cam;
    int32_t tiles_x, tiles_y, tile_off, cell_off;
    uint32_t cell_shift, pad;
    int64_t pix_off;
    float *out_rgb;        // [H][W][3]
    const float *dl_drgb;  // [H][W][3], backward only
};

// Header of the device view table; the ViewDesc array follows it.  Kernels
// read the view count and the tile total from here, so a captured graph can be
// replayed with other cameras and resolutions.
//
// Convexes are binned by cell, a block of S x S tiles of a view (S = 1, 2 or 4):
// one (cell, convex) pair carries the mask of the cell's tiles that the convex
// can reach, so one sorted pair stands for up to S^2 (tile, convex) pairs (at
// 1M convexes, 1080p: 2.3 M sorted pairs instead of 8.9 M), and a tile's
// depth-ordered list is its cell's list filtered by the tile's mask bit.  A
// view has the smallest cells of which VIEW_CELLS cover it, at most 4 x 4: a
// small view's convexes are smaller than a few tiles, and large cells would
// only lengthen the lists that its tiles filter (200k convexes at 256 x 256, a
// whole render: 0.42 ms with the 256 tiles as cells, 0.46 ms with 16 cells).
// A pair's sort key holds the cell in its low key_bits bits, the mask above:
// 16 + 16 bits, or 28 + 4 (cells of at most 2 x 2) when a call has more cells.
struct FrameHeader {
    uint32_t nviews, total_tiles;
    int64_t total_pix;
    uint32_t total_cells, key_bits;
    uint32_t pad[10];
};
constexpr uint32_t VIEW_CELLS = 512; // one 9-bit pass sorts a view's pairs
constexpr uint32_t MAX_CELLS_16 = 1u << 16;
constexpr uint32_t MAX_CELL_PAIRS = (1u << 30) - 1u; // (cell, convex) pairs of one call stay below this
static_assert(sizeof(FrameHeader) == 64, "frame header is 64 bytes");

// The view that owns the global tile gt.
__device__ __forceinline__ int find_view(const ViewDesc *__restrict__ views, int nviews, int gt)
{
    int lo = 0, hi = nviews - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].tile_off <= gt) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}
// The global cell of a view's tile (tx, ty).
__host__ __device__ __forceinline__ uint32_t tile_cell(const ViewDesc &vd, uint32_t tx, uint32_t ty)
{
    const uint32_t s = vd.cell_shift;
    return (uint32_t)vd.cell_off + (ty >> s) * (((uint32_t)vd.tiles_x + (1u << s) - 1u) >> s) + (tx >> s);
}
// The key bit of a view's tile (tx, ty) in its cell's pairs.
__host__ __device__ __forceinline__ uint32_t tile_bit(const ViewDesc &vd, uint32_t key_bits, uint32_t tx, uint32_t ty)
{
    const uint32_t s = vd.cell_shift, side = (1u << s) - 1u;
    return 1u << (key_bits + ((ty & side) << s) + (tx & side));
}

constexpr int MAX_VIEWS = 256;
constexpr int NUM_QUEUES = 8; // one work queue per XCD
// Per-workgroup slots of the forward's work counters (tested, full pairs): each
// workgroup of the persistent grid stores its sums in a slot of its own and
// readers add the slots (same-address atomics from every wavefront serialise)
constexpr int EVAL_SLOTS = 16384;
// fields of a slot: pairs tested (pixel in the record's box), pairs past the
// max-line test (full), the sum of the hull size T over the full pairs, and
// wavefront-level record evaluations (some lane full); the backward's slots
// follow the forward's EVAL_SLOTS
enum : int { EV_TESTED = 0, EV_FULL = 1, EV_SUM_T = 2, EV_WAVES = 3, EVAL_FIELDS = 4 };

// Per-instance binning record (16 bytes): the tile rectangle, tx0 | ty0 << 16
// and tx1 | ty1 << 16 (empty when tx0 > tx1; a view has at most 2048 tiles a
// side), the view's cell shift and the number of (cell, convex) pairs in the bits
// between (bin_cells), and 64 bits of kept tiles:
//  - a rectangle of at most 64 tiles: the mask of kept tiles (bit
//    (ty - ty0) * width + (tx - tx0));
//  - a larger one: its rows are grouped into at most BIG_BANDS bands of
//    ceil(th / BIG_BANDS) tile rows and its columns into at most 2^BIG_BITS
//    blocks of ceil(tw / 2^BIG_BITS) tiles; field r (2 BIG_BITS bits) holds
//    band r's kept blocks as the interval bx0 | bx1 << BIG_BITS (empty when
//    bx0 > bx1), and the band keeps every tile of those blocks.

// The cells that hold a kept tile of a rectangle of at most 64 tiles, each by
// one bit: that of the cell's first tile in the rectangle (kept or not).
__host__ __device__ inline uint64_t cell_marks(uint64_t mask, uint32_t tx0, uint32_t ty0, uint32_t tw, uint32_t th, uint32_t s)
{
    if (s == 0) return mask;
    const uint32_t side = 1u << s, first = side - (tx0 & (side - 1u)); // columns of the first cell
    const uint64_t rowmask = tw < 64 ? (1ull << tw) - 1ull : ~0ull;
    const uint64_t starts = ((s == 1 ? 0x5555555555555555ull : 0x1111111111111111ull) << first) & rowmask; // of the others
    uint64_t marks = 0;
    for (uint32_t r = 0, next; r < th; r = next) { // one row of cells: the tile rows r .. next - 1
        next = ((ty0 + r) | (side - 1u)) + 1u - ty0;
        next = next < th ? next : th;
        const uint32_t bits = (next - r) * tw;
        uint64_t row = (mask >> (r * tw)) & (bits < 64 ? (1ull << bits) - 1ull : ~0ull);
        if (next - r > 1) { // (tw <= 32) the columns kept in one of them
            row |= row >> tw;
            row |= (row >> tw) >> tw;
            row &= rowmask;
        }
        uint64_t any = row | (row >> 1);
        if (s > 1) any |= any >> 2;
        marks |= ((any & starts) | ((row & ((1ull << first) - 1ull)) != 0ull ? 1ull : 0ull)) << (r * tw);
    }
    return marks;
}
__host__ __device__ inline uint32_t bin_shift(uint4 b) { return (b.x >> 11) & 3u; }
__host__ __device__ inline uint32_t bin_tx0(uint4 b) { return b.x & 0x7FFu; }
__host__ __device__ inline uint32_t bin_ty0(uint4 b) { return (b.x >> 16) & 0x7FFu; }
__host__ __device__ inline uint32_t bin_tx1(uint4 b) { return b.y & 0x7FFu; }
__host__ __device__ inline uint32_t bin_ty1(uint4 b) { return (b.y >> 16) & 0x7FFu; }
#ifndef CS_BIG_BANDS
#define CS_BIG_BANDS 4
#endif
constexpr int BIG_BANDS = CS_BIG_BANDS;
constexpr int BIG_BITS = 32 / BIG_BANDS;
constexpr uint64_t BIG_FIELD = (1ull << (2 * BIG_BITS)) - 1ull;
constexpr uint64_t big_empty()
{
    uint64_t m = 0;
    for (int r = 0; r < BIG_BANDS; ++r) m |= ((1ull << BIG_BITS) - 1ull) << (2 * BIG_BITS * r);
    return m;
}
constexpr uint64_t BIG_EMPTY = big_empty(); // every band of a large rectangle empty
__host__ __device__ inline int big_bw(int tw) { return (tw + (1 << BIG_BITS) - 1) >> BIG_BITS; }
__host__ __device__ inline int big_bh(int th) { return (th + BIG_BANDS - 1) / BIG_BANDS; }
__host__ __device__ inline uint64_t big_field(int bx0, int bx1, int r)
{
    return ((uint64_t)bx0 | ((uint64_t)bx1 << BIG_BITS)) << (2 * BIG_BITS * r);
}
// Band r of a large rectangle: its first tile row (rectangle-relative) *row0,
// its tile rows *nrow, first kept tile column *col0 and kept columns *ncol
// (both 0 when the band is empty).
__host__ __device__ inline void big_band(uint64_t mask, int tw, int th, int r, int *row0, int *nrow, int *col0,
                                         int *ncol)
{
    const int bw = big_bw(tw), bh = big_bh(th);
    const uint32_t f = (uint32_t)(mask >> (2 * BIG_BITS * r)) & (uint32_t)BIG_FIELD;
    const int bx0 = (int)(f & ((1u << BIG_BITS) - 1u)), bx1 = (int)(f >> BIG_BITS);
    *row0 = r * bh;
    *nrow = th - r * bh < bh ? th - r * bh : bh;
    const int cend = (bx1 + 1) * bw < tw ? (bx1 + 1) * bw : tw;
    *col0 = bx0 * bw;
    *ncol = (bx0 <= bx1 && *nrow > 0) ? cend - bx0 * bw : 0;
    if (*ncol == 0) *nrow = 0;
}
__device__ inline uint32_t bin_count(uint4 b)
{
    const int tx0 = (int)bin_tx0(b), ty0 = (int)bin_ty0(b), tx1 = (int)bin_tx1(b), ty1 = (int)bin_ty1(b);
    if (tx0 > tx1 || ty0 > ty1) return 0u;
    const int tw = tx1 - tx0 + 1, th = ty1 - ty0 + 1;
    const uint64_t mask = (uint64_t)b.z | ((uint64_t)b.w << 32);
    if (tw * th <= 64) return (uint32_t)(__popc(b.z) + __popc(b.w));
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < BIG_BANDS; ++r) {
        int row0, nrow, col0, ncol;
        big_band(mask, tw, th, r, &row0, &nrow, &col0, &ncol);
        c += (uint32_t)(nrow * ncol);
    }
    return c;
}

// Cells from tile t0 to tile t1 of a row or column.
__host__ __device__ inline uint32_t cells_met(int t0, int t1, uint32_t s) { return ((uint32_t)t1 >> s) - ((uint32_t)t0 >> s) + 1u; }
// The block of cells that band r of a larger rectangle meets: its first cell
// and its cells across and down (0 when the band is empty).
struct CellBlock { uint32_t x, y, nx, ny; };
__host__ __device__ inline CellBlock band_cells(uint64_t mask, int tx0, int ty0, int tw, int th, int r, uint32_t s)
{
    int row0, nrow, col0, ncol;
    big_band(mask, tw, th, r, &row0, &nrow, &col0, &ncol);
    const uint32_t x = (uint32_t)(tx0 + col0) >> s, y = (uint32_t)(ty0 + row0) >> s;
    if (ncol == 0) return {x, y, 0u, 0u};
    return {x, y, ((uint32_t)(tx0 + col0 + ncol - 1) >> s) - x + 1u, ((uint32_t)(ty0 + row0 + nrow - 1) >> s) - y + 1u};
}
// (cell, convex) pairs of a rectangle, never more than its (tile, convex) pairs:
//  - of at most 64 tiles: one for every cell that it meets where these are no more
//    than its kept tiles (a cell without any then makes a pair with an empty mask),
//    else one for every cell with a kept tile.  (Only cells with a kept tile
//    for every convex: 3 % fewer pairs, but a step of 1M convexes at 1920 x 1080 takes 916
//    instead of 912 us, of 317k at 979 x 546 419 instead of 416: preprocess and emission
//    tell the cells apart for longer than their pairs would take.)
//  - of more: one for every band that has kept tiles in a cell, with the band's part
//    of the tiles.
__host__ __device__ inline uint32_t rect_cells(int tx0, int ty0, int tx1, int ty1, uint64_t mask, uint32_t s)
{
    if (tx0 > tx1 || ty0 > ty1) return 0u;
    const int tw = tx1 - tx0 + 1, th = ty1 - ty0 + 1;
    if (tw * th <= 64) {
        const uint32_t kept = (uint32_t)__builtin_popcountll(mask), all = cells_met(tx0, tx1, s) * cells_met(ty0, ty1, s);
        if (s == 0 || all <= kept) return s == 0 ? kept : all;
        return (uint32_t)__builtin_popcountll(cell_marks(mask, (uint32_t)tx0, (uint32_t)ty0, (uint32_t)tw, (uint32_t)th, s));
    }
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < BIG_BANDS; ++r) {
        const CellBlock k = band_cells(mask, tx0, ty0, tw, th, r, s);
        c += k.nx * k.ny;
    }
    return c;
}
// The record holds the count in 18 bits (all ones: not held), 3 and 5 in x, 5 and 5 in
// y: counted again by the pair scan, it took that from 31 to 51 us (1M
// convexes, 1920 x 1080).
constexpr uint32_t BIN_CELLS_LATER = (1u << 18) - 1u;
__host__ __device__ inline uint4 make_bin(int tx0, int ty0, int tx1, int ty1, uint64_t mask, uint32_t shift)
{
    const uint32_t n = rect_cells(tx0, ty0, tx1, ty1, mask, shift), c = n < BIN_CELLS_LATER ? n : BIN_CELLS_LATER;
    return make_uint4((uint32_t)tx0 | (shift << 11) | ((c & 7u) << 13) | ((uint32_t)ty0 << 16) | (((c >> 3) & 31u) << 27),
                      (uint32_t)tx1 | (((c >> 8) & 31u) << 11) | ((uint32_t)ty1 << 16) | ((c >> 13) << 27), (uint32_t)mask,
                      (uint32_t)(mask >> 32));
}
__host__ __device__ inline uint32_t bin_cells(uint4 b)
{
    const uint32_t c = ((b.x >> 13) & 7u) | ((b.x >> 27) << 3) | (((b.y >> 11) & 31u) << 8) | ((b.y >> 27) << 13);
    if (c != BIN_CELLS_LATER) return c;
    return rect_cells((int)bin_tx0(b), (int)bin_ty0(b), (int)bin_tx1(b), (int)bin_ty1(b),
                      (uint64_t)b.z | ((uint64_t)b.w << 32), bin_shift(b));
}

// Up to three word ranges that a kernel clears on the side (each block its
// share), in place of clearing launches of their own: the ranges' next users
// run after the kernel in the stream.  `claims` (nullable): also the first word
// of nclaims blocks of QUEUE_STRIDE words (the compositing's claim counters).
constexpr int QUEUE_STRIDE = 1024; // 4 KiB
struct ZeroSpans {
    uint32_t *p[3] = {nullptr, nullptr, nullptr};
    uint32_t n[3] = {0u, 0u, 0u};
    uint32_t *claims = nullptr;
    uint32_t nclaims = 0;
};
__device__ inline void zero_share(const ZeroSpans &z)
{
    const uint32_t nb = gridDim.x * gridDim.y, b = blockIdx.y * gridDim.x + blockIdx.x;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (!z.p[k]) continue;
        const uint32_t per = (z.n[k] + nb - 1) / nb;
        const uint32_t lo = min(b * per, z.n[k]), hi = min(lo + per, z.n[k]);
        for (uint32_t i = lo + threadIdx.x; i < hi; i += blockDim.x) z.p[k][i] = 0u;
    }
    if (z.claims && b == 0 && threadIdx.x < z.nclaims) z.claims[threadIdx.x * QUEUE_STRIDE] = 0u;
}

// Layout of a frame's counter buffer (32-bit words):
//   [0, CNT_WORDS)            counters read back by the host:
//     CNT_SORT_ERR: a radix-sort look-back wait ran out of its bound (never expected)
//     CNT_PAIRS: (cell, convex) pairs; CNT_PAIRS_EFF: those that fit the buffers
//     CNT_TILE_PAIRS: (tile, convex) pairs that they stand for (at most 2^32 - 1)
//     CNT_SCAN_TILE: tile claims of the pair-offset scan
//   [CNT_QUEUE, CNT_QUEUE_B)  the forward compositing's work queues' claim
//                             counters, one per QUEUE_STRIDE words: device-scope
//                             atomics on one memory block serialise, so each
//                             queue's counter sits in a block of its own
//   [CNT_QUEUE_B, CNT_STATUS) the backward compositing's (cleared with the rest
//                             when the forward starts)
//   [CNT_STATUS, ...)         the pair-offset scan's look-back status (u64 per tile)
enum : int { CNT_PAIRS = 0, CNT_PAIRS_EFF = 1, CNT_OVERFLOW = 2, CNT_SORT_ERR = 3, CNT_TILE_PAIRS = 4, CNT_SCAN_TILE = 20, CNT_WORDS = 32 };
constexpr int CNT_QUEUE = CNT_WORDS;
constexpr int QUEUE_WORDS = NUM_QUEUES * QUEUE_STRIDE;
constexpr int CNT_QUEUE_B = CNT_QUEUE + QUEUE_WORDS;
constexpr int CNT_STATUS = CNT_QUEUE_B + QUEUE_WORDS;

// Host-visible debug record (mirrors cs_debug_convex of the public header).
struct DebugConvex {
    int32_t status, T;
    int32_t hull[MAXK];
    uint32_t depth_key;
    int32_t clampmask;
    double A[MAXK], B[MAXK], C[MAXK];
    double d, delta_p, sigma_p;
    float rgb[3];
    int32_t tile_rect[4];
};

} // namespace cs
