// Initial convex set from a point cloud (gfx950), paper Sec. 3.3
// "Initialization and losses" and Supp. Initialization & Hyperparameters: one
// convex per cloud point, its K points spread uniformly over a sphere round
// the cloud point (Fibonacci sphere), the sphere's radius a multiple of the
// mean distance to the point's three nearest neighbours in the cloud.
//
// The three nearest neighbours are exact.  Small clouds are searched by brute
// force (every thread keeps its three smallest squared distances over all
// points).  Larger ones are sorted along a Morton curve and cut into leaves of
// 16 consecutive points, 64 leaves to a node, each with its bounding box; a
// wavefront takes a leaf's 16 points as queries, starts with the leaves beside
// it on the curve and then visits every leaf whose box is nearer than the
// farthest third neighbour it still has.  A box's distance is computed with the
// operations of a point's (subtract, square, add, each rounded monotonically),
// so it never exceeds the computed distance of a point inside: pruning drops no
// neighbour, and the three distances are the brute-force search's bit for bit.
// Should the sort report that one of its bounded waits ran out, the points keep the
// cloud's order: the search is exact in any order, only slower.
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.hpp"
#include "convexsplat.h"
#include "runtime.hpp"
#include "sh.hpp"

namespace cs {
bool radix_sort(hipStream_t, uint32_t **, uint32_t **, uint32_t **, uint32_t **, uint32_t, const uint32_t *, uint32_t, int,
                uint32_t *, int, uint32_t *, bool, uint2 *, uint32_t);
size_t sort_temp_words(uint32_t, int, int);
size_t radix_sort_words(uint32_t, bool, uint32_t, int, int);

namespace {

constexpr int KN_BLOCK = 256;
// Clouds up to this size are searched by brute force, whose time grows with n
// (60 us at 500 points, 103 us at 1000, the whole call); the curve's dozen
// launches take 80 us there and 86 us at 1500 points.
constexpr int BRUTE_MAX = 768;

struct InitArgs {
    int n, K, nsh;
    float radius_scale, radius_min;
    float delta0, sigma0, opacity0;
    float dir[3 * CS_MAX_K]; // unit Fibonacci-sphere directions
};

__global__ __launch_bounds__(KN_BLOCK) void knn3_mean_kernel(int n, const float *__restrict__ xyz,
                                                             float *__restrict__ mean_dist)
{
    __shared__ float s_p[3 * KN_BLOCK];
    const int i = blockIdx.x * KN_BLOCK + threadIdx.x;
    const float qx = i < n ? xyz[3 * i] : 0.0f, qy = i < n ? xyz[3 * i + 1] : 0.0f, qz = i < n ? xyz[3 * i + 2] : 0.0f;
    float d0 = INFINITY, d1 = INFINITY, d2 = INFINITY; // ascending
    for (int base = 0; base < n; base += KN_BLOCK) {
        const int cnt = min(KN_BLOCK, n - base);
        __syncthreads();
        for (int j = threadIdx.x; j < 3 * cnt; j += KN_BLOCK) s_p[j] = xyz[3 * (size_t)base + j];
        __syncthreads();
        for (int c = 0; c < cnt; ++c) {
            const float dx = s_p[3 * c] - qx, dy = s_p[3 * c + 1] - qy, dz = s_p[3 * c + 2] - qz;
            const float d = (dx * dx + dy * dy) + dz * dz;
            const bool self = base + c == i;
            if (!self && d < d2) {
                if (d < d1) {
                    d2 = d1;
                    if (d < d0) { d1 = d0; d0 = d; }
                    else d1 = d;
                } else {
                    d2 = d;
                }
            }
        }
    }
    if (i >= n) return;
    // fewer than three other points: the mean of those there are
    float sum = 0.0f;
    int m = 0;
    if (d0 < INFINITY) { sum += sqrtf(d0); ++m; }
    if (d1 < INFINITY) { sum += sqrtf(d1); ++m; }
    if (d2 < INFINITY) { sum += sqrtf(d2); ++m; }
    mean_dist[i] = m ? sum / (float)m : 0.0f;
}

// ------------------------------------------------- search along a curve ----

constexpr int LEAF = 16;  // points of a leaf
constexpr int NODE = 64;  // leaves of a node: one per lane
constexpr int CURVE_SAMPLES = 1024;
constexpr uint32_t KEY_NOT_FINITE = 1u << 30; // behind every 30-bit Morton key

__device__ __forceinline__ bool finite3(float x, float y, float z)
{
    return fabsf(x) < INFINITY && fabsf(y) < INFINITY && fabsf(z) < INFINITY;
}

// The curve's cube from a sample of the cloud: mean -+ 3 sigma per axis over the
// samples within 3 sigma of the last estimate, so that a few far points (usual
// in structure-from-motion clouds) do not stretch it; points outside fall into
// its border cells.  cube[0..2] low corner, cube[3..5] cells per length.  One
// workgroup; it also sets the sort's error word to err0.
__global__ __launch_bounds__(CURVE_SAMPLES) void curve_cube_kernel(int n, const float *__restrict__ xyz,
                                                                   float *__restrict__ cube, uint32_t *__restrict__ err,
                                                                   uint32_t err0)
{
    __shared__ float s_sum[CURVE_SAMPLES / 64][7], s_tot[7];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (t == 0) *err = err0;
    const size_t i = (size_t)t * (size_t)n / CURVE_SAMPLES;
    const float x = xyz[3 * i], y = xyz[3 * i + 1], z = xyz[3 * i + 2];
    const bool ok = finite3(x, y, z);
    const float p[3] = {x, y, z};
    float lo[3] = {-INFINITY, -INFINITY, -INFINITY}, hi[3] = {INFINITY, INFINITY, INFINITY};
    // deviations from the last mean (first: from a sample), so that coordinates
    // far from the origin lose no digits
    __shared__ float s_ref[3];
    if (t < 3) s_ref[t] = fabsf(xyz[t]) < INFINITY ? xyz[t] : 0.0f;
    __syncthreads();
    float ref[3] = {s_ref[0], s_ref[1], s_ref[2]};
    for (int round = 0; round < 4; ++round) {
        bool in = ok;
        for (int d = 0; d < 3; ++d) in = in && p[d] >= lo[d] && p[d] <= hi[d];
        float v[7];
        for (int d = 0; d < 3; ++d) {
            const float dev = p[d] - ref[d];
            v[d] = in ? dev : 0.0f;
            v[3 + d] = in ? dev * dev : 0.0f;
        }
        v[6] = in ? 1.0f : 0.0f;
#pragma unroll
        for (int q = 0; q < 7; ++q) {
            for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o, 64);
            if (lane == 0) s_sum[wave][q] = v[q];
        }
        __syncthreads();
        if (t < 7) {
            float a = 0.0f;
            for (int w = 0; w < CURVE_SAMPLES / 64; ++w) a += s_sum[w][t];
            s_tot[t] = a;
        }
        __syncthreads();
        float tot[7];
        for (int q = 0; q < 7; ++q) tot[q] = s_tot[q];
        for (int d = 0; d < 3; ++d) {
            const float m = tot[d] / fmaxf(tot[6], 1.0f), var = tot[3 + d] / fmaxf(tot[6], 1.0f) - m * m;
            const float sd = sqrtf(fmaxf(var, 0.0f));
            ref[d] += m;
            lo[d] = ref[d] - 3.0f * sd;
            hi[d] = ref[d] + 3.0f * sd;
        }
    }
    if (t < 3) {
        const float w = hi[t] - lo[t];
        cube[t] = lo[t];
        cube[3 + t] = w > 0.0f && w < INFINITY ? 1024.0f / w : 0.0f;
    }
}

// Bits 0-9 of v spread to every third bit.
__device__ __forceinline__ uint32_t spread3(uint32_t v)
{
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    return (v | (v << 2)) & 0x09249249u;
}

__global__ __launch_bounds__(KN_BLOCK) void morton_kernel(int n, const float *__restrict__ xyz,
                                                          const float *__restrict__ cube, uint32_t *__restrict__ keys,
                                                          uint32_t *__restrict__ ids, ZeroSpans zero)
{
    zero_share(zero); // the sort's temporaries
    const int i = blockIdx.x * KN_BLOCK + threadIdx.x;
    if (i >= n) return;
    const float p[3] = {xyz[3 * (size_t)i], xyz[3 * (size_t)i + 1], xyz[3 * (size_t)i + 2]};
    uint32_t key = KEY_NOT_FINITE;
    if (finite3(p[0], p[1], p[2])) {
        key = 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) { // (fmaxf drops a NaN of an unusable cube)
            const float c = fminf(fmaxf((p[d] - cube[d]) * cube[3 + d], 0.0f), 1023.0f);
            key |= spread3((uint32_t)c) << d;
        }
    }
    keys[i] = key;
    ids[i] = (uint32_t)i;
}

// Boxes: two float4 (low corner, high corner); of no finite point: +inf, -inf.
// Reduced over groups of G lanes, stored by the first of each.
template <int G> __device__ __forceinline__ void store_box(float4 *box, float3 lo, float3 hi)
{
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) {
        lo.x = fminf(lo.x, __shfl_xor(lo.x, o, 64)); hi.x = fmaxf(hi.x, __shfl_xor(hi.x, o, 64));
        lo.y = fminf(lo.y, __shfl_xor(lo.y, o, 64)); hi.y = fmaxf(hi.y, __shfl_xor(hi.y, o, 64));
        lo.z = fminf(lo.z, __shfl_xor(lo.z, o, 64)); hi.z = fmaxf(hi.z, __shfl_xor(hi.z, o, 64));
    }
    if ((threadIdx.x & (G - 1)) == 0) {
        box[0] = make_float4(lo.x, lo.y, lo.z, 0.0f);
        box[1] = make_float4(hi.x, hi.y, hi.z, 0.0f);
    }
}

// The points in curve order (w: the cloud index; places past n are not a
// number) and the leaves' boxes: 16 lanes per leaf.  *err nonzero (the sort
// failed: ids may name a point twice and another not at all): in the cloud's order.
__global__ __launch_bounds__(KN_BLOCK) void leaf_kernel(int n, int nleaves, const float *__restrict__ xyz,
                                                        const uint32_t *__restrict__ ids, const uint32_t *__restrict__ err,
                                                        float4 *__restrict__ pts, float4 *__restrict__ boxes)
{
    const size_t r = (size_t)blockIdx.x * KN_BLOCK + threadIdx.x;
    const size_t leaf = r / LEAF;
    if (leaf >= (size_t)nleaves) return; // whole groups of LEAF lanes
    float4 p = make_float4(NAN, NAN, NAN, 0.0f);
    if (r < (size_t)n) {
        const uint32_t i = *err ? (uint32_t)r : min(ids[r], (uint32_t)n - 1u);
        p = make_float4(xyz[3 * (size_t)i], xyz[3 * (size_t)i + 1], xyz[3 * (size_t)i + 2], __uint_as_float(i));
    }
    pts[r] = p;
    const bool ok = finite3(p.x, p.y, p.z);
    const float I = INFINITY;
    store_box<LEAF>(boxes + 2 * leaf, ok ? make_float3(p.x, p.y, p.z) : make_float3(I, I, I),
                    ok ? make_float3(p.x, p.y, p.z) : make_float3(-I, -I, -I));
}

// The nodes' boxes: one wavefront per node of 64 leaves.
__global__ __launch_bounds__(NODE) void node_kernel(int nleaves, const float4 *__restrict__ boxes,
                                                    float4 *__restrict__ nodes)
{
    const int leaf = blockIdx.x * NODE + threadIdx.x;
    const float I = INFINITY;
    float4 lo = make_float4(I, I, I, 0.0f), hi = make_float4(-I, -I, -I, 0.0f);
    if (leaf < nleaves) {
        lo = boxes[2 * (size_t)leaf];
        hi = boxes[2 * (size_t)leaf + 1];
    }
    store_box<NODE>(nodes + 2 * (size_t)blockIdx.x, make_float3(lo.x, lo.y, lo.z), make_float3(hi.x, hi.y, hi.z));
}

// Squared distance of [alo, ahi] and the box b (0 where they overlap).
__device__ __forceinline__ float box_gap2(float3 alo, float3 ahi, float4 blo, float4 bhi)
{
    const float gx = fmaxf(fmaxf(blo.x - ahi.x, alo.x - bhi.x), 0.0f);
    const float gy = fmaxf(fmaxf(blo.y - ahi.y, alo.y - bhi.y), 0.0f);
    const float gz = fmaxf(fmaxf(blo.z - ahi.z, alo.z - bhi.z), 0.0f);
    return (gx * gx + gy * gy) + gz * gz;
}

// One wavefront per leaf: its 16 points are the queries, held by each of the
// wavefront's four groups of 16 lanes, and the groups scan four leaves at a
// time; a query's bound is the least of its four lanes' third distances, and
// their neighbours are merged at the end.  Bound by VALU issue (about 13
// instructions per query and candidate) and by how few leaves are visited: 100k
// points take 7.83 ms by brute force, 0.31 ms with 64 queries and 64-point
// leaves, 1.71 ms with leaves chosen by the 16 points' box alone, 0.11 ms here.
__global__ __launch_bounds__(KN_BLOCK) void knn3_curve_kernel(int nleaves, int nnodes, const float4 *__restrict__ pts,
                                                              const float4 *__restrict__ boxes,
                                                              const float4 *__restrict__ nodes, int n,
                                                              float *__restrict__ mean_dist)
{
    const int leaf = __builtin_amdgcn_readfirstlane((int)((blockIdx.x * KN_BLOCK + threadIdx.x) >> 6));
    if (leaf >= nleaves) return;
    const int lane = threadIdx.x & 63, ql = lane & (LEAF - 1), group = lane / LEAF;
    const float4 q = pts[(size_t)leaf * LEAF + ql];
    const bool active = finite3(q.x, q.y, q.z);
    const float4 l4 = boxes[2 * (size_t)leaf], h4 = boxes[2 * (size_t)leaf + 1];
    const float3 glo = make_float3(l4.x, l4.y, l4.z), ghi = make_float3(h4.x, h4.y, h4.z);
    float d0 = INFINITY, d1 = INFINITY, d2 = INFINITY; // this lane's, ascending
    float bound = INFINITY; // the query's (not active: below 0), and the largest of the 16
    float gmax = INFINITY;
    auto insert = [&](float d) {
        d2 = __builtin_amdgcn_fmed3f(d1, d2, d);
        d1 = __builtin_amdgcn_fmed3f(d0, d1, d);
        d0 = fminf(d0, d);
    };
    // each group scans its leaf l (none: l < 0)
    auto scan = [&](int l) {
        const float4 *__restrict__ c = pts + (size_t)max(l, 0) * LEAF;
        const bool own = l == leaf;
#pragma unroll 8
        for (int j = 0; j < LEAF; ++j) {
            const float4 p = c[j];
            const float dx = p.x - q.x, dy = p.y - q.y, dz = p.z - q.z;
            const float e = (dx * dx + dy * dy) + dz * dz;
            insert(e < INFINITY && l >= 0 && !(own && j == ql) ? e : INFINITY); // not a number: no neighbour
        }
        bound = fminf(d2, __shfl_xor(d2, 16, 64));
        bound = fminf(bound, __shfl_xor(bound, 32, 64));
        bound = active ? bound : -1.0f;
        float m = bound;
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        gmax = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(m)));
    };
    {
        const int l = leaf - 1 + group;
        scan(l < nleaves ? l : -1); // (l = -1 before the first leaf)
    }
    // whether the lane's box holds a point that some query may need: the 16
    // points' leaf may span a jump of the curve, so its box alone says little
    auto needed = [&](float4 blo, float4 bhi) {
        bool any = false;
#pragma unroll
        for (int i = 0; i < LEAF; ++i) {
            auto of = [&](float v) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), i)); };
            const float3 p = make_float3(of(q.x), of(q.y), of(q.z));
            any = any || box_gap2(p, p, blo, bhi) < of(bound);
        }
        return any;
    };
    for (int nb = 0; nb < nnodes; nb += 64) {
        const int nd = min(nb + lane, nnodes - 1);
        const float4 nlo = nodes[2 * (size_t)nd], nhi = nodes[2 * (size_t)nd + 1];
        uint64_t near = __ballot(nb + lane < nnodes && box_gap2(glo, ghi, nlo, nhi) < gmax);
        if (near) near &= __ballot(needed(nlo, nhi));
        while (near) {
            const int k = __builtin_ctzll(near);
            near &= near - 1;
            const int first = (nb + k) * NODE, lf = first + lane, lc = min(lf, nleaves - 1);
            const float4 blo = boxes[2 * (size_t)lc], bhi = boxes[2 * (size_t)lc + 1];
            const bool todo = lf < nleaves && !(lf >= leaf - 1 && lf <= leaf + 2);
            uint64_t leaves = __ballot(todo && box_gap2(glo, ghi, blo, bhi) < gmax);
            if (leaves) leaves &= __ballot(needed(blo, bhi));
            while (leaves) {
                int mine = -1;
#pragma unroll
                for (int g = 0; g < 64 / LEAF; ++g) {
                    if (leaves == 0) break;
                    const int j = __builtin_ctzll(leaves);
                    leaves &= leaves - 1;
                    if (group == g) mine = first + j;
                }
                scan(mine);
            }
        }
    }
    // the four lanes' neighbours of a query
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {
        const float e0 = __shfl_xor(d0, o, 64), e1 = __shfl_xor(d1, o, 64), e2 = __shfl_xor(d2, o, 64);
        insert(e0);
        insert(e1);
        insert(e2);
    }
    if (group != 0 || (size_t)leaf * LEAF + ql >= (size_t)n) return;
    float sum = 0.0f;
    int m = 0;
    if (active) {
        if (d0 < INFINITY) { sum += sqrtf(d0); ++m; }
        if (d1 < INFINITY) { sum += sqrtf(d1); ++m; }
        if (d2 < INFINITY) { sum += sqrtf(d2); ++m; }
    }
    mean_dist[__float_as_uint(q.w)] = m ? sum / (float)m : 0.0f;
}

// A block's convexes fill contiguous runs of the output rows, so the rows are
// written cooperatively (consecutive threads, consecutive floats): HBM-bound,
// 32.8 -> 11.4 us at 100k convexes, degree 3, against one row per thread.
__global__ __launch_bounds__(KN_BLOCK) void init_convex_kernel(const float *__restrict__ xyz,
                                                               const float *__restrict__ rgb,
                                                               const float *__restrict__ mean_dist, InitArgs a,
                                                               cs_param_set out)
{
    __shared__ float s_c[KN_BLOCK][3], s_f[KN_BLOCK][3], s_r[KN_BLOCK];
    const int base = blockIdx.x * KN_BLOCK, cnt = min(KN_BLOCK, a.n - base), t = threadIdx.x;
    if (t < cnt) {
        const size_t i = (size_t)base + t;
        s_r[t] = a.radius_scale * fmaxf(mean_dist[i], a.radius_min);
        for (int c = 0; c < 3; ++c) {
            s_c[t][c] = xyz[3 * i + c];
            // colour = 0.5 + Y00 f_dc (the renderer's convention): f_dc = (rgb - 0.5) / Y00, higher orders 0
            s_f[t][c] = rgb ? (rgb[3 * i + c] - 0.5f) / SH_C0 : 0.0f;
        }
        out.delta[i] = a.delta0;
        out.sigma[i] = a.sigma0;
        out.opacity[i] = a.opacity0;
    }
    __syncthreads();
    // element j of a run of rows of W values: row and column without a division per element
    auto rows = [&](int W, auto value, float *dst) {
        const int drow = KN_BLOCK / W, dcol = KN_BLOCK - drow * W;
        int row = t / W, col = t - row * W;
        for (int j = t; j < cnt * W; j += KN_BLOCK) {
            dst[j] = value(row, col);
            row += drow;
            col += dcol;
            if (col >= W) { col -= W; ++row; }
        }
    };
    rows(3 * a.K, [&](int r, int e) { return s_c[r][e % 3] + s_r[r] * a.dir[e]; }, out.points + (size_t)base * 3 * a.K);
    rows(a.nsh, [&](int r, int e) { return e < 3 ? s_f[r][e] : 0.0f; }, out.sh + (size_t)base * a.nsh);
}

// The scratch of a neighbour search: the mean distances, and for the search
// along the curve its cube and the sort's error word, keys and indices (with the
// sort's second pair and temporaries), the sorted points and the boxes.
struct NeighbourScratch {
    size_t bytes = 0, md = 0, cube = 0, pair[4] = {}, temp = 0, pts = 0, box = 0, node = 0;
    explicit NeighbourScratch(int n)
    {
        const size_t N = (size_t)n, nleaves = (N + LEAF - 1) / LEAF, nnodes = (nleaves + NODE - 1) / NODE;
        auto carve = [&](size_t b) {
            const size_t at = bytes;
            bytes = (bytes + b + 255) & ~(size_t)255;
            return at;
        };
        md = carve(4 * N);
        if (n <= BRUTE_MAX) return;
        cube = carve(64);
        for (size_t &o : pair) o = carve(4 * N);
        temp = carve(4 * sort_temp_words((uint32_t)n, 31, 8));
        pts = carve(16 * LEAF * nleaves);
        box = carve(32 * nleaves);
        node = carve(32 * nnodes);
    }
};

} // namespace

size_t neighbour_scratch_bytes(int n) { return NeighbourScratch(n).bytes; }

// Mean distance of every point to its three nearest others, at the start of the
// scratch (neighbour_scratch_bytes).  err0: what the sort's error word starts
// from; 0 but where a test has the search go without the sort.
void launch_neighbour_means(hipStream_t st, int n, const float *xyz, uint8_t *scr, uint32_t err0)
{
    const NeighbourScratch o(n);
    const dim3 grid((n + KN_BLOCK - 1) / KN_BLOCK), block(KN_BLOCK);
    float *md = reinterpret_cast<float *>(scr + o.md);
    if (n <= BRUTE_MAX) {
        hipLaunchKernelGGL(knn3_mean_kernel, grid, block, 0, st, n, xyz, md);
        return;
    }
    const size_t nleaves = ((size_t)n + LEAF - 1) / LEAF, nnodes = (nleaves + NODE - 1) / NODE;
    float *cube = reinterpret_cast<float *>(scr + o.cube);
    uint32_t *err = reinterpret_cast<uint32_t *>(cube) + 8;
    uint32_t *keys = reinterpret_cast<uint32_t *>(scr + o.pair[0]), *ids = reinterpret_cast<uint32_t *>(scr + o.pair[1]);
    uint32_t *keys2 = reinterpret_cast<uint32_t *>(scr + o.pair[2]), *ids2 = reinterpret_cast<uint32_t *>(scr + o.pair[3]);
    float4 *pts = reinterpret_cast<float4 *>(scr + o.pts), *boxes = reinterpret_cast<float4 *>(scr + o.box);
    float4 *nodes = reinterpret_cast<float4 *>(scr + o.node);
    hipLaunchKernelGGL(curve_cube_kernel, dim3(1), dim3(CURVE_SAMPLES), 0, st, n, xyz, cube, err, err0);
    uint32_t *temp = reinterpret_cast<uint32_t *>(scr + o.temp);
    const ZeroSpans z{{temp}, {(uint32_t)radix_sort_words((uint32_t)n, false, (uint32_t)n, 31, 8)}};
    hipLaunchKernelGGL(morton_kernel, grid, block, 0, st, n, xyz, cube, keys, ids, z);
    radix_sort(st, &keys, &ids, &keys2, &ids2, (uint32_t)n, nullptr, (uint32_t)n, 31, temp, 8, err, true, nullptr, 0);
    const dim3 lgrid((unsigned)((nleaves * LEAF + KN_BLOCK - 1) / KN_BLOCK));
    hipLaunchKernelGGL(leaf_kernel, lgrid, block, 0, st, n, (int)nleaves, xyz, ids, err, pts, boxes);
    hipLaunchKernelGGL(node_kernel, dim3((unsigned)nnodes), dim3(NODE), 0, st, (int)nleaves, boxes, nodes);
    hipLaunchKernelGGL(knn3_curve_kernel, dim3((unsigned)((nleaves * 64 + KN_BLOCK - 1) / KN_BLOCK)), block, 0, st, (int)nleaves,
                       (int)nnodes, pts, boxes, nodes, n, md);
}

} // namespace cs

using namespace cs;

extern "C" {

int cs_init_from_points(cs_ctx *ctx, int32_t n, const float *xyz, const float *rgb, int32_t k, int32_t sh_degree,
                        const cs_init_params *prm, const cs_param_set *out, void *hip_stream)
{
    if (!ctx) return fail(CS_EINVAL, "ctx is NULL");
    if (n < 0 || k < 3 || k > CS_MAX_K || sh_degree < 0 || sh_degree > CS_MAX_SH_DEGREE)
        return fail(CS_EINVAL, "bad n, k or sh_degree");
    if (!prm) return fail(CS_EINVAL, "params is NULL");
    if (n == 0) return CS_OK;
    if (!xyz || !out || !out->points || !out->delta || !out->sigma || !out->opacity || !out->sh)
        return fail(CS_EINVAL, "array pointer is NULL");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(CS_EHIP, "hipSetDevice failed");
    hipStream_t st = (hipStream_t)hip_stream;
    InitArgs a;
    a.n = n;
    a.K = k;
    a.nsh = 3 * (sh_degree + 1) * (sh_degree + 1);
    a.radius_scale = prm->radius_scale;
    a.radius_min = prm->radius_min;
    a.delta0 = prm->delta0;
    a.sigma0 = prm->sigma0;
    a.opacity0 = prm->opacity0;
    // Fibonacci sphere: heights 1 - (2j + 1) / K, azimuth steps of the golden angle
    const double golden = M_PI * (3.0 - std::sqrt(5.0));
    for (int j = 0; j < k; ++j) {
        const double yv = 1.0 - (2.0 * j + 1.0) / k, rxy = std::sqrt(1.0 - yv * yv), phi = golden * j;
        a.dir[3 * j] = (float)(std::cos(phi) * rxy);
        a.dir[3 * j + 1] = (float)yv;
        a.dir[3 * j + 2] = (float)(std::sin(phi) * rxy);
    }
    uint8_t *scr = nullptr;
    hipError_t e = hipMallocAsync((void **)&scr, neighbour_scratch_bytes(n), st);
    if (e != hipSuccess) return fail(CS_ENOMEM, "init scratch: %s", hipGetErrorString(e));
    launch_neighbour_means(st, n, xyz, scr, 0);
    const float *md = reinterpret_cast<const float *>(scr);
    const dim3 grid((n + KN_BLOCK - 1) / KN_BLOCK), block(KN_BLOCK);
    hipLaunchKernelGGL(init_convex_kernel, grid, block, 0, st, xyz, rgb, md, a, *out);
    e = hipGetLastError();
    (void)hipFreeAsync(scr, st);
    return e == hipSuccess ? CS_OK : fail(CS_EHIP, "init launch: %s", hipGetErrorString(e));
}

} // extern "C"
