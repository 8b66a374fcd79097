// Training-step kernels around the rasterizer (gfx950), paper Sec. 3.3
// "Initialization and losses":
//
// * the photometric loss L = (1 - lambda) L1 + lambda (1 - SSIM) and its
//   gradient with respect to the rendered image, in one pass down strips of
//   columns: the rows' moments x, y, (x - y)^2 and xy are blurred with the
//   11x11 Gaussian window (separably, zero padding), each row of blurred
//   moments gives the SSIM map and its partial derivatives with respect to
//   them, and the partials' rows are blurred in turn (the window is symmetric:
//   the same blur is its adjoint) and combined with x and y into dL/dx; small
//   and narrow images take the two blurs as two passes over tiles, with the
//   partials in memory between them;
// * the fused Adam step on the raw parameters with their activations
//   (sigmoid opacity, exponential delta and sigma): one launch for all arrays,
//   four elements per thread; an element reads raw, m, v and dL/d(activated)
//   (16 B) and writes raw, m, v and the new activated value (16 B).
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "convexsplat.h"
#include "runtime.hpp"

namespace cs {

namespace {

// ------------------------------------------------------- L1 + D-SSIM ----

constexpr int SS_R = 5;                     // window radius
constexpr int SS_N = 2 * SS_R + 1;          // taps
constexpr float SS_C1 = 0.01f * 0.01f;      // SSIM constants for values in [0, 1]
constexpr float SS_C2 = 0.03f * 0.03f;

struct SsimArgs {
    int W, W3, H;     // pixels and floats per row (three interleaved channels), rows
    int rows;         // output rows of a workgroup
    float lambda;
    float inv_n;      // 1 / (3 W H): the means run over pixels and channels
    float g[SS_N];    // normalised Gaussian window, sigma 1.5
};

// ---- two passes over tiles, with the partials of every pixel in memory between
//      them: small and narrow images (ssim_by_tiles)

constexpr int SS_TILE = 16;                 // output pixels per side of a workgroup
constexpr int SS_IN = SS_TILE + 2 * SS_R;   // input rows / columns with the halo

// Pass 1: per pixel and channel the SSIM value S and its partial derivatives
// with respect to the blurred moments mu_x, E[x^2] and E[xy] (mu_y and E[y^2]
// do not depend on the rendered image); the loss terms are summed into *loss.
__global__ __launch_bounds__(SS_TILE * SS_TILE) void ssim_moments_kernel(const float *__restrict__ x,
                                                                         const float *__restrict__ y, SsimArgs a,
                                                                         float *__restrict__ part,
                                                                         float *__restrict__ block_loss)
{
    constexpr int NM = 15; // per channel: x, y, x^2, y^2, xy
    __shared__ float s_in[SS_IN * SS_IN * 6];
    __shared__ float s_h[SS_IN * SS_TILE * NM];
    const int tx0 = blockIdx.x * SS_TILE - SS_R, ty0 = blockIdx.y * SS_TILE - SS_R;
    {
        // the halo tile: every load of a thread issued before its LDS stores
        constexpr int NIN = SS_IN * SS_IN, PER = (NIN + SS_TILE * SS_TILE - 1) / (SS_TILE * SS_TILE);
        float xv[PER][3], yv[PER][3];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int j = threadIdx.x + k * SS_TILE * SS_TILE;
            const int r = j / SS_IN, c = j - r * SS_IN, u = tx0 + c, v = ty0 + r;
            const bool in = j < NIN && u >= 0 && u < a.W && v >= 0 && v < a.H;
            const size_t p = in ? 3 * ((size_t)v * a.W + u) : 0; // unconditional loads, zeroed after
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                const float xl = x[p + ch], yl = y[p + ch];
                xv[k][ch] = in ? xl : 0.0f;
                yv[k][ch] = in ? yl : 0.0f;
            }
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int j = threadIdx.x + k * SS_TILE * SS_TILE;
            if (j < NIN)
#pragma unroll
                for (int ch = 0; ch < 3; ++ch) {
                    s_in[j * 6 + ch] = xv[k][ch];
                    s_in[j * 6 + 3 + ch] = yv[k][ch];
                }
        }
    }
    __syncthreads();
    // horizontal pass: rows of the halo, the tile's columns
    for (int j = threadIdx.x; j < SS_IN * SS_TILE; j += SS_TILE * SS_TILE) {
        const int r = j / SS_TILE, c = j - r * SS_TILE;
        float acc[NM];
#pragma unroll
        for (int q = 0; q < NM; ++q) acc[q] = 0.0f;
#pragma unroll
        for (int t = 0; t <= 2 * SS_R; ++t) {
            const float *e = &s_in[(r * SS_IN + c + t) * 6];
            const float w = a.g[t];
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                const float xv = e[ch], yv = e[3 + ch];
                acc[5 * ch] = fmaf(w, xv, acc[5 * ch]);
                acc[5 * ch + 1] = fmaf(w, yv, acc[5 * ch + 1]);
                acc[5 * ch + 2] = fmaf(w, xv * xv, acc[5 * ch + 2]);
                acc[5 * ch + 3] = fmaf(w, yv * yv, acc[5 * ch + 3]);
                acc[5 * ch + 4] = fmaf(w, xv * yv, acc[5 * ch + 4]);
            }
        }
#pragma unroll
        for (int q = 0; q < NM; ++q) s_h[j * NM + q] = acc[q];
    }
    __syncthreads();
    const int cx = threadIdx.x % SS_TILE, cy = threadIdx.x / SS_TILE;
    const int u = blockIdx.x * SS_TILE + cx, v = blockIdx.y * SS_TILE + cy;
    float contrib = 0.0f;
    if (u < a.W && v < a.H) {
        float m[NM];
#pragma unroll
        for (int q = 0; q < NM; ++q) m[q] = 0.0f;
#pragma unroll
        for (int t = 0; t <= 2 * SS_R; ++t) {
            const float *e = &s_h[((cy + t) * SS_TILE + cx) * NM];
            const float w = a.g[t];
#pragma unroll
            for (int q = 0; q < NM; ++q) m[q] = fmaf(w, e[q], m[q]);
        }
        const size_t p = 3 * ((size_t)v * a.W + u);
        const float *xin = &s_in[((cy + SS_R) * SS_IN + cx + SS_R) * 6];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            const float mx = m[5 * ch], my = m[5 * ch + 1];
            const float sxx = m[5 * ch + 2] - mx * mx, syy = m[5 * ch + 3] - my * my, sxy = m[5 * ch + 4] - mx * my;
            const float A1 = 2.0f * mx * my + SS_C1, A2 = 2.0f * sxy + SS_C2;
            const float B1 = mx * mx + my * my + SS_C1, B2 = sxx + syy + SS_C2;
            const float S = (A1 * A2) / (B1 * B2);
            // dS/dmu_x, dS/dE[x^2], dS/dE[xy]
            part[3 * p + 3 * ch] = S * (2.0f * my / A1 - 2.0f * my / A2 - 2.0f * mx / B1 + 2.0f * mx / B2);
            part[3 * p + 3 * ch + 1] = -S / B2;
            part[3 * p + 3 * ch + 2] = 2.0f * S / A2;
            contrib += (1.0f - a.lambda) * fabsf(xin[ch] - xin[3 + ch]) - a.lambda * S;
        }
    }
    // the block's loss terms into its own slot (same-address atomics from
    // every block would serialise); a last pass adds the slots
    __shared__ float s_w[SS_TILE * SS_TILE / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) contrib += __shfl_xor(contrib, o, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = contrib;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.0f;
        for (int w = 0; w < SS_TILE * SS_TILE / 64; ++w) t += s_w[w];
        block_loss[blockIdx.y * gridDim.x + blockIdx.x] = t;
    }
}

// Pass 2: dL/dx = (1 - lambda) sign(x - y) / n - lambda / n (G*d_mu + 2 x G*d_xx + y G*d_xy).
__global__ __launch_bounds__(SS_TILE * SS_TILE) void ssim_grad_kernel(const float *__restrict__ x,
                                                                      const float *__restrict__ y, SsimArgs a,
                                                                      const float *__restrict__ part,
                                                                      float *__restrict__ grad)
{
    constexpr int NP = 9;
    __shared__ float s_in[SS_IN * SS_IN * NP];
    __shared__ float s_h[SS_IN * SS_TILE * NP];
    const int tx0 = blockIdx.x * SS_TILE - SS_R, ty0 = blockIdx.y * SS_TILE - SS_R;
    {
        // the halo tile of the partials: every load of a thread issued before its LDS stores
        constexpr int NE = SS_IN * SS_IN * NP, PER = (NE + SS_TILE * SS_TILE - 1) / (SS_TILE * SS_TILE);
        float pv[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int j = threadIdx.x + k * SS_TILE * SS_TILE;
            const int pix = j / NP, q = j - pix * NP;
            const int r = pix / SS_IN, c = pix - r * SS_IN, u = tx0 + c, v = ty0 + r;
            const bool in = j < NE && u >= 0 && u < a.W && v >= 0 && v < a.H;
            const float l = part[in ? NP * ((size_t)v * a.W + u) + q : 0]; // unconditional load, zeroed after
            pv[k] = in ? l : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int j = threadIdx.x + k * SS_TILE * SS_TILE;
            if (j < NE) s_in[j] = pv[k];
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < SS_IN * SS_TILE; j += SS_TILE * SS_TILE) {
        const int r = j / SS_TILE, c = j - r * SS_TILE;
        float acc[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) acc[q] = 0.0f;
#pragma unroll
        for (int t = 0; t <= 2 * SS_R; ++t) {
            const float *e = &s_in[(r * SS_IN + c + t) * NP];
            const float w = a.g[t];
#pragma unroll
            for (int q = 0; q < NP; ++q) acc[q] = fmaf(w, e[q], acc[q]);
        }
#pragma unroll
        for (int q = 0; q < NP; ++q) s_h[j * NP + q] = acc[q];
    }
    __syncthreads();
    const int cx = threadIdx.x % SS_TILE, cy = threadIdx.x / SS_TILE;
    const int u = blockIdx.x * SS_TILE + cx, v = blockIdx.y * SS_TILE + cy;
    if (u >= a.W || v >= a.H) return;
    float b[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) b[q] = 0.0f;
#pragma unroll
    for (int t = 0; t <= 2 * SS_R; ++t) {
        const float *e = &s_h[((cy + t) * SS_TILE + cx) * NP];
        const float w = a.g[t];
#pragma unroll
        for (int q = 0; q < NP; ++q) b[q] = fmaf(w, e[q], b[q]);
    }
    const size_t p = 3 * ((size_t)v * a.W + u);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        const float xv = x[p + ch], yv = y[p + ch], d = xv - yv;
        const float sg = d > 0.0f ? 1.0f : (d < 0.0f ? -1.0f : 0.0f);
        const float ds = b[3 * ch] + 2.0f * xv * b[3 * ch + 1] + yv * b[3 * ch + 2];
        grad[p + ch] = a.inv_n * ((1.0f - a.lambda) * sg - a.lambda * ds);
    }
}

// ---- one pass down strips of columns

// A workgroup takes SS_OUT float columns of `rows` output rows and walks down
// them, one thread per column (columns are channels of pixels, so taps are 3
// floats apart).  Per step a thread blurs a row of moments horizontally out of
// LDS and adds it to the vertical sums of the 11 rows it belongs to; the row
// that completes gives its partial derivatives, which go through LDS and a
// second pair of blurs in the step after; the row of partials that completes
// there gives an output row.  The sums are registers (the row loop is unrolled
// over the 11 phases of their rotation), input rows are loaded two steps ahead,
// and one barrier a step suffices with both LDS rows double-buffered.
//
// Bound by VALU issue: 154 fused multiply-adds of the blurs and about 80 other
// instructions per column and step, 20 warm-up rows per workgroup and 30 of 256
// columns of halo.  Two passes over tiles with the nine partials of a pixel in
// memory between them, which read 26 x 26 pixels for 16 x 16, take 144 us at
// 1920x1080; this takes 103 us.
template <int P> struct Phase { static constexpr int value = P; };
constexpr int SS_BLOCK = 256;
constexpr int SS_HALO = 3 * SS_R;
constexpr int SS_OUT = SS_BLOCK - 2 * SS_HALO;
__global__ __launch_bounds__(SS_BLOCK) void ssim_kernel(const float *__restrict__ x, const float *__restrict__ y, SsimArgs a,
                                                        float *__restrict__ grad, float *__restrict__ block_loss)
{
    __shared__ float4 s_in[2][SS_BLOCK + 2 * SS_HALO]; // x, y, (x - y)^2, xy
    __shared__ float4 s_p[2][SS_BLOCK + 2 * SS_HALO];  // dS/dmu_x, dS/dE[x^2], dS/dE[xy]
    const int t = threadIdx.x;
    const int c = blockIdx.x * SS_OUT - SS_HALO + t; // the thread's column
    const int r0 = blockIdx.y * a.rows, r1 = min(r0 + a.rows, a.H);
    const bool col_in = c >= 0 && c < a.W3;
    const bool owner = col_in && t >= SS_HALO && t < SS_HALO + SS_OUT; // of the column's outputs and loss terms
    // the input columns: entry t (column c - SS_HALO) and, for the first 2
    // SS_HALO threads, entry SS_BLOCK + t
    const int ca = c - SS_HALO, cb = ca + SS_BLOCK;
    const bool in_a = ca >= 0 && ca < a.W3, in_b = t < 2 * SS_HALO && cb >= 0 && cb < a.W3;
    float xa, ya, xb, yb; // the row in flight
    auto load = [&](int r) { // unconditional loads (a clamped address), zeroed after
        const bool ok = r >= 0 && r < a.H && r < r1 + 2 * SS_R;
        const size_t row = (size_t)(ok ? r : 0) * a.W3;
        const size_t pa = row + (in_a ? ca : 0), pb = row + (in_b ? cb : 0);
        xa = x[pa]; ya = y[pa]; xb = x[pb]; yb = y[pb];
        if (!(ok && in_a)) xa = ya = 0.0f;
        if (!(ok && in_b)) xb = yb = 0.0f;
    };
    auto store = [&](int buf) {
        const float da = xa - ya, db = xb - yb;
        s_in[buf][t] = make_float4(xa, ya, da * da, xa * ya);
        if (t < 2 * SS_HALO) s_in[buf][SS_BLOCK + t] = make_float4(xb, yb, db * db, xb * yb);
    };
    // the halves of s_p's halo that no thread writes are read only for columns
    // without an output
    float m[SS_N][4] = {}; // vertical sums of the moments, one slot per row under way
    float b[SS_N][3] = {}; // of the partials
    for (int j = t; j < 2 * (SS_BLOCK + 2 * SS_HALO); j += SS_BLOCK) (&s_p[0][0])[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    float sum = 0.0f; // loss terms
    float nx = 0.0f, ny = 0.0f;
    const int top = r0 - 2 * SS_R, steps = r1 - r0 + 4 * SS_R + 1;
    load(top);
    store(0);
    load(top + 1);
    __syncthreads();
    // one step; its phase (i modulo 11) is a constant, so that the slots are registers
    auto step = [&](auto phase, int i) __attribute__((always_inline)) {
        constexpr int p = decltype(phase)::value;
        const int r = top + i, out_row = r - 2 * SS_R - 1;
        // the next row leaves its registers, the one after it starts
        store((i + 1) & 1);
        load(r + 2);
        // x and y of this step's output row, loaded in the last one
        const bool out_ok = owner && out_row >= r0;
        const float ox = nx, oy = ny;
        const size_t op = out_ok ? (size_t)out_row * a.W3 + c : 0;
        const size_t np = owner && out_row + 1 >= r0 && out_row + 1 < r1 ? (size_t)(out_row + 1) * a.W3 + c : 0;
        nx = x[np];
        ny = y[np];
        // moments of input row r, horizontally, into the rows r - 5 .. r + 5
        float4 h = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < SS_N; ++k) {
            const float4 e = s_in[i & 1][t + 3 * k];
            h.x = fmaf(a.g[k], e.x, h.x);
            h.y = fmaf(a.g[k], e.y, h.y);
            h.z = fmaf(a.g[k], e.z, h.z);
            h.w = fmaf(a.g[k], e.w, h.w);
        }
#pragma unroll
        for (int j = 0; j < SS_N; ++j) {
            float *q = m[(p + SS_R - j + SS_N) % SS_N]; // row r + 5 - j
            q[0] = j == 0 ? a.g[0] * h.x : fmaf(a.g[j], h.x, q[0]);
            q[1] = j == 0 ? a.g[0] * h.y : fmaf(a.g[j], h.y, q[1]);
            q[2] = j == 0 ? a.g[0] * h.z : fmaf(a.g[j], h.z, q[2]);
            q[3] = j == 0 ? a.g[0] * h.w : fmaf(a.g[j], h.w, q[3]);
        }
        {   // row r - 5 is complete: S = A1 A2 / (B1 B2) and its partials, with A1 = B1 - md^2
            // and A2 = B2 - v, v the variance of x - y: small differences taken as such
            // (equal images have a gradient of exactly 0), and B2's variances as v and twice the
            // covariance, whose terms are no larger than the sum
            const float *q = m[(p + SS_R + 1) % SS_N];
            const int s = r - SS_R;
            const float mx = q[0], my = q[1], md = mx - my, v = fmaf(-md, md, q[2]);
            const float i1 = 1.0f / (fmaf(mx, mx, my * my) + SS_C1);
            const float i2 = 1.0f / ((2.0f * fmaf(-mx, my, q[3]) + SS_C2) + v);
            const float l = md * md * i1, w = v * i2, q1 = 1.0f - l, q2 = 1.0f - w; // q1 = A1 / B1, q2 = A2 / B2
            const float S = q1 * q2;
            const bool ok = col_in && s >= 0 && s < a.H;
            const float d0 = 2.0f * (i1 * q2 * fmaf(mx, l, -md) + i2 * q1 * fmaf(-mx, w, md));
            s_p[i & 1][SS_HALO + t] =
                make_float4(ok ? d0 : 0.0f, ok ? -S * i2 : 0.0f, ok ? 2.0f * q1 * i2 : 0.0f, 0.0f);
            if (owner && s >= r0 && s < r1) sum -= a.lambda * S;
        }
        // partials of row r - 6 (last step's), into the rows r - 11 .. r - 1
        float3 u = make_float3(0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < SS_N; ++k) {
            const float4 e = s_p[(i + 1) & 1][t + 3 * k];
            u.x = fmaf(a.g[k], e.x, u.x);
            u.y = fmaf(a.g[k], e.y, u.y);
            u.z = fmaf(a.g[k], e.z, u.z);
        }
#pragma unroll
        for (int j = 0; j < SS_N; ++j) {
            float *q = b[(p + SS_R - j + SS_N) % SS_N];
            q[0] = j == 0 ? a.g[0] * u.x : fmaf(a.g[j], u.x, q[0]);
            q[1] = j == 0 ? a.g[0] * u.y : fmaf(a.g[j], u.y, q[1]);
            q[2] = j == 0 ? a.g[0] * u.z : fmaf(a.g[j], u.z, q[2]);
        }
        if (out_ok) { // dL/dx = (1 - lambda) sign(x - y) / n - lambda / n (G*d_mu + 2 x G*d_xx + y G*d_xy)
            const float *q = b[(p + SS_R + 1) % SS_N];
            const float d = ox - oy;
            const float sg = d > 0.0f ? 1.0f : (d < 0.0f ? -1.0f : 0.0f);
            const float ds = q[0] + 2.0f * ox * q[1] + oy * q[2];
            grad[op] = a.inv_n * ((1.0f - a.lambda) * sg - a.lambda * ds);
            sum += (1.0f - a.lambda) * fabsf(d);
        }
        __syncthreads();
    };
    for (int i = 0; i < steps; i += SS_N) {
        step(Phase<0>{}, i);
        if (i + 1 < steps) step(Phase<1>{}, i + 1);
        if (i + 2 < steps) step(Phase<2>{}, i + 2);
        if (i + 3 < steps) step(Phase<3>{}, i + 3);
        if (i + 4 < steps) step(Phase<4>{}, i + 4);
        if (i + 5 < steps) step(Phase<5>{}, i + 5);
        if (i + 6 < steps) step(Phase<6>{}, i + 6);
        if (i + 7 < steps) step(Phase<7>{}, i + 7);
        if (i + 8 < steps) step(Phase<8>{}, i + 8);
        if (i + 9 < steps) step(Phase<9>{}, i + 9);
        if (i + 10 < steps) step(Phase<10>{}, i + 10);
    }
    // the block's loss terms into its own slot (same-address atomics from
    // every block would serialise); a last pass adds the slots
    __shared__ float s_w[SS_BLOCK / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if ((t & 63) == 0) s_w[t >> 6] = sum;
    __syncthreads();
    if (t == 0) block_loss[blockIdx.y * gridDim.x + blockIdx.x] = (s_w[0] + s_w[1]) + (s_w[2] + s_w[3]);
}

// Output rows of a workgroup: fewer rows mean more workgroups on a CU, which
// hide each other's latencies, and more warm-up steps.  A step of k workgroups
// on one CU (at most 4 fit) was measured at 1.08, 1.40, 1.74 and 2.1 us for k = 1
// to 4 (120, 60, 40 and 30 rows at 1920x1080: 152, 113, 106, 108 us): 0.74 + 0.34
// k; the rows with the least steps x price are taken.  *us: that product.
int ssim_rows(int strips, int H, int cus, double *us)
{
    int best = H;
    *us = 1e300;
    for (int rows = H;;) {
        const int segs = (H + rows - 1) / rows, k = (strips * segs + cus - 1) / cus;
        if (k > 8 && segs > 1) break;
        const double cost = (rows + 4 * SS_R + 1) * (k / 4 * 2.1 + (k % 4 ? 0.74 + 0.34 * (k % 4) : 0.0));
        if (cost < *us) {
            *us = cost;
            best = rows;
        }
        if (rows == 1) break;
        const int more = (H + rows - 2) / (rows - 1); // segments of a row less
        rows = (H + more - 1) / more;
    }
    return best;
}

// Whether an image goes through the tiles: a strip's step costs about a
// microsecond however few workgroups run, and strips of a narrow image are
// partly empty, where tiles undercut them.  Tiles take 15.6 us + 15.8 ns each and
// no less than 24 us, strips 2 us over their steps (above).  us, strips / tiles:
// 16x16 27 / 25, 300x300 32 / 26, 16x4096 44 / 27, 640x427 41 / 35, 900x600 56 / 50,
// 979x546 55 / 51, 1000x640 60 / 54, 76x16384 110 / 96; 500x1500 60 / 65, 160x8192
// 90 / 97, 1100x700 59 / 65, 100x16384 110 / 126, 1297x840 72 / 85, 1920x1080
// 103 / 144.
bool ssim_by_tiles(int width, int height, double strips_us)
{
    const double tiles = (double)((width + SS_TILE - 1) / SS_TILE) * ((height + SS_TILE - 1) / SS_TILE);
    return std::max(24.0, 15.6 + 0.0158 * tiles) <= strips_us + 2.0;
}

__global__ __launch_bounds__(256) void copy_floats_kernel(size_t n, const float *__restrict__ from, float *__restrict__ to)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) to[i] = from[i];
}

// loss += lambda + inv_n * (sum of the blocks' terms): one workgroup.
__global__ __launch_bounds__(1024) void ssim_loss_sum_kernel(const float *__restrict__ block_loss, int nb, SsimArgs a,
                                                             float *__restrict__ loss)
{
    __shared__ float s_w[16];
    float t = 0.0f;
    for (int b = threadIdx.x; b < nb; b += 1024) t += block_loss[b];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        float u = 0.0f;
        for (int w = 0; w < 16; ++w) u += s_w[w];
        *loss += a.lambda + u * a.inv_n;
    }
}

enum : int { ACT_ID = 0, ACT_EXP = 1, ACT_SIGMOID = 2 };

template <int ACT> __device__ __forceinline__ float activate(float r)
{
    if constexpr (ACT == ACT_EXP) return expf(r);
    else if constexpr (ACT == ACT_SIGMOID) return 1.0f / (1.0f + expf(-r));
    else return r;
}

// One parameter array of an Adam step.  Elements e with row > 0 and
// e % row >= first take the second step size.
struct AdamPart {
    const float *g;
    float *raw, *m, *v, *act; // act nullable
    size_t n;
    uint32_t first_block;  // of the grid: the part's chunks
    int kind, row, first;
    float step_size;       // lr / (1 - beta1^t) of the first rate
    float step_size2;      // the same for the second rate (SH coefficients past the first)
    bool vec;              // every array 16-byte aligned
};
constexpr int ADAM_PARTS = 5;
struct AdamArgs {
    float beta2, omb1, omb2, eps; // beta2, 1 - betas (formed in double)
    float bc2_sqrt;               // sqrt(1 - beta2^t)
    AdamPart part[ADAM_PARTS];
};

// One parameter element: the activation's derivative at the current raw
// value, the moment updates and the step on the raw value.
template <int ACT>
__device__ __forceinline__ void adam_element(float r, float gact, float m0, float v0, float ss, const AdamArgs &a, float &rn,
                                             float &mm, float &vv)
{
    float da = 1.0f; // d activated / d raw at the current raw value
    if constexpr (ACT == ACT_EXP) da = expf(r);
    else if constexpr (ACT == ACT_SIGMOID) {
        const float s = 1.0f / (1.0f + expf(-r));
        da = s * (1.0f - s);
    }
    const float g = gact * da;
    mm = m0 + a.omb1 * (g - m0);
    vv = a.beta2 * v0 + a.omb2 * (g * g);
    const float denom = sqrtf(vv) / a.bc2_sqrt + a.eps;
    rn = r - ss * (mm / denom);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int ADAM_BLOCK = 256, ADAM_CHUNK = ADAM_BLOCK * 4; // elements a workgroup

template <int ACT>
__device__ __forceinline__ void adam_chunk(const AdamArgs &a, const AdamPart &p, uint32_t chunk)
{
    const size_t e0 = (size_t)chunk * ADAM_CHUNK;
    const uint32_t left = (uint32_t)min(p.n - e0, (size_t)ADAM_CHUNK), row = (uint32_t)p.row;
    // the chunk's first element's place in its row
    const uint32_t c0 = row ? (chunk % row) * (ADAM_CHUNK % row) % row : 0u;
    auto rate = [&](uint32_t col) { return row && (int)col >= p.first ? p.step_size2 : p.step_size; };
    auto one = [&](uint32_t i) {
        const size_t e = e0 + i;
        float rn, mm, vv;
        adam_element<ACT>(p.raw[e], p.g[e], p.m[e], p.v[e], rate(row ? (c0 + i) % row : 0u), a, rn, mm, vv);
        p.raw[e] = rn;
        p.m[e] = mm;
        p.v[e] = vv;
        if (p.act) p.act[e] = activate<ACT>(rn);
    };
    if (!p.vec) {
        for (uint32_t i = threadIdx.x; i < left; i += ADAM_BLOCK) one(i);
        return;
    }
    const f32x4 *raw = reinterpret_cast<const f32x4 *>(p.raw + e0), *g = reinterpret_cast<const f32x4 *>(p.g + e0);
    const f32x4 *m = reinterpret_cast<const f32x4 *>(p.m + e0), *v = reinterpret_cast<const f32x4 *>(p.v + e0);
    const uint32_t full = left / 4, q = threadIdx.x;
    if (q < full) {
        const f32x4 r4 = __builtin_nontemporal_load(raw + q), g4 = __builtin_nontemporal_load(g + q);
        const f32x4 m4 = __builtin_nontemporal_load(m + q), v4 = __builtin_nontemporal_load(v + q);
        uint32_t col = row ? (c0 + 4u * q) % row : 0u;
        f32x4 rn, mm, vv, av;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float x, y, z;
            adam_element<ACT>(r4[j], g4[j], m4[j], v4[j], rate(col), a, x, y, z);
            rn[j] = x;
            mm[j] = y;
            vv[j] = z;
            av[j] = activate<ACT>(x);
            col = col + 1 == row ? 0u : col + 1;
        }
        __builtin_nontemporal_store(rn, reinterpret_cast<f32x4 *>(p.raw + e0) + q);
        __builtin_nontemporal_store(mm, reinterpret_cast<f32x4 *>(p.m + e0) + q);
        __builtin_nontemporal_store(vv, reinterpret_cast<f32x4 *>(p.v + e0) + q);
        if (p.act) reinterpret_cast<f32x4 *>(p.act + e0)[q] = av;
    }
    if (threadIdx.x < left % 4) one(4 * full + threadIdx.x); // the array's last ones
}

// One step on every parameter array: a workgroup updates one chunk of one array
// in 16-byte accesses (element by element where an array is not so aligned).
// HBM-bound: 4 reads and 4 writes an element.  What the step itself reads only
// once does not go through the caches, the activated values that the next render
// reads do: 1M convexes (K = 6, degree 3; 2.2 GB) 380 us, with every access cached
// 428, with none 429, with only the loads cached 438; a launch per array 445.
// 16 bytes a thread and array; 32 or 64 at once are no faster (394, 377).
__global__ __launch_bounds__(ADAM_BLOCK) void adam_kernel(AdamArgs a)
{
    int k = 0;
#pragma unroll
    for (int j = 1; j < ADAM_PARTS; ++j) k = blockIdx.x >= a.part[j].first_block ? j : k;
    const AdamPart &p = a.part[k];
    const uint32_t chunk = blockIdx.x - p.first_block;
    if (p.kind == ACT_ID) adam_chunk<ACT_ID>(a, p, chunk);
    else if (p.kind == ACT_EXP) adam_chunk<ACT_EXP>(a, p, chunk);
    else adam_chunk<ACT_SIGMOID>(a, p, chunk);
}

bool set_complete(const cs_param_set *p)
{
    return p && p->points && p->delta && p->sigma && p->opacity && p->sh;
}

} // namespace

} // namespace cs

using namespace cs;

extern "C" {

int cs_adam_step(cs_ctx *ctx, int32_t n, int32_t k, int32_t sh_degree, const cs_grads *grad, const cs_param_set *raw,
                 const cs_param_set *m, const cs_param_set *v, const cs_param_set *activated,
                 const cs_adam_params *prm, void *hip_stream)
{
    if (!ctx) return fail(CS_EINVAL, "ctx is NULL");
    if (n < 0 || k < 3 || k > CS_MAX_K || sh_degree < 0 || sh_degree > CS_MAX_SH_DEGREE)
        return fail(CS_EINVAL, "bad n, k or sh_degree");
    if (!prm) return fail(CS_EINVAL, "params is NULL");
    if (prm->step < 1) return fail(CS_EINVAL, "adam step %d < 1", prm->step);
    if (!(prm->beta1 >= 0.0 && prm->beta1 < 1.0 && prm->beta2 >= 0.0 && prm->beta2 < 1.0))
        return fail(CS_EINVAL, "betas outside [0, 1)");
    if (n == 0) return CS_OK;
    if (!grad || !grad->points || !grad->delta || !grad->sigma || !grad->opacity || !grad->sh || !set_complete(raw) ||
        !set_complete(m) || !set_complete(v) || (activated && !set_complete(activated)))
        return fail(CS_EINVAL, "array pointer is NULL");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(CS_EHIP, "hipSetDevice failed");
    hipStream_t st = (hipStream_t)hip_stream;
    const double bc1 = 1.0 - std::pow(prm->beta1, (double)prm->step);
    const double bc2 = 1.0 - std::pow(prm->beta2, (double)prm->step);
    AdamArgs a{};
    a.beta2 = (float)prm->beta2;
    a.omb1 = (float)(1.0 - prm->beta1);
    a.omb2 = (float)(1.0 - prm->beta2);
    a.eps = prm->eps;
    a.bc2_sqrt = (float)std::sqrt(bc2);
    const size_t N = (size_t)n;
    const int nsh = 3 * (sh_degree + 1) * (sh_degree + 1);
    uint32_t blocks = 0, parts = 0;
    auto add = [&](int kind, size_t count, float *cs_grads::*gf, float *cs_param_set::*f, float lr, float lr2, int row, int first) {
        AdamPart &p = a.part[parts++];
        p = {grad->*gf, raw->*f, m->*f, v->*f, activated ? activated->*f : nullptr, count, blocks, kind, row, first,
             (float)(lr / bc1), (float)(lr2 / bc1), true};
        for (const float *q : {p.g, (const float *)p.raw, (const float *)p.m, (const float *)p.v, (const float *)p.act})
            p.vec = p.vec && ((uintptr_t)q & 15u) == 0;
        blocks += (uint32_t)((count + ADAM_CHUNK - 1) / ADAM_CHUNK); // (count < 2^31 * 48)
    };
    add(ACT_ID, N * 3 * k, &cs_grads::points, &cs_param_set::points, prm->lr_points, prm->lr_points, 0, 0);
    add(ACT_EXP, N, &cs_grads::delta, &cs_param_set::delta, prm->lr_delta, prm->lr_delta, 0, 0);
    add(ACT_EXP, N, &cs_grads::sigma, &cs_param_set::sigma, prm->lr_sigma, prm->lr_sigma, 0, 0);
    add(ACT_SIGMOID, N, &cs_grads::opacity, &cs_param_set::opacity, prm->lr_opacity, prm->lr_opacity, 0, 0);
    add(ACT_ID, N * nsh, &cs_grads::sh, &cs_param_set::sh, prm->lr_sh_dc, prm->lr_sh_rest, nsh, 3);
    hipLaunchKernelGGL(adam_kernel, dim3(blocks), dim3(ADAM_BLOCK), 0, st, a);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? CS_OK : fail(CS_EHIP, "adam launch: %s", hipGetErrorString(e));
}

int cs_ssim_loss_grad(cs_ctx *ctx, const float *rgb, const float *target, int32_t width, int32_t height, float lambda,
                      float *dl_drgb, float *loss, void *hip_stream)
{
    if (!ctx || !rgb || !target || !dl_drgb || !loss) return fail(CS_EINVAL, "NULL argument");
    if (width <= 0 || height <= 0 || width > 16384 || height > 16384) return fail(CS_EINVAL, "bad image size");
    if (!(lambda >= 0.0f && lambda <= 1.0f)) return fail(CS_EINVAL, "lambda outside [0, 1]");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(CS_EHIP, "hipSetDevice failed");
    hipStream_t st = (hipStream_t)hip_stream;
    SsimArgs a;
    a.W = width;
    a.W3 = 3 * width;
    a.H = height;
    a.lambda = lambda;
    a.inv_n = (float)(1.0 / (3.0 * (double)width * (double)height));
    double gs[SS_N], tot = 0.0;
    for (int t = -SS_R; t <= SS_R; ++t) tot += gs[t + SS_R] = std::exp(-(double)(t * t) / (2.0 * 1.5 * 1.5));
    for (int t = 0; t < SS_N; ++t) a.g[t] = (float)(gs[t] / tot);
    int cus = 256;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device);
    const int strips = (a.W3 + SS_OUT - 1) / SS_OUT;
    double strips_us = 0.0;
    a.rows = ssim_rows(strips, height, std::max(1, cus), &strips_us);
    const size_t n = 3 * (size_t)width * height;
    const bool tiles = ssim_by_tiles(width, height, strips_us);
    const dim3 grid = tiles ? dim3((width + SS_TILE - 1) / SS_TILE, (height + SS_TILE - 1) / SS_TILE)
                            : dim3(strips, (height + a.rows - 1) / a.rows);
    const int nb = (int)(grid.x * grid.y);
    // strips read rows that other workgroups have done: a gradient written over
    // an input goes through scratch
    auto overlaps = [&](const float *p) { return dl_drgb < p + n && p < dl_drgb + n; };
    const bool aside = !tiles && (overlaps(rgb) || overlaps(target));
    float *block_loss = nullptr;
    hipError_t e = hipMallocAsync((void **)&block_loss, (nb + (tiles ? 3 * n : aside ? n : 0)) * sizeof(float), st);
    if (e != hipSuccess) return fail(CS_ENOMEM, "ssim scratch: %s", hipGetErrorString(e));
    float *rest = block_loss + nb; // the partials, or the gradient aside
    if (tiles)
        hipLaunchKernelGGL(ssim_moments_kernel, grid, dim3(SS_TILE * SS_TILE), 0, st, rgb, target, a, rest, block_loss);
    else
        hipLaunchKernelGGL(ssim_kernel, grid, dim3(SS_BLOCK), 0, st, rgb, target, a, aside ? rest : dl_drgb, block_loss);
    hipLaunchKernelGGL(ssim_loss_sum_kernel, dim3(1), dim3(1024), 0, st, block_loss, nb, a, loss);
    if (tiles)
        hipLaunchKernelGGL(ssim_grad_kernel, grid, dim3(SS_TILE * SS_TILE), 0, st, rgb, target, a, rest, dl_drgb);
    else if (aside)
        hipLaunchKernelGGL(copy_floats_kernel, dim3((unsigned)std::min<size_t>((n + 255) / 256, 4096)), dim3(256), 0, st, n,
                           rest, dl_drgb);
    e = hipGetLastError();
    (void)hipFreeAsync(block_loss, st);
    return e == hipSuccess ? CS_OK : fail(CS_EHIP, "ssim launch: %s", hipGetErrorString(e));
}

} // extern "C"
