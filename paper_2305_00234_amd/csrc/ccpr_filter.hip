// gfx950 kernels of the design filtering and projection (Sec. "Filtering and
// projection"): the cone filter of Eq. FilterFunction, the smoothed Heaviside
// of Eq. Projection, their chain rule (Eq. GradientsFiltered) and the measure
// of non-discreteness (Eq. MeasureOfNon-discretness), on the per-voxel density
// grid of the design box ([nz][ny][nx], x fastest; distances in voxels).
//
// The filter is a 3-D stencil over the sphere |d| < R (R <= 17), summed tap by
// tap, so it is bound by the FMA rate, not by memory (905 taps a voxel at R = 6
// against 16 bytes).  What the taps read has to cost less than the FMAs: a
// thread owns 8 consecutive outputs of a row and slides an 8-value register
// window along the staged row, so a tap is 8 FMAs, one LDS value and one
// broadcast weight (one output a thread needs three LDS words for two FMAs).
// A workgroup owns a 32 x 32 tile of Q planes and stages each input plane (tile
// plus halo) in LDS once for all Q; 4 lanes along x and 16 rows a wave with a row
// stride of 1 modulo 8 words keep the float reads free of bank conflicts.  The
// denominator (weight sum inside the box) is summed tap by tap beside the values,
// once a thread where the tile and its halo lie inside the box along x (all its
// outputs then see the same weights) and once an output elsewhere.  (Looked up in
// cumulative weights instead it rounds differently, by up to 2e-5 in rho_b.)
//
// Per-edge design variables (one density per E edge at the staggered edge
// centres: x edges at (i+1/2, j, k), y edges at (i, j+1/2, k), z edges at
// (i, j, k+1/2) of an N-cell design, component c holding N_l + 1 - delta(c,l)
// edges along axis l; flat arrays hold the x, y, z edges in turn, each x
// fastest) use the same kernels: Eq. FilterFunction's sphere around an edge
// takes in the edges of all three components, and between component b and the
// output's component a the index offset o maps to the distance |o + h_b - h_a|,
// h_c the half-cell vector along axis c (|o| < R + 1/2).  One launch covers the
// three output components.
//
// The order of a sum (component, z, y, x offset) does not depend on the tile.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/ccprfdtd.h"

namespace {

constexpr int kTX = 32;      // tile width (x)

// The grid of one component per part: one part (voxels) or three (edges).
struct FilterGeom {
    int nc;
    int shp[3][3];     // [component] (x, y, z) extents
    long long off[3];  // first flat index of each component
    int zb[4];         // first z block of each component (Q planes each)
    int H;             // largest integer offset
    int W;             // row stride of the staged tile
    int rows;          // tile height (y)
    int nbx, nby;      // tiles along x and y
};

// Row stride of the weight table, and the words of LDS before the tile: weights
// [D][stride] and the inside mask of a tile row (both multiples of 4 words).
__host__ __device__ inline int weight_stride(int H) { return (2 * H + 1 + 7) / 8 * 8; }
__host__ __device__ inline int mask_words(int H) { return (kTX + 2 * H + 8 + 3) / 4 * 4; }
__host__ __device__ inline int table_words(int H) { return (2 * H + 1) * weight_stride(H) + mask_words(H); }

// The offsets of row dy inside the sphere's disk at z distance fz (z offset
// dz) between components shifted by (sx, sy): n of them from 'first' on.
template <bool EDGE>
__device__ __forceinline__ void disk_row(int H, float R, float R2, float sx, float sy, float fz, int dy, int dz,
                                         int& first, int& n)
{
    if constexpr (EDGE) {
        const float fy = (float)dy + sy, rest = fy * fy + fz * fz;
        auto in = [&](int dx) {
            const float fx = (float)dx + sx;
            return fx * fx + rest < R2;
        };
        const float rr = sqrtf(fmaxf(R2 - rest, 0.f));
        int lo = max(-H, (int)floorf(-sx - rr)), hi = min(H, (int)ceilf(-sx + rr));
        while (lo <= hi && !in(lo)) ++lo;
        while (hi >= lo && !in(hi)) --hi;
        first = lo;
        n = hi - lo + 1;
    } else {
        const float ry2 = R * R - (float)(dz * dz) - (float)(dy * dy);
        const int m = ry2 > 0.f ? (int)ceilf(sqrtf(ry2)) - 1 : -1;
        first = -m;
        n = m < 0 ? 0 : 2 * m + 1;
    }
}

// The disk's weights, each row's from slot 0 of its table row on.
template <bool EDGE>
__device__ __forceinline__ void disk_weights(int H, float R, float R2, float sx, float sy, float fz, int dz, float* wts)
{
    const int D = 2 * H + 1, WS = weight_stride(H);
    const int t0 = threadIdx.x & 7;
    for (int r = threadIdx.x >> 3; r < D; r += blockDim.x >> 3) {
        const int dy = r - H;
        int first, n;
        disk_row<EDGE>(H, R, R2, sx, sy, fz, dy, dz, first, n);
        for (int t = t0; t < n; t += 8) {
            const int dx = first + t;
            if constexpr (EDGE) {
                const float fx = (float)dx + sx, fy = (float)dy + sy;
                wts[r * WS + t] = R - sqrtf(fx * fx + fy * fy + fz * fz);
            } else {
                wts[r * WS + t] = R - sqrtf((float)(dx * dx + dy * dy + dz * dz));
            }
        }
    }
}

// One row's n taps on P consecutive outputs, in order: sum[p] += w[t] rp[p + t];
// DEN 1: den[0] += w[t] yf; DEN 2: den[p] += w[t] yf mp[p + t] (yf, mp: 1 inside
// the box, 0 outside).  Each block of 8 taps loads its 8 new values and 8 weights
// before any is used (values past the run are padding or neighbours, not used).
template <typename T, int P, int DEN>
__device__ __forceinline__ void row_taps(const T* rp, const float* wp, const float* mp, float yf, int n, T (&sum)[P],
                                         float (&den)[P])
{
    T X[P + 8];
    float M[DEN == 2 ? P + 8 : 1];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        X[p] = rp[p];
        if constexpr (DEN == 2) M[p] = mp[p];
    }
    for (int t = 0; t < n; t += 8) {
        float w[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            w[q] = wp[t + q];
            X[P + q] = rp[t + P + q];
            if constexpr (DEN == 2) M[P + q] = mp[t + P + q];
        }
        const int m = n - t;  // uniform
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (q < m) {
                const T wt = (T)w[q];
#pragma unroll
                for (int p = 0; p < P; ++p) sum[p] = fma(wt, X[p + q], sum[p]);
                if constexpr (DEN == 1) den[0] = fmaf(w[q], yf, den[0]);
                if constexpr (DEN == 2) {
                    const float wy = w[q] * yf;
#pragma unroll
                    for (int p = 0; p < P; ++p) den[p] = fmaf(wy, M[p + q], den[p]);
                }
            }
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            X[p] = X[p + 8];
            if constexpr (DEN == 2) M[p] = M[p + 8];
        }
    }
}

// Tile of block 'L' (x tile fastest, then y, then z blocks component by
// component): output component, first column, row and plane.
struct Tile {
    int a, x0, y0, k0;
    bool any;  // false where this component has no outputs in the tile
};
template <int Q>
__device__ __forceinline__ Tile tile_of(const FilterGeom& g, int L)
{
    const int u = L / g.nbx, z = u / g.nby;
    int c = 0;
    while (c + 1 < g.nc && z >= g.zb[c + 1]) ++c;
    Tile t;
    t.a = c;
    t.x0 = (L - u * g.nbx) * kTX;
    t.y0 = (u - z * g.nby) * g.rows;
    t.k0 = (z - g.zb[c]) * Q;
    t.any = t.x0 < g.shp[c][0] && t.y0 < g.shp[c][1];
    return t;
}

// The taps of one workgroup's tile: sum[q][p] of the staged values and (DEN)
// den[q][p] of the weights inside the box, for the Q planes from k0 on of
// component a.  stage.load(m) reads flat index m, stage.value forms its value.
// DEN 1 where every offset of the tile lies inside the box along x (one
// denominator a thread), DEN 2 elsewhere.
template <typename T, int P, int Q, bool EDGE, int DEN, typename Stage>
__device__ __forceinline__ void sphere_sums(const FilterGeom& g, const Tile& tl, float R, float R2, unsigned char* lds,
                                            Stage stage, T (&sum)[Q][P], float (&den)[Q][P])
{
    constexpr int LX = kTX / P;  // lanes along x
    const int H = g.H, W = g.W, D = 2 * H + 1, WS = weight_stride(H), rows = g.rows;
    float* const wts = reinterpret_cast<float*>(lds);
    float* const mask = wts + D * WS;
    T* const tile = reinterpret_cast<T*>(mask + mask_words(H));
    const int lane = threadIdx.x & 63;
    // staged positions; t / wide = t * inv >> 20 for t < total <= 98 * 66 (+ a batch)
    const int wide = kTX + 2 * H, total = wide * (rows + 2 * H);
    const unsigned inv = ((1u << 20) + wide - 1) / wide;
    const int tx = threadIdx.x % LX, ty = threadIdx.x / LX;
    const int a = tl.a, k0 = tl.k0, gx0 = tl.x0, gy0 = tl.y0, j = gy0 + ty;
    const int ka1 = min(k0 + Q, g.shp[a][2]);
    for (int b = 0; b < (EDGE ? 3 : 1); ++b) {
        const float sx = EDGE ? 0.5f * ((b == 0) - (a == 0)) : 0.f, sy = EDGE ? 0.5f * ((b == 1) - (a == 1)) : 0.f,
                    sz = EDGE ? 0.5f * ((b == 2) - (a == 2)) : 0.f;
        const int bx = g.shp[b][0], by = g.shp[b][1], bz = g.shp[b][2];
        for (int kk = max(0, k0 - H); kk <= min(bz - 1, ka1 - 1 + H); ++kk) {
            __syncthreads();
            const long long plane = g.off[b] + (long long)kk * by * bx;
            // the tile, a batch of positions a thread: every load before the first
            // value is formed (one at a time, the loads' latency bound the pass)
            for (int t0 = threadIdx.x; t0 < total; t0 += Stage::kBatch * blockDim.x) {
                typename Stage::Raw raw[Stage::kBatch];
                int at[Stage::kBatch];
#pragma unroll
                for (int u = 0; u < Stage::kBatch; ++u) {
                    const int t = t0 + u * blockDim.x, ly = (int)(((unsigned)t * inv) >> 20), lx = t - ly * wide;
                    const int gx = gx0 - H + lx, gy = gy0 - H + ly;
                    const bool in = t < total && gx >= 0 && gx < bx && gy >= 0 && gy < by;
                    at[u] = t < total ? (ly * W + lx) * 2 + (in ? 1 : 0) : -1;
                    raw[u] = typename Stage::Raw{};
                    if (in) raw[u] = stage.load(plane + (long long)gy * bx + gx);
                }
#pragma unroll
                for (int u = 0; u < Stage::kBatch; ++u)
                    if (at[u] >= 0) tile[at[u] >> 1] = (at[u] & 1) ? stage.value(raw[u]) : (T)0;
            }
            if (DEN == 2)
                for (int lx = threadIdx.x; lx < wide; lx += blockDim.x)
                    mask[lx] = gx0 - H + lx >= 0 && gx0 - H + lx < bx ? 1.f : 0.f;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int k = k0 + q, dz = kk - k;
                const float fz = (float)dz + sz;
                if (k >= ka1 || dz < -H || dz > H || fz * fz >= R2) continue;  // uniform
                if (q > 0) __syncthreads();
                disk_weights<EDGE>(H, R, R2, sx, sy, fz, dz, wts);
                __syncthreads();
                // lane r holds the run of row r (D <= 35): first column, count
                int first, n;
                disk_row<EDGE>(H, R, R2, sx, sy, fz, min(lane, D - 1) - H, dz, first, n);
                const int run = n > 0 ? (H + first) | n << 16 : 0;
                for (int r = 0; r < D; ++r) {
                    const int rr = __builtin_amdgcn_readlane(run, r);
                    if (rr == 0) continue;
                    const int lx = P * tx + (rr & 0xffff), gy = j + r - H;
                    const float* wp = static_cast<const float*>(__builtin_assume_aligned(wts + r * WS, 16));
                    row_taps<T, P, DEN>(tile + (ty + r) * W + lx, wp, mask + lx, gy >= 0 && gy < by ? 1.f : 0.f,
                                        rr >> 16, sum[q], den[q]);
                }
            }
        }
    }
}

// Staged values: the density, or v of the chain rule.
struct StageDensity {
    static constexpr int kBatch = 5;
    typedef float Raw;
    const float* rho;
    __device__ __forceinline__ Raw load(long long m) const { return rho[m]; }
    __device__ __forceinline__ float value(Raw r) const { return r; }
};
struct StageGradient {
    static constexpr int kBatch = 5;
    struct Raw {
        double g;
        float t, w;
    };
    const double* g_b;
    const float* rho_t;
    const float* wsum;
    double slope, beta, eta;  // slope = 4 beta / (tanh beta eta + tanh beta (1 - eta))
    __device__ __forceinline__ Raw load(long long m) const { return Raw{g_b[m], rho_t[m], wsum[m]}; }
    __device__ __forceinline__ double value(Raw r) const
    {
        const double e = exp(-2.0 * fabs(beta * ((double)r.t - eta))), d = 1.0 + e;
        return r.g * (slope * e) / (d * d * (double)r.w);
    }
};

// Eq. FilterFunction and Eq. Projection: rho -> rho_t (filtered), rho_b
// (projected) and W (cone-weight sum of the design positions in the sphere).
// 160x160x80 voxels at R = 3 / 6 / 12: 84 / 420 / 2346 us with one output a thread
// (three LDS words for two FMAs), 51 / 174 / 906 us now; 100x25x100 per edge at
// R = 3 / 7.5: 213 / 1584 and 132 / 809 us.
template <int P, bool EDGE>
__global__ __launch_bounds__(256) void filter_project_kernel(const float* __restrict__ rho, float* rho_t, float* rho_b,
                                                             float* wsum, const FilterGeom g, float R, float R2,
                                                             float beta, float eta, float tbe, float inv_den)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const Tile tl = tile_of<1>(g, blockIdx.x);
    if (!tl.any) return;  // uniform
    const int a = tl.a, k0 = tl.k0;
    float num[1][P], den[1][P];
#pragma unroll
    for (int p = 0; p < P; ++p) num[0][p] = den[0][p] = 0.f;
    const StageDensity stage{rho};
    // all the tile's offsets inside the box along x: one denominator a thread
    int bx = g.shp[0][0];
    if (EDGE) bx = min(bx, min(g.shp[1][0], g.shp[2][0]));
    if (tl.x0 - g.H >= 0 && tl.x0 + kTX - 1 + g.H < bx) {
        sphere_sums<float, P, 1, EDGE, 1>(g, tl, R, R2, lds, stage, num, den);
#pragma unroll
        for (int p = 1; p < P; ++p) den[0][p] = den[0][0];
    } else {
        sphere_sums<float, P, 1, EDGE, 2>(g, tl, R, R2, lds, stage, num, den);
    }
    constexpr int LX = kTX / P;
    const int i0 = tl.x0 + P * (threadIdx.x % LX), j = tl.y0 + threadIdx.x / LX;
    if (j >= g.shp[a][1]) return;
    const long long n = g.off[a] + ((long long)k0 * g.shp[a][1] + j) * g.shp[a][0] + i0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (i0 + p >= g.shp[a][0]) break;
        const float rt = num[0][p] / den[0][p];
        rho_t[n + p] = rt;
        wsum[n + p] = den[0][p];
        rho_b[n + p] = (tbe + tanhf(beta * (rt - eta))) * inv_den;
    }
}

// Eq. GradientsFiltered: dF/drho[n] = sum_m w(m,n) v[m] over the design
// positions m of the sphere around n, v = dF/drho_b * d rho_b/d rho_t / W, all in
// FP64.  v is formed while its plane is staged: with e = exp(-2 |x|), the
// projection's slope 1 - tanh^2 x is 4 e / (1 + e)^2 (no cancellation where it
// is small), and one division serves it and W.  160x160x80 voxels at R = 3 / 6 / 12:
// 204 / 795 / 4019 us with one output a thread, 88 / 297 / 1383 us now;
// 100x25x100 per edge at R = 3 / 7.5: 444 / 2514 and 225 / 1062 us.
template <int P, int Q, bool EDGE>
__global__ __launch_bounds__(256) void filter_project_grad_kernel(const double* __restrict__ g_b,
                                                                  const float* __restrict__ rho_t,
                                                                  const float* __restrict__ wsum, double* gout,
                                                                  const FilterGeom g, float R, float R2, double beta,
                                                                  double eta, double inv_den)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const Tile tl = tile_of<Q>(g, blockIdx.x);
    if (!tl.any) return;  // uniform
    const int a = tl.a, k0 = tl.k0;
    double sum[Q][P];
    float none[Q][P];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int p = 0; p < P; ++p) sum[q][p] = 0.0;
    const StageGradient stage{g_b, rho_t, wsum, 4.0 * beta * inv_den, beta, eta};
    sphere_sums<double, P, Q, EDGE, 0>(g, tl, R, R2, lds, stage, sum, none);
    constexpr int LX = kTX / P;
    const int i0 = tl.x0 + P * (threadIdx.x % LX), j = tl.y0 + threadIdx.x / LX;
    if (j >= g.shp[a][1]) return;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (k0 + q >= g.shp[a][2]) break;
        const long long n = g.off[a] + ((long long)(k0 + q) * g.shp[a][1] + j) * g.shp[a][0] + i0;
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (i0 + p < g.shp[a][0]) gout[n + p] = sum[q][p];
    }
}

constexpr int kFT = 16;                // output tile edge (x and y)
constexpr int kMaxRi = 16;             // largest integer offset (radius <= 17)
constexpr int kTW = kFT + 2 * kMaxRi;  // staged tile edge
constexpr int kMaxH = 17;              // per edge: |offset| < radius + 1/2
constexpr int kTWE = kFT + 2 * kMaxH;

// The same per voxel with one output a thread: a workgroup owns a 16 x 16 tile of
// one output plane; for every z offset it stages the input plane's tile plus an
// R-wide halo as (value, inside) pairs, with the cone weights of that offset's
// disk, and each lane sums the disk straight from LDS (three LDS words for two
// FMAs, but four times the waves; see one_output).
__global__ __launch_bounds__(256) void voxel_filter_kernel(const float* __restrict__ rho, float* rho_t,
                                                             float* rho_b, float* wsum, int nx, int ny, int nz,
                                                             float R, int Ri, float beta, float eta, float tbe,
                                                             float inv_den)
{
    __shared__ float2 tile[kTW * kTW];  // (density, 1) inside the box, (0, 0) outside
    __shared__ float wts[(2 * kMaxRi + 1) * (2 * kMaxRi + 1)];  // cone weights of one z offset
    const int tx = threadIdx.x % kFT, ty = threadIdx.x / kFT;
    const int i = blockIdx.x * kFT + tx, j = blockIdx.y * kFT + ty, k = blockIdx.z;
    const int W = kFT + 2 * Ri, D = 2 * Ri + 1;
    const int gx0 = blockIdx.x * kFT - Ri, gy0 = blockIdx.y * kFT - Ri;
    float num = 0.f, den = 0.f;
    for (int dz = -Ri; dz <= Ri; ++dz) {
        const int kk = k + dz;
        const float rz2 = R * R - (float)(dz * dz);
        if (kk < 0 || kk >= nz || rz2 <= 0.f) continue;  // uniform
        __syncthreads();
        for (int t = threadIdx.x; t < W * W; t += blockDim.x) {
            const int ly = t / W, lx = t - ly * W;
            const int gx = gx0 + lx, gy = gy0 + ly;
            const bool in = gx >= 0 && gx < nx && gy >= 0 && gy < ny;
            tile[t] = in ? make_float2(rho[((long long)kk * ny + gy) * nx + gx], 1.f) : make_float2(0.f, 0.f);
        }
        for (int t = threadIdx.x; t < D * D; t += blockDim.x) {
            const int qy = t / D - Ri, qx = t % D - Ri;
            wts[t] = R - sqrtf((float)(qx * qx + qy * qy + dz * dz));  // used inside the sphere only
        }
        __syncthreads();
        for (int dy = -Ri; dy <= Ri; ++dy) {
            const float ry2 = rz2 - (float)(dy * dy);
            if (ry2 <= 0.f) continue;  // uniform
            const int dxm = (int)ceilf(sqrtf(ry2)) - 1;  // dx^2 < ry2
            const float2* row = tile + (ty + Ri + dy) * W + (tx + Ri);
            const float* wrow = wts + (dy + Ri) * D + Ri;
            for (int dx = -dxm; dx <= dxm; ++dx) {
                const float w = wrow[dx];
                const float2 v = row[dx];
                num = fmaf(w, v.x, num);
                den = fmaf(w, v.y, den);
            }
        }
    }
    if (i < nx && j < ny) {
        const long long n = ((long long)k * ny + j) * nx + i;
        const float rt = num / den;
        rho_t[n] = rt;
        wsum[n] = den;
        rho_b[n] = (tbe + tanhf(beta * (rt - eta))) * inv_den;
    }
}

__global__ __launch_bounds__(256) void voxel_filter_grad_kernel(const double* __restrict__ g_b,
                                                                  const float* __restrict__ rho_t,
                                                                  const float* __restrict__ wsum, double* g,
                                                                  int nx, int ny, int nz, float R, int Ri,
                                                                  double beta, double eta, double inv_den)
{
    __shared__ double tile[kTW * kTW];
    __shared__ float wts[(2 * kMaxRi + 1) * (2 * kMaxRi + 1)];  // cone weights of one z offset
    const int tx = threadIdx.x % kFT, ty = threadIdx.x / kFT;
    const int i = blockIdx.x * kFT + tx, j = blockIdx.y * kFT + ty, k = blockIdx.z;
    const int W = kFT + 2 * Ri, D = 2 * Ri + 1;
    const int gx0 = blockIdx.x * kFT - Ri, gy0 = blockIdx.y * kFT - Ri;
    double acc = 0.0;
    for (int dz = -Ri; dz <= Ri; ++dz) {
        const int kk = k + dz;
        const float rz2 = R * R - (float)(dz * dz);
        if (kk < 0 || kk >= nz || rz2 <= 0.f) continue;  // uniform
        __syncthreads();
        for (int t = threadIdx.x; t < W * W; t += blockDim.x) {
            const int ly = t / W, lx = t - ly * W;
            const int gx = gx0 + lx, gy = gy0 + ly;
            double v = 0.0;
            if (gx >= 0 && gx < nx && gy >= 0 && gy < ny) {
                const long long m = ((long long)kk * ny + gy) * nx + gx;
                const double th = tanh(beta * ((double)rho_t[m] - eta));
                v = g_b[m] * (beta * (1.0 - th * th) * inv_den) / (double)wsum[m];
            }
            tile[t] = v;
        }
        for (int t = threadIdx.x; t < D * D; t += blockDim.x) {
            const int qy = t / D - Ri, qx = t % D - Ri;
            wts[t] = R - sqrtf((float)(qx * qx + qy * qy + dz * dz));
        }
        __syncthreads();
        for (int dy = -Ri; dy <= Ri; ++dy) {
            const float ry2 = rz2 - (float)(dy * dy);
            if (ry2 <= 0.f) continue;  // uniform
            const int dxm = (int)ceilf(sqrtf(ry2)) - 1;
            const double* row = tile + (ty + Ri + dy) * W + (tx + Ri);
            const float* wrow = wts + (dy + Ri) * D + Ri;
            for (int dx = -dxm; dx <= dxm; ++dx) acc = fma((double)wrow[dx], row[dx], acc);
        }
    }
    if (i < nx && j < ny) g[((long long)k * ny + j) * nx + i] = acc;
}

// Per edge with one output a thread, where 32 x 32 tiles stay mostly empty or the
// sphere holds few taps (one_output); one launch per output component.  Per input
// component: the sum over its taps around the output tile; 'stage'
// fills the tile (one LDS word per position, zero outside b's edges) and
// 'tap' consumes one staged word with its weight.  Offsets and weights are
// uniform across the workgroup: each z offset's cone weights (zero outside
// the sphere) are tabulated once in LDS (wts, (2H+1)^2 words) while the
// tile is staged, so a tap costs two LDS reads and the accumulation.
template <typename Stage, typename Tap>
__device__ __forceinline__ void edge_taps(int a, int b, const FilterGeom& g, int k, float R, float R2, int H,
                                          float* wts, Stage stage, Tap tap)
{
    const int tx = threadIdx.x % kFT, ty = threadIdx.x / kFT;
    const float sx = 0.5f * ((b == 0) - (a == 0)), sy = 0.5f * ((b == 1) - (a == 1)),
                sz = 0.5f * ((b == 2) - (a == 2));
    const int W = kFT + 2 * H, D = 2 * H + 1;
    for (int dz = -H; dz <= H; ++dz) {
        const int kk = k + dz;
        const float fz = (float)dz + sz;
        const float rz2 = R2 - fz * fz;
        if (kk < 0 || kk >= g.shp[b][2] || rz2 <= 0.f) continue;  // uniform
        __syncthreads();
        stage(kk, W);
        for (int t = threadIdx.x; t < D * D; t += blockDim.x) {
            const int qy = t / D, qx = t - qy * D;
            const float fx = (float)(qx - H) + sx, fy = (float)(qy - H) + sy;
            const float d2 = fx * fx + fy * fy + fz * fz;
            wts[t] = d2 < R2 ? R - sqrtf(d2) : 0.f;
        }
        __syncthreads();
        for (int dy = -H; dy <= H; ++dy) {
            const float fy = (float)dy + sy;
            const float ry2 = rz2 - fy * fy;
            if (ry2 <= 0.f) continue;  // uniform
            const float rr = sqrtf(ry2);
            const int dxl = max(-H, (int)floorf(-sx - rr)), dxh = min(H, (int)ceilf(-sx + rr));
            const int rowb = (ty + H + dy) * W + (tx + H);
            const float* wrow = wts + (dy + H) * D + H;
            for (int dx = dxl; dx <= dxh; ++dx) tap(rowb + dx, wrow[dx]);  // zero weight outside the sphere
        }
    }
}

__global__ __launch_bounds__(256) void edge_filter_project_kernel(const float* __restrict__ rho, float* rho_t,
                                                                  float* rho_b, float* wsum, const FilterGeom g,
                                                                  int a, float R, float R2, int H, float beta,
                                                                  float eta, float tbe, float inv_den)
{
    __shared__ float2 tile[kTWE * kTWE];  // (density, 1) on an edge of b, (0, 0) elsewhere
    __shared__ float wts[(2 * kMaxH + 1) * (2 * kMaxH + 1)];
    const int tx = threadIdx.x % kFT, ty = threadIdx.x / kFT;
    const int i = blockIdx.x * kFT + tx, j = blockIdx.y * kFT + ty, k = blockIdx.z;
    const int gx0 = blockIdx.x * kFT - H, gy0 = blockIdx.y * kFT - H;
    float num = 0.f, den = 0.f;
    for (int b = 0; b < 3; ++b) {
        const int bx = g.shp[b][0], by = g.shp[b][1];
        const float* src = rho + g.off[b];
        auto stage = [&](int kk, int W) {
            for (int t = threadIdx.x; t < W * W; t += blockDim.x) {
                const int ly = t / W, lx = t - ly * W;
                const int gx = gx0 + lx, gy = gy0 + ly;
                const bool in = gx >= 0 && gx < bx && gy >= 0 && gy < by;
                tile[t] = in ? make_float2(src[((long long)kk * by + gy) * bx + gx], 1.f) : make_float2(0.f, 0.f);
            }
        };
        auto tap = [&](int idx, float w) {
            const float2 v = tile[idx];
            num = fmaf(w, v.x, num);
            den = fmaf(w, v.y, den);
        };
        edge_taps(a, b, g, k, R, R2, H, wts, stage, tap);
    }
    if (i < g.shp[a][0] && j < g.shp[a][1]) {
        const long long n = g.off[a] + ((long long)k * g.shp[a][1] + j) * g.shp[a][0] + i;
        const float rt = num / den;
        rho_t[n] = rt;
        wsum[n] = den;
        rho_b[n] = (tbe + tanhf(beta * (rt - eta))) * inv_den;
    }
}

__global__ __launch_bounds__(256) void edge_filter_project_grad_kernel(const double* __restrict__ g_b,
                                                                       const float* __restrict__ rho_t,
                                                                       const float* __restrict__ wsum, double* gout,
                                                                       const FilterGeom g, int a, float R, float R2,
                                                                       int H, double beta, double eta,
                                                                       double inv_den)
{
    __shared__ double tile[kTWE * kTWE];  // v = dF/drho_b * drho_b/drho_t / W on an edge of b, 0 elsewhere
    __shared__ float wts[(2 * kMaxH + 1) * (2 * kMaxH + 1)];
    const int tx = threadIdx.x % kFT, ty = threadIdx.x / kFT;
    const int i = blockIdx.x * kFT + tx, j = blockIdx.y * kFT + ty, k = blockIdx.z;
    const int gx0 = blockIdx.x * kFT - H, gy0 = blockIdx.y * kFT - H;
    double acc = 0.0;
    for (int b = 0; b < 3; ++b) {
        const int bx = g.shp[b][0], by = g.shp[b][1];
        const long long ob = g.off[b];
        auto stage = [&](int kk, int W) {
            for (int t = threadIdx.x; t < W * W; t += blockDim.x) {
                const int ly = t / W, lx = t - ly * W;
                const int gx = gx0 + lx, gy = gy0 + ly;
                double v = 0.0;
                if (gx >= 0 && gx < bx && gy >= 0 && gy < by) {
                    const long long m = ob + ((long long)kk * by + gy) * bx + gx;
                    const double th = tanh(beta * ((double)rho_t[m] - eta));
                    v = g_b[m] * (beta * (1.0 - th * th) * inv_den) / (double)wsum[m];
                }
                tile[t] = v;
            }
        };
        auto tap = [&](int idx, float w) { acc = fma((double)w, tile[idx], acc); };
        edge_taps(a, b, g, k, R, R2, H, wts, stage, tap);
    }
    if (i < g.shp[a][0] && j < g.shp[a][1]) gout[g.off[a] + ((long long)k * g.shp[a][1] + j) * g.shp[a][0] + i] = acc;
}

// Eq. MeasureOfNon-discretness: one workgroup, fixed summation order (lanes,
// wave shuffles, then LDS), so the result does not depend on the launch.  One
// CU's loads bound it (64 bytes a clock): 16-byte loads, four in flight a lane
// (160x160x80 voxels: 586 us with one 4-byte load at a time, 168 us now);
// unaligned input takes the same values in the same order by 4-byte loads.
__device__ __forceinline__ double nd_term(float r) { return 4.0 * (double)r * (1.0 - (double)r); }

__global__ __launch_bounds__(1024) void nondiscreteness_kernel(const float* __restrict__ rb, long long n, double* out)
{
    __shared__ double part[16];
    constexpr int kU = 4;
    double s[kU] = {0.0, 0.0, 0.0, 0.0};
    const bool aligned = (reinterpret_cast<uintptr_t>(rb) & 15) == 0;
    const long long n4 = n / 4, step = (long long)kU * blockDim.x;
    for (long long t = threadIdx.x; t < n4; t += step) {
        float4 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const long long q = t + (long long)u * blockDim.x;
            v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (q < n4) {
                if (aligned) v[u] = reinterpret_cast<const float4*>(rb)[q];
                else v[u] = make_float4(rb[4 * q], rb[4 * q + 1], rb[4 * q + 2], rb[4 * q + 3]);
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) s[u] += (nd_term(v[u].x) + nd_term(v[u].y)) + (nd_term(v[u].z) + nd_term(v[u].w));
    }
    const long long r = 4 * n4 + threadIdx.x;
    if (r < n) s[0] += nd_term(rb[r]);
    double sum = (s[0] + s[1]) + (s[2] + s[3]);
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) tot += part[w];
        out[0] = tot / (double)n * 100.0;
    }
}

bool edge_dims_ok(const int* d)
{
    return d && d[0] >= 1 && d[1] >= 1 && d[2] >= 1 && d[2] + 1 <= 65535;
}

bool dims_ok(const int* d)
{
    return d && d[0] >= 1 && d[1] >= 1 && d[2] >= 1 && d[2] <= 65535;
}

int radius_to_offsets(double R)
{
    // largest integer offset with |d| < R
    return (int)std::ceil(R) - 1;
}

// Launch of the filter kernels: geometry, grid, workgroup and LDS.
struct FilterPlan {
    FilterGeom g;
    dim3 grid;
    unsigned threads;
    size_t lds;
};

FilterPlan plan_filter(const int* d, bool edges, int H, int P, int Q, size_t word, int threads)
{
    FilterPlan L{};
    FilterGeom& g = L.g;
    g.nc = edges ? 3 : 1;
    g.H = H;
    g.W = kTX + 2 * H + 8;  // a block of 8 past a run's end reads up to 8 columns more
    while (g.W % 8 != 1) ++g.W;
    L.threads = (unsigned)threads;
    g.rows = threads * P / kTX;
    int mx = 0, my = 0, z = 0;
    long long o = 0;
    for (int c = 0; c < g.nc; ++c) {
        long long n = 1;
        for (int l = 0; l < 3; ++l) {
            g.shp[c][l] = d[l] + (edges && l != c ? 1 : 0);
            n *= g.shp[c][l];
        }
        g.off[c] = o;
        o += n;
        g.zb[c] = z;
        z += (g.shp[c][2] + Q - 1) / Q;
        mx = std::max(mx, g.shp[c][0]);
        my = std::max(my, g.shp[c][1]);
    }
    g.zb[g.nc] = z;
    g.nbx = (mx + kTX - 1) / kTX;
    g.nby = (my + g.rows - 1) / g.rows;
    L.grid = dim3((unsigned)((long long)g.nbx * g.nby * z));
    L.lds = (size_t)(g.rows + 2 * H) * g.W * word + (size_t)table_words(H) * 4;
    return L;
}

template <int P, bool EDGE>
void launch_filter(const float* rho, float* rho_t, float* rho_b, float* wsum, const int* dims, double radius,
                   double beta, double eta, int threads, hipStream_t stream)
{
    const int H = EDGE ? (int)std::ceil(radius) : radius_to_offsets(radius);
    const double den = std::tanh(beta * eta) + std::tanh(beta * (1.0 - eta));
    const float R = (float)radius, R2 = EDGE ? (float)(radius * radius) : R * R;
    const FilterPlan L = plan_filter(dims, EDGE, H, P, 1, sizeof(float), threads);
    hipLaunchKernelGGL((filter_project_kernel<P, EDGE>), L.grid, dim3(L.threads), L.lds, stream, rho, rho_t, rho_b,
                       wsum, L.g, R, R2, (float)beta, (float)eta, (float)std::tanh(beta * eta), (float)(1.0 / den));
}

template <int P, int Q, bool EDGE>
void launch_filter_grad(const double* g_b, const float* rho_t, const float* wsum, double* g, const int* dims,
                        double radius, double beta, double eta, int threads, hipStream_t stream)
{
    const int H = EDGE ? (int)std::ceil(radius) : radius_to_offsets(radius);
    const double den = std::tanh(beta * eta) + std::tanh(beta * (1.0 - eta));
    const float R = (float)radius, R2 = EDGE ? (float)(radius * radius) : R * R;
    const FilterPlan L = plan_filter(dims, EDGE, H, P, Q, sizeof(double), threads);
    hipLaunchKernelGGL((filter_project_grad_kernel<P, Q, EDGE>), L.grid, dim3(L.threads), L.lds, stream, g_b, rho_t,
                       wsum, g, L.g, R, R2, beta, eta, 1.0 / den);
}

// Tiles of e x e outputs of all output planes.
long long filter_tiles(const int* d, bool edges, int e = 32)
{
    const int x = d[0] + (edges ? 1 : 0), y = d[1] + (edges ? 1 : 0);
    return (long long)((x + e - 1) / e) * ((y + e - 1) / e) * (edges ? 3LL * d[2] + 2 : d[2]);
}

// Whether one output a thread in 16 x 16 tiles is faster than 4 or 8 in 32 x 32 ones.
// Those need enough tiles to fill the chip, tiles that are not mostly empty (q: 16 x 16
// tiles of the outputs per 32 x 32 tile, 4 where all are full) and a sphere large
// enough that the taps and not the staging are the work.  Timed on 520 grids a
// kernel (us, one output / several):
//  - voxels forward: too few tiles 100x25x100 R 3 24 / 38, 33x65x31 R 4.3 33 / 50; empty
//    10x10x2000 (q 1) R 5 0.74 to 1, 14x200x300 (1.9) R 3 / 4 0.93, 1.02; small spheres
//    48x48x800 (2.25) R 2 / 3 0.77, 1.01, 300x300x40 (3.6) R 1.2 / 2 1.00, 1.17, all of
//    them R 1 (a voxel reads only itself: 300x300x40 21 / 42);
//  - voxels chain rule: 24^3 45 / 55 but 100x25x100 R 3 45 / 34; 16x16x1000 (1) 0.82,
//    14x100x100 (1.75) R 3 0.85, 33x33x1000 (2.25) R 2 / 3 0.99, 1.20;
//  - per edge, where three components share the staging, only empty tiles and the
//    smallest spheres: forward 8x8x1200 (1) R 3 180 / 257, 10x10x300 1.30, 14x200x300 R
//    1.5 / 2 0.82, 1.03, 33x33x1000 R 1.5 0.92; chain rule 8x8x1200 262 / 396, 14x100x100
//    R 1.5 / 2 0.82, 1.06, 200x10x100 1.11.
bool one_output(const int* d, double radius, bool edges, bool grad)
{
    const long long tiles = filter_tiles(d, edges), full = filter_tiles(d, edges, kFT);
    const double q = (double)full / (double)tiles;
    if (!edges && radius <= 1.0) return true;
    if (d[1] >= 65535 * kFT) return false;  // (rows beyond the 16 x 16 tiles' grid)
    if (edges) {
        const int x = d[0] + 1;  // a half-empty last tile along x only: 1 to 1.5
        const bool narrow = 2 * ((x + kFT - 1) / kFT) <= 3 * ((x + 31) / 32);
        if (q < 1.5) return (double)tiles >= (!grad && radius < 1.75 ? 700.0 : 1000.0 + 250.0 * radius);
        if (grad) return radius < 1.75 && tiles >= 1024 && q < 2.4 && narrow;
        return radius < (x <= kFT ? 2.25 : 1.75) && tiles >= 800 && q < 2.6;
    }
    if (grad) return tiles < 300 || q < 1.75 || (q < 2.5 && full < 1300) || (radius <= 2.0 && q >= 2.0 && q < 2.5);
    if (tiles < 1024 || q < 1.75) return true;
    if (radius <= 2.0) return radius < 1.3 || q < 3.0 || tiles < 1800;
    return full < (radius <= 3.0 ? 4500 : radius <= 5.0 ? 3800 : 2500);
}

// Grid of 16 x 16 output tiles of every plane.
dim3 tiles16(const int* d)
{
    return dim3((unsigned)((d[0] + kFT - 1) / kFT), (unsigned)((d[1] + kFT - 1) / kFT), (unsigned)d[2]);
}

// 8 outputs a thread and two waves a workgroup where the tiles fill the chip,
// 4 and four waves below (per edge, us: 100x25x100, 1204 tiles, R = 3 / 7.5: 142 / 807
// and 164 / 890; 24^3, 74 tiles, R = 2 / 5: 61 / 256 and 52 / 221).
template <bool EDGE>
ccpr_status run_filter(const float* rho, float* rho_t, float* rho_b, float* wsum, const int* dims, double radius,
                       double beta, double eta, void* hip_stream)
{
    hipStream_t s = (hipStream_t)hip_stream;
    if (one_output(dims, radius, EDGE, false)) {
        const double den = std::tanh(beta * eta) + std::tanh(beta * (1.0 - eta));
        const float R = (float)radius, b = (float)beta, e = (float)eta, tbe = (float)std::tanh(beta * eta),
                    inv = (float)(1.0 / den);
        if constexpr (EDGE) {
            const int H = (int)std::ceil(radius);
            const FilterGeom g = plan_filter(dims, true, H, 1, 1, sizeof(float), kFT * kFT).g;
            for (int a = 0; a < 3; ++a)
                hipLaunchKernelGGL(edge_filter_project_kernel, tiles16(g.shp[a]), dim3(kFT * kFT), 0, s, rho, rho_t, rho_b,
                                   wsum, g, a, R, (float)(radius * radius), H, b, e, tbe, inv);
        } else {
            hipLaunchKernelGGL(voxel_filter_kernel, tiles16(dims), dim3(kFT * kFT), 0, s, rho, rho_t, rho_b, wsum,
                               dims[0], dims[1], dims[2], R, radius_to_offsets(radius), b, e, tbe, inv);
        }
    } else if (!EDGE || filter_tiles(dims, EDGE) >= 1024) {
        launch_filter<8, EDGE>(rho, rho_t, rho_b, wsum, dims, radius, beta, eta, 128, s);
    } else if constexpr (EDGE) {
        launch_filter<4, true>(rho, rho_t, rho_b, wsum, dims, radius, beta, eta, 256, s);
    }
    return hipGetLastError() == hipSuccess ? CCPR_OK : CCPR_EDEVICE;
}

// Two planes a workgroup where that leaves enough of them: v is then formed
// once for both (160x160x80 at R = 12 1735 -> 1432 us).
template <bool EDGE>
ccpr_status run_filter_grad(const double* g_b, const float* rho_t, const float* wsum, double* g, const int* dims,
                            double radius, double beta, double eta, void* hip_stream)
{
    hipStream_t s = (hipStream_t)hip_stream;
    const long long tiles = filter_tiles(dims, EDGE);
    if (one_output(dims, radius, EDGE, true)) {
        const double inv = 1.0 / (std::tanh(beta * eta) + std::tanh(beta * (1.0 - eta)));
        const float R = (float)radius;
        if constexpr (EDGE) {
            const int H = (int)std::ceil(radius);
            const FilterGeom geo = plan_filter(dims, true, H, 1, 1, sizeof(double), kFT * kFT).g;
            for (int a = 0; a < 3; ++a)
                hipLaunchKernelGGL(edge_filter_project_grad_kernel, tiles16(geo.shp[a]), dim3(kFT * kFT), 0, s, g_b, rho_t,
                                   wsum, g, geo, a, R, (float)(radius * radius), H, beta, eta, inv);
        } else {
            hipLaunchKernelGGL(voxel_filter_grad_kernel, tiles16(dims), dim3(kFT * kFT), 0, s, g_b, rho_t, wsum, g,
                               dims[0], dims[1], dims[2], R, radius_to_offsets(radius), beta, eta, inv);
        }
    } else if (tiles >= 1536) {
        launch_filter_grad<8, 2, EDGE>(g_b, rho_t, wsum, g, dims, radius, beta, eta, 128, s);
    } else if (tiles >= 1024) {
        launch_filter_grad<8, 1, EDGE>(g_b, rho_t, wsum, g, dims, radius, beta, eta, 128, s);
    } else {
        launch_filter_grad<4, 1, EDGE>(g_b, rho_t, wsum, g, dims, radius, beta, eta, 256, s);
    }
    return hipGetLastError() == hipSuccess ? CCPR_OK : CCPR_EDEVICE;
}

}  // namespace

extern "C" {

ccpr_status ccpr_filter_project(const float* rho, float* rho_filtered, float* rho_projected, float* weight_sum,
                                const int dims[3], double radius, double beta, double eta, void* hip_stream)
{
    if (!rho || !rho_filtered || !rho_projected || !weight_sum || !dims_ok(dims)) return CCPR_EINVAL;
    if (!(radius >= 1.0 && radius <= 17.0) || !(beta > 0) || !(eta >= 0 && eta <= 1)) return CCPR_EINVAL;
    return run_filter<false>(rho, rho_filtered, rho_projected, weight_sum, dims, radius, beta, eta, hip_stream);
}

ccpr_status ccpr_filter_project_grad(const double* dF_dprojected, const float* rho_filtered, const float* weight_sum,
                                     double* dF_drho, const int dims[3], double radius, double beta, double eta,
                                     void* hip_stream)
{
    if (!dF_dprojected || !rho_filtered || !weight_sum || !dF_drho || !dims_ok(dims)) return CCPR_EINVAL;
    if (!(radius >= 1.0 && radius <= 17.0) || !(beta > 0) || !(eta >= 0 && eta <= 1)) return CCPR_EINVAL;
    return run_filter_grad<false>(dF_dprojected, rho_filtered, weight_sum, dF_drho, dims, radius, beta, eta,
                                  hip_stream);
}

ccpr_status ccpr_filter_project_edges(const float* rho, float* rho_filtered, float* rho_projected,
                                      float* weight_sum, const int dims[3], double radius, double beta, double eta,
                                      void* hip_stream)
{
    if (!rho || !rho_filtered || !rho_projected || !weight_sum || !edge_dims_ok(dims)) return CCPR_EINVAL;
    if (!(radius >= 1.0 && radius <= 17.0) || !(beta > 0) || !(eta >= 0 && eta <= 1)) return CCPR_EINVAL;
    return run_filter<true>(rho, rho_filtered, rho_projected, weight_sum, dims, radius, beta, eta, hip_stream);
}

ccpr_status ccpr_filter_project_grad_edges(const double* dF_dprojected, const float* rho_filtered,
                                           const float* weight_sum, double* dF_drho, const int dims[3], double radius,
                                           double beta, double eta, void* hip_stream)
{
    if (!dF_dprojected || !rho_filtered || !weight_sum || !dF_drho || !edge_dims_ok(dims)) return CCPR_EINVAL;
    if (!(radius >= 1.0 && radius <= 17.0) || !(beta > 0) || !(eta >= 0 && eta <= 1)) return CCPR_EINVAL;
    return run_filter_grad<true>(dF_dprojected, rho_filtered, weight_sum, dF_drho, dims, radius, beta, eta, hip_stream);
}

ccpr_status ccpr_nondiscreteness(const float* rho_projected, long long n, double* out, void* hip_stream)
{
    if (!rho_projected || !out || n < 1) return CCPR_EINVAL;
    hipLaunchKernelGGL(nondiscreteness_kernel, dim3(1), dim3(1024), 0, (hipStream_t)hip_stream, rho_projected, n,
                       out);
    return hipGetLastError() == hipSuccess ? CCPR_OK : CCPR_EDEVICE;
}

}  // extern "C"
