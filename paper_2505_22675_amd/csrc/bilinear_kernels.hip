// Bilinear (Sec. III-A) and Catmull-Rom bicubic (Sec. III-B) resampling of
// one grid onto another.
//
// The source index coordinate of a node is computed in FP64 with the same
// operations, in the same order, as its definition (no contraction), so the
// corner choice is exact; the blend itself is FP32 in lerp form (top, bottom, then vertical),
// which keeps constants exact and lets a NaN corner propagate: a hole.
#include "resample_axis.hpp"

#include <algorithm>
#include <climits>
#include <cmath>

namespace auv {

namespace {

struct BilArgs {
    const float *src;
    float *dst;
    double sx0, sy0, sdx, sdy;
    double dx0, dy0, ddx, ddy;
    int snx, sny, dnx, dny;
    int rows;  // destination rows per block
};

// Patch of a block in a 1-D launch of ncb x nrb patches (row-major: column
// band fastest).  Blocks are dealt round-robin to the 8 XCDs; each XCD takes
// a contiguous run of patches, so it writes whole destination rows instead of
// one column band of every row.
__device__ inline void patch_of(int ncb, int nrb, int *bx, int *by)
{
    const int total = ncb * nrb;
    const int b = (int)blockIdx.x;
    const int xcd = b & 7, q = total >> 3, rem = total & 7;
    const int t = xcd * q + min(xcd, rem) + (b >> 3);
    *bx = t % ncb;
    *by = t / ncb;
}

// Both resamplers: one thread per destination column walks down the rows of its
// block, keeping in registers the source rows that its nodes lie between, each
// already interpolated along x; a row is computed when it enters the window.
// The stores of a wave are whole lines whatever the row length.  The block's
// source rectangle is staged in LDS where it fits.
constexpr int kCols = 256;    // destination columns per block (one per thread)
constexpr int kRows = 32;     // destination rows per block, at most (a lane each)
constexpr int kStage = 5120;  // source values staged in LDS, at most

// The source rectangle that a block reads and where it is: staged in LDS
// (kStaged) or the source grid itself.
template <bool kStaged>
struct Rect {
    const float *src;
    int il, jl, pitch;

    // value at source row j and a column that column() gave
    __device__ __forceinline__ float at(int j, int c) const
    {
        if constexpr (kStaged)
            return src[(j - jl) * pitch + c];
        else
            return src[(int64_t)j * pitch + c];
    }
    __device__ __forceinline__ int column(int i) const { return kStaged ? i - il : i; }
};

// Stages source rows [jl, jl + sh) x columns [il, il + sw): a wave takes every
// fourth row, four of them in flight.
__device__ __forceinline__ void stage_rows(const BilArgs &p, int jl, int sh, int il, int sw,
                                           float *s_src)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = (int)threadIdx.x & 63;
    for (int j = wave; j < sh; j += 16) {
        for (int c = lane; c < sw; c += 64) {
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[k] = p.src[(int64_t)(jl + min(j + 4 * k, sh - 1)) * p.snx + (il + c)];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (j + 4 * k < sh)
                    s_src[(j + 4 * k) * sw + c] = v[k];
        }
    }
}

// Bilinear resample: two source rows in the window, one lerp along y per node.
// Bound by the stores on large grids.  Kernel times on an MI355X, four columns
// per thread with 16-byte stores and up to eight staged groups of 8 rows per
// block / this form: 4096^2 to 8192^2 85 / 54 us (6.2 TB/s), 1501 x 1300 to
// 3199 x 2500 25 / 12, 3000^2 to 3001 x 2999 46 / 20, 60^2 to 150^2 7.5 / 3.7.
template <bool kStaged>
__global__ __launch_bounds__(kCols) void k_bilinear(const BilArgs p)
{
    extern __shared__ float s_src[];
    __shared__ float s_row[kRows];  // fraction of each row
    __shared__ int s_edge[2];
    int pbx, pby;
    patch_of((p.dnx + kCols - 1) / kCols, (p.dny + p.rows - 1) / p.rows, &pbx, &pby);
    const int col = pbx * kCols + (int)threadIdx.x, row0 = pby * p.rows;
    const int nrow = min(p.rows, p.dny - row0);
    const bool on = col < p.dnx;
    // columns past the grid repeat the last one and store nothing (every lane
    // stays active: the rows' table is read across lanes)
    const Axis ax = axis_of(p.dx0, p.ddx, min(col, p.dnx - 1), p.sx0, p.sdx, p.snx);
    int j0_l;  // lane r of every wave: source row of row r
    {
        const int r = min((int)threadIdx.x & 63, nrow - 1);
        const Axis a = axis_of(p.dy0, p.ddy, row0 + r, p.sy0, p.sdy, p.sny);
        j0_l = a.i0;
        if ((int)threadIdx.x < nrow)
            s_row[threadIdx.x] = a.t;
    }
    auto row_j0 = [&](int r) { return __builtin_amdgcn_readlane(j0_l, r); };
    Rect<kStaged> rc{p.src, 0, 0, p.snx};
    if constexpr (kStaged) {
        if (threadIdx.x == 0)
            s_edge[0] = ax.i0;
        if (threadIdx.x == kCols - 1)
            s_edge[1] = ax.i1;
        __syncthreads();
        const int sw = s_edge[1] - s_edge[0] + 1;
        rc = Rect<kStaged>{s_src, s_edge[0], row_j0(0), sw};
        stage_rows(p, rc.jl, min(row_j0(nrow - 1) + 1, p.sny - 1) - rc.jl + 1, rc.il, sw, s_src);
    }
    __syncthreads();
    const int c0 = rc.column(ax.i0), c1 = rc.column(ax.i1);
    // source row j at this thread's column
    auto hrow = [&](int j) {
        const float q0 = rc.at(j, c0), q1 = rc.at(j, c1);
        return q0 + ax.t * (q1 - q0);
    };
    float top = 0.0f, bot = 0.0f;
    int cur = INT_MIN;  // source row of `top`
    float *out = p.dst + (int64_t)row0 * p.dnx + min(col, p.dnx - 1);
#pragma unroll 1
    for (int r = 0; r < nrow; ++r) {
        const int j0 = row_j0(r);
        const float s = s_row[r];
        if (j0 != cur) {
            top = j0 == cur + 1 ? bot : hrow(j0);
            bot = hrow(min(j0 + 1, p.sny - 1));
            cur = j0;
        }
        const float v = top + s * (bot - top);
        if (on)
            __builtin_nontemporal_store(v, out);  // not re-read by this kernel
        out += p.dnx;
    }
}

// Catmull-Rom cubic (Sec. III-B) at t in [0, 1] between p1 and p2, as p1 plus
// weighted differences from it: the weights of p0, p2 and p3 (p1's makes their
// sum one).  A non-finite tap always gives a non-finite result (0 * inf is NaN).
struct CubW {
    float w0, w2, w3;
};
__device__ inline CubW cubic_weights(float t)
{
    const float u = 1.0f - t;
    return CubW{-0.5f * t * u * u, 0.5f * t * fmaf(t, fmaf(-3.0f, t, 4.0f), 1.0f),
                -0.5f * t * t * u};
}
__device__ inline float cubic(float p0, float p1, float p2, float p3, float w0, float w2, float w3)
{
    return p1 + fmaf(w3, p3 - p1, fmaf(w2, p2 - p1, w0 * (p0 - p1)));
}

// Catmull-Rom resample.  Taps are the source indices i0 - 1 .. i0 + 2 (clamped
// to the grid) around each node's cell; the cubic runs along x on the 4 tap
// rows, then along y.  The cubic is separable: walking down its column, a
// thread keeps the horizontal cubics of the 4 current tap rows in registers and
// computes a tap row's cubic only when the row enters the window, so each node
// costs one vertical cubic (7 operations; the rows' weights come from LDS).  A
// node with a non-finite tap takes the bilinear value of its 4 inner taps, NaN
// when one of them is NaN: a hole.
//
// Bound by vector instruction issue and the stores.  Four columns per thread
// left a row length that is no multiple of four with stores of 4 bytes at a
// stride of 16, and 8 rows per block paid a block's start (FP64 axis maps, tap
// columns, the first four rows) four times as often.  Kernel times on an
// MI355X, that form with the cubic in Horner form / this form:
// 1501 x 1300 to 3199 x 2500 31.9 / 17.4 us, 2048^2 to 4096^2 29.4 / 24.0, 4096^2
// to 8192^2 114 / 77, 60^2 to 150^2 10.4 / 5.0; error against 64 bits (rms)
// 5.0e-8 / 3.8e-8.
template <bool kStaged>
__global__ __launch_bounds__(kCols) void k_bicubic(const BilArgs p)
{
    extern __shared__ float s_src[];
    __shared__ float4 s_row[kRows];  // weights and fraction of each row
    __shared__ int s_edge[2];
    int pbx, pby;
    patch_of((p.dnx + kCols - 1) / kCols, (p.dny + p.rows - 1) / p.rows, &pbx, &pby);
    const int col = pbx * kCols + (int)threadIdx.x, row0 = pby * p.rows;
    const int nrow = min(p.rows, p.dny - row0);
    const bool on = col < p.dnx;
    // columns past the grid repeat the last one and store nothing (every lane
    // stays active: the rows' table is read across lanes)
    const Axis ax = axis_of(p.dx0, p.ddx, min(col, p.dnx - 1), p.sx0, p.sdx, p.snx);
    int j0_l;  // lane r of every wave: source row of row r
    {
        const int r = min((int)threadIdx.x & 63, nrow - 1);
        const Axis a = axis_of(p.dy0, p.ddy, row0 + r, p.sy0, p.sdy, p.sny);
        j0_l = a.i0;
        if ((int)threadIdx.x < nrow) {
            const CubW w = cubic_weights(a.t);
            s_row[threadIdx.x] = make_float4(w.w0, w.w2, w.w3, a.t);
        }
    }
    auto row_j0 = [&](int r) { return __builtin_amdgcn_readlane(j0_l, r); };
    Rect<kStaged> rc{p.src, 0, 0, p.snx};
    if constexpr (kStaged) {
        // every tap of the patch, clamped to the grid (the maps are monotone)
        if (threadIdx.x == 0)
            s_edge[0] = ax.i0;
        if (threadIdx.x == kCols - 1)
            s_edge[1] = ax.i0;
        __syncthreads();
        const int il = max(s_edge[0] - 1, 0), jl = max(row_j0(0) - 1, 0);
        const int sw = min(s_edge[1] + 2, p.snx - 1) - il + 1;
        rc = Rect<kStaged>{s_src, il, jl, sw};
        stage_rows(p, jl, min(row_j0(nrow - 1) + 2, p.sny - 1) - jl + 1, il, sw, s_src);
    }
    __syncthreads();
    int tc[4];  // tap columns
#pragma unroll
    for (int q = 0; q < 4; ++q)
        tc[q] = rc.column(min(max(ax.i0 - 1 + q, 0), p.snx - 1));
    const CubW wx = cubic_weights(ax.t);
    auto clampr = [&](int j) { return min(max(j, 0), p.sny - 1); };
    auto at = [&](int j, int c) { return rc.at(j, c); };
    // horizontal cubic of source row j at this thread's column
    auto hrow = [&](int j) {
        j = clampr(j);
        return cubic(at(j, tc[0]), at(j, tc[1]), at(j, tc[2]), at(j, tc[3]), wx.w0, wx.w2, wx.w3);
    };
    float h0 = 0.0f, h1 = 0.0f, h2 = 0.0f, h3 = 0.0f;
    int cur = INT_MIN;  // j0 of the rows held in h0..h3
    float *out = p.dst + (int64_t)row0 * p.dnx + min(col, p.dnx - 1);
#pragma unroll 1
    for (int r = 0; r < nrow; ++r) {
        const int j0 = row_j0(r);
        const float4 w = s_row[r];
        if (j0 == cur + 1) {
            h0 = h1;
            h1 = h2;
            h2 = h3;
            h3 = hrow(j0 + 2);
        } else if (j0 != cur) {
            h0 = hrow(j0 - 1);
            h1 = hrow(j0);
            h2 = hrow(j0 + 1);
            h3 = hrow(j0 + 2);
        }
        cur = j0;
        float v = cubic(h0, h1, h2, h3, w.x, w.y, w.z);
        if (!isfinite(v)) {
            // bilinear on the inner taps (the corners of the node's cell)
            const int ja = clampr(j0), jb = clampr(j0 + 1);
            const float q00 = at(ja, tc[1]), q10 = at(ja, tc[2]);
            const float q01 = at(jb, tc[1]), q11 = at(jb, tc[2]);
            const float top = q00 + ax.t * (q10 - q00);
            const float bot = q01 + ax.t * (q11 - q01);
            v = top + w.w * (bot - top);
        }
        if (on)
            __builtin_nontemporal_store(v, out);  // not re-read by this kernel
        out += p.dnx;
    }
}

// Launch geometry: rows per block and the LDS of the rectangle (`halo` source
// rows and columns beyond the nodes' extent, slack for the rounding of the axis
// maps included, see axis_maps_fine); 0 bytes: read from memory.  More rows share a block's start,
// but a small grid needs the blocks (halved, down to 8, while under 2048, eight
// to a CU), and the rectangle has to fit kStage values, which leave eight
// blocks to a CU.
size_t resample_geometry(const auv_grid_desc &s, const auv_grid_desc &d, double halo, int *rows,
                         unsigned *blocks)
{
    const int64_t ncb = (d.nx + kCols - 1) / kCols;
    int n = kRows;
    while (n > 8 && ncb * ((d.ny + n - 1) / n) < 2048)
        n /= 2;
    const double sw = std::min((double)s.nx, std::ceil((kCols - 1) * d.dx / s.dx) + halo);
    auto rect = [&](int k) {
        return sw * std::min((double)s.ny, std::ceil((k - 1) * d.dy / s.dy) + halo);
    };
    while (n > 8 && rect(n) > kStage)
        n /= 2;
    *rows = n;
    *blocks = (unsigned)(ncb * ((d.ny + n - 1) / n));
    return rect(n) <= kStage && axis_maps_fine(s, d) ? sizeof(float) * (size_t)rect(n) : 0;
}

BilArgs resample_args(const float *src, const auv_grid_desc &s, float *dst,
                      const auv_grid_desc &d)
{
    BilArgs p;
    p.src = src;
    p.dst = dst;
    p.sx0 = s.x0;
    p.sy0 = s.y0;
    p.sdx = s.dx;
    p.sdy = s.dy;
    p.dx0 = d.x0;
    p.dy0 = d.y0;
    p.ddx = d.dx;
    p.ddy = d.dy;
    p.snx = s.nx;
    p.sny = s.ny;
    p.dnx = d.nx;
    p.dny = d.ny;
    return p;
}

}  // namespace

auv_status launch_bicubic(const float *src, const auv_grid_desc &s, float *dst,
                          const auv_grid_desc &d, hipStream_t st)
{
    BilArgs p = resample_args(src, s, dst, d);
    unsigned blocks;
    const size_t lds = resample_geometry(s, d, 6.0, &p.rows, &blocks);
    if (lds > 0)
        k_bicubic<true><<<blocks, kCols, lds, st>>>(p);
    else
        k_bicubic<false><<<blocks, kCols, 0, st>>>(p);
    AUV_HIP(hipGetLastError());
    return AUV_OK;
}

auv_status launch_bilinear(const float *src, const auv_grid_desc &s, float *dst,
                           const auv_grid_desc &d, hipStream_t st)
{
    BilArgs p = resample_args(src, s, dst, d);
    unsigned blocks;
    const size_t lds = resample_geometry(s, d, 4.0, &p.rows, &blocks);
    if (lds > 0)
        k_bilinear<true><<<blocks, kCols, lds, st>>>(p);
    else
        k_bilinear<false><<<blocks, kCols, 0, st>>>(p);
    AUV_HIP(hipGetLastError());
    return AUV_OK;
}

}  // namespace auv
