// Ordinary kriging resample of one grid onto another (Sec. III-C).
//
// A destination node maps to the source index coordinate u (as in the
// bilinear resample); its neighbourhood is the 5 x 5 source nodes centred on
// the node nearest to u, moved inward at the grid edges.  The weights solve
// the ordinary-kriging system
//     [ G  1 ] [ lambda ]   [ g ]
//     [ 1' 0 ] [   mu   ] = [ 1 ]
// with G the variogram between the 25 nodes, g the variogram between each node
// and the destination point and gamma(h) = 1 - exp(-h / a) (the sill cancels
// from the weights).  K = [G 1; 1' 0] depends only on the node spacing and the
// range, not on where the window sits, so it is inverted once on the host
// (FP64, Gauss-Jordan with partial pivoting) and, written as
//     z = z_c + sum_j g_j w_j,   w = K^-1 (z - z_c, 0)
// (z_c: the window centre; K is symmetric), w depends only on the window: a
// thread walking down a column computes it once per window and each node adds
// one 26-term product.
//
// K commutes with the mirror images of the window in x and in y, so in the
// basis of sums and differences of mirrored nodes (per axis: a0+a4, a1+a3,
// a2 | a0-a4, a1-a3) its inverse is block diagonal, with blocks for the four
// parity classes (even/odd in y, even/odd in x) of 10 (with the unbiasedness
// row), 6, 6 and 4 rows: w costs 178 multiply-adds and two 40-add transforms
// instead of 650 multiply-adds.  A window with a non-finite value falls back to
// bilinear.
#include "resample_axis.hpp"

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstring>
#include <mutex>
#include <type_traits>

namespace auv {

namespace {

constexpr int kKrigCols = 256;    // destination columns per block (one per thread)
constexpr int kKrigRows = 32;     // destination rows per block, at most
constexpr int kKrigStage = 6144;  // source values staged in LDS
constexpr int kBlockFloats = 10 * 9 + 6 * 6 + 6 * 6 + 4 * 4;
constexpr double kMaxRangeSpacings = 1e4;  // the FP64 inverse stays well conditioned

struct KrigArgs {
    const float *src;
    float *dst;
    double sx0, sy0, sdx, sdy;
    double dx0, dy0, ddx, ddy;
    int snx, sny, dnx, dny;
    float fdx, fdy;  // source spacing
    float c2;        // (log2(e) / range)^2, or (1 / range)^2 for the series form
    int rows;        // destination rows per block (8 .. kKrigRows)
    // the diagonal blocks of K^-1 in the mirror basis, row-major: even-even
    // 10 x 9 (rows: 9 nodes and the unbiasedness entry; its column is never
    // used since the data vector has a zero there), even-odd 6 x 6, odd-even
    // 6 x 6, odd-odd 4 x 4
    float mb[kBlockFloats];
};

using cfloat = const __attribute__((address_space(4))) float;

// First index of the 5-node window centred on the node nearest to u.
__device__ inline int window_start(double u, int n)
{
    const int c = (int)floor(u + 0.5);
    return min(max(c - 2, 0), n - 5);
}

// 1 - exp(-t) from t = h / range (kSeries: Taylor series to t^7, t <= 1/4) or
// from t log2(e).
template <bool kSeries>
__device__ __forceinline__ float one_minus_exp(float t)
{
    if constexpr (kSeries) {
        // t (1 - t/2 (1 - t/3 (... (1 - t/7))))
        float g = fmaf(-t, 1.0f / 7.0f, 1.0f);
        g = fmaf(-t * (1.0f / 6.0f), g, 1.0f);
        g = fmaf(-t * (1.0f / 5.0f), g, 1.0f);
        g = fmaf(-t * (1.0f / 4.0f), g, 1.0f);
        g = fmaf(-t * (1.0f / 3.0f), g, 1.0f);
        g = fmaf(-t * 0.5f, g, 1.0f);
        return t * g;
    } else {
        return 1.0f - __builtin_amdgcn_exp2f(-t);
    }
}

// Mirror transform of a window per row (x), then per column (y); component
// order per axis: sums 0+4, 1+3, 2 | differences 0-4, 1-3.
__device__ __forceinline__ void mirror(float (&d)[25])
{
    float t[25];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        t[k * 5 + 0] = d[k * 5 + 0] + d[k * 5 + 4];
        t[k * 5 + 1] = d[k * 5 + 1] + d[k * 5 + 3];
        t[k * 5 + 2] = d[k * 5 + 2];
        t[k * 5 + 3] = d[k * 5 + 0] - d[k * 5 + 4];
        t[k * 5 + 4] = d[k * 5 + 1] - d[k * 5 + 3];
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        d[0 * 5 + i] = t[0 * 5 + i] + t[4 * 5 + i];
        d[1 * 5 + i] = t[1 * 5 + i] + t[3 * 5 + i];
        d[2 * 5 + i] = t[2 * 5 + i];
        d[3 * 5 + i] = t[0 * 5 + i] - t[4 * 5 + i];
        d[4 * 5 + i] = t[1 * 5 + i] - t[3 * 5 + i];
    }
}

// Back to nodes: transpose of the mirror transform, y then x.
__device__ __forceinline__ void mirror_back(const float (&u)[25], float (&w)[25])
{
    float t[25];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        t[0 * 5 + i] = u[0 * 5 + i] + u[3 * 5 + i];
        t[4 * 5 + i] = u[0 * 5 + i] - u[3 * 5 + i];
        t[1 * 5 + i] = u[1 * 5 + i] + u[4 * 5 + i];
        t[3 * 5 + i] = u[1 * 5 + i] - u[4 * 5 + i];
        t[2 * 5 + i] = u[2 * 5 + i];
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        w[k * 5 + 0] = t[k * 5 + 0] + t[k * 5 + 3];
        w[k * 5 + 4] = t[k * 5 + 0] - t[k * 5 + 3];
        w[k * 5 + 1] = t[k * 5 + 1] + t[k * 5 + 4];
        w[k * 5 + 3] = t[k * 5 + 1] - t[k * 5 + 4];
        w[k * 5 + 2] = t[k * 5 + 2];
    }
}

// K^-1 (v, unbias) in the mirror basis, in place, for an unbiasedness entry of
// 1 or 0; `last` gets the product's unbiasedness entry (without the part that
// the entry 1 itself would add).  The blocks are read from the argument segment
// through scalar loads: an opaque pointer keeps the 178 values from being held
// in registers across the caller's loop.
__device__ __forceinline__ void inverse_blocks(float (&v)[25], bool unbias, float &last)
{
    cfloat *mb = (cfloat *)((const __attribute__((address_space(4))) char *)
                                __builtin_amdgcn_kernarg_segment_ptr() +
                            offsetof(KrigArgs, mb));
    asm volatile("" : "+s"(mb));
    float u[25];
    // even-even: y components 0..2, x components 0..2, then the unbiasedness
    // row (the inverse is symmetric: that row is its column too)
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        float acc = unbias && r < 9 ? mb[90 - 9 + r] : 0.0f;
#pragma unroll
        for (int c = 0; c < 9; ++c)
            acc = fmaf(mb[r * 9 + c], v[(c / 3) * 5 + c % 3], acc);
        if (r < 9)
            u[(r / 3) * 5 + r % 3] = acc;
        else
            last = acc;
    }
    // even-odd: y 0..2, x 3..4
#pragma unroll
    for (int r = 0; r < 6; ++r) {
        float acc = 0.0f;
#pragma unroll
        for (int c = 0; c < 6; ++c)
            acc = fmaf(mb[90 + r * 6 + c], v[(c / 2) * 5 + 3 + c % 2], acc);
        u[(r / 2) * 5 + 3 + r % 2] = acc;
    }
    // odd-even: y 3..4, x 0..2
#pragma unroll
    for (int r = 0; r < 6; ++r) {
        float acc = 0.0f;
#pragma unroll
        for (int c = 0; c < 6; ++c)
            acc = fmaf(mb[126 + r * 6 + c], v[(3 + c / 3) * 5 + c % 3], acc);
        u[(3 + r / 3) * 5 + r % 3] = acc;
    }
    // odd-odd: y 3..4, x 3..4
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float acc = 0.0f;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            acc = fmaf(mb[162 + r * 4 + c], v[(3 + c / 2) * 5 + 3 + c % 2], acc);
        u[(3 + r / 2) * 5 + 3 + r % 2] = acc;
    }
#pragma unroll
    for (int q = 0; q < 25; ++q)
        v[q] = u[q];
}

// The inverse of the kriging matrix K = [G 1; 1' 0] splits as [A b; b' c]
// with 1'A = 0 and 1'b = 1 (the weights A g + b sum to one for any g).  For
// w = K^-1 (z - z_c, 0), sum_q w_q = 0, so with g_q = 1 - e_q,
// e_q = exp(-h_q / range):
//     z = z_c + sum_q g_q w_q + w_25 = z_c + w_25 - sum_q e_q w_q.
// The entries of A grow with range / spacing while g shrinks, so the FP32
// rounding of e_q (about 6e-8 near 1) times w_q grows with the range: the
// exp form is kept to ranges under 16 hypot(dx, dy) (22.6 spacings on a
// square grid; relative depth error of a few 1e-6).  A window node lies at
// most 4 spacings per axis from the destination point (2.5 inside the grid,
// 4 where the window is moved in at an edge), so from there on every t =
// h / range is at most 1/4 and kSeries evaluates g_q = 1 - exp(-t) by its
// Taylor series to t^7 (truncation under 2e-9 relative), whose rounding is
// relative to g_q itself, and sums z = z_c + w_25 + sum_q g_q w_q.
template <bool kSeries>
__global__ __launch_bounds__(kKrigCols) void k_kriging(const KrigArgs p)
{
    __shared__ int s_wx[kKrigCols], s_i0[kKrigCols], s_i1[kKrigCols];
    __shared__ float s_du[kKrigCols], s_t[kKrigCols];
    __shared__ int s_wy[kKrigRows], s_j0[kKrigRows], s_j1[kKrigRows];
    __shared__ float s_dv[kKrigRows], s_s[kKrigRows];
    __shared__ float s_src[kKrigStage];
    const int col0 = blockIdx.x * kKrigCols;
    const int row0 = blockIdx.y * p.rows;
    const int ncol = min(kKrigCols, p.dnx - col0);
    const int nrow = min(p.rows, p.dny - row0);
    {
        const int c = threadIdx.x;
        const Axis a = axis_of(p.dx0, p.ddx, min(col0 + c, p.dnx - 1), p.sx0, p.sdx, p.snx);
        const int wx = window_start(a.u, p.snx);
        s_wx[c] = wx;
        s_du[c] = (float)(a.u - wx);
        s_i0[c] = a.i0;
        s_i1[c] = a.i1;
        s_t[c] = a.t;
    }
    if (threadIdx.x < p.rows) {
        const int r = threadIdx.x;
        const Axis a = axis_of(p.dy0, p.ddy, min(row0 + r, p.dny - 1), p.sy0, p.sdy, p.sny);
        const int wy = window_start(a.u, p.sny);
        s_wy[r] = wy;
        s_dv[r] = (float)(a.u - wy);
        s_j0[r] = a.i0;
        s_j1[r] = a.i1;
        s_s[r] = a.t;
    }
    __syncthreads();
    // source rectangle of every window of the patch (window starts are
    // monotone); the bilinear corners of a node lie inside its window
    const int il = s_wx[0], ih = s_wx[ncol - 1] + 4;
    const int jl = s_wy[0], jh = s_wy[nrow - 1] + 4;
    const int sw = ih - il + 1, sh = jh - jl + 1;
    const bool staged = (long long)sw * sh <= kKrigStage;
    if (staged) {
        stage_rect(p.src, p.snx, jl, il, sw, sh, s_src, kKrigCols);
        __syncthreads();
    }
    const int c = threadIdx.x;
    if (c >= ncol)
        return;
    // separate instantiations keep LDS and global reads apart (a value that
    // may come from either would make every read a flat load)
    auto walk = [&](auto staged_t) {
        constexpr bool kStaged = decltype(staged_t)::value;
        auto at = [&](int j, int i) {  // source value at row j, column i
            if constexpr (kStaged)
                return s_src[(j - jl) * sw + (i - il)];
            else
                return p.src[(int64_t)j * p.snx + i];
        };
        const int wx = s_wx[c];
        // squared x offsets to the window columns, scaled by (log2(e) / range)^2
        float ex2[5];
        {
            const float du = s_du[c];
    #pragma unroll
            for (int i = 0; i < 5; ++i) {
                const float e = ((float)i - du) * p.fdx;
                ex2[i] = e * e * p.c2;
            }
        }
        // the node's 25 covariance terms depend only on its offsets in the
        // window: x is fixed for the thread's column and rows cycle through a
        // few y offsets (two at a 2x resample), so the terms of the last two
        // offsets are kept and reused when a row's offset recurs
        float ca[25], cb[25];
        float dva = NAN, dvb = NAN;
        bool fill_a = true;
        auto terms = [&](float (&e)[25], float dv) {
    #pragma unroll
            for (int k = 0; k < 5; ++k) {
                const float ey = ((float)k - dv) * p.fdy;
                const float ey2 = ey * ey * p.c2;
    #pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const float t = __builtin_amdgcn_sqrtf(ex2[i] + ey2);
                    if constexpr (kSeries)
                        e[k * 5 + i] = one_minus_exp<true>(t);
                    else
                        e[k * 5 + i] = __builtin_amdgcn_exp2f(-t);
                }
            }
        };
        float w[25], w25 = 0.0f;
        auto dot = [&](const float (&e)[25]) {
            float acc = 0.0f;
    #pragma unroll
            for (int q = 0; q < 25; ++q)
                acc = fmaf(e[q], w[q], acc);
            return acc;
        };
        float zc = 0.0f;
        bool bad = false;
        int cur = -1;  // window row start of w (the same for every thread of the block)
        for (int r = 0; r < nrow; ++r) {
            const int wy = s_wy[r];
            if (wy != cur) {
                float dz[25];
                zc = at(wy + 2, wx + 2);
                bad = false;
    #pragma unroll
                for (int q = 0; q < 25; ++q) {
                    const float z = at(wy + q / 5, wx + q % 5);
                    bad |= !isfinite(z);
                    dz[q] = z - zc;
                }
                mirror(dz);
                inverse_blocks(dz, false, w25);
                mirror_back(dz, w);
                cur = wy;
            }
            float v;
            if (bad) {
                // a non-finite neighbour: bilinear on the node's cell corners
                const int i0 = s_i0[c], i1 = s_i1[c], j0 = s_j0[r], j1 = s_j1[r];
                const float t = s_t[c], s = s_s[r];
                const float q00 = at(j0, i0), q10 = at(j0, i1);
                const float q01 = at(j1, i0), q11 = at(j1, i1);
                const float top = q00 + t * (q10 - q00);
                const float bot = q01 + t * (q11 - q01);
                v = top + s * (bot - top);
            } else {
                const float dv = s_dv[r];
                float acc;
                if (dv == dva) {
                    acc = dot(ca);
                } else if (dv == dvb) {
                    acc = dot(cb);
                } else if (fill_a) {
                    terms(ca, dv);
                    dva = dv;
                    fill_a = false;
                    acc = dot(ca);
                } else {
                    terms(cb, dv);
                    dvb = dv;
                    fill_a = true;
                    acc = dot(cb);
                }
                v = kSeries ? zc + (w25 + acc) : zc + (w25 - acc);
            }
            p.dst[(int64_t)(row0 + r) * p.dnx + col0 + c] = v;
        }
    };
    if (staged)
        walk(std::true_type{});
    else
        walk(std::false_type{});
}

// The same resample where the destination rows repeat at most two y offsets
// (spacing equal to the source's, or half of it): the kriging weights
//     lambda = A g + b,   z = z_c + sum_q lambda_q (z_q - z_c)
// depend on a node's offsets in its window alone, so a thread walking down a
// column keeps the weights of its last two y offsets in registers (K^-1 is
// applied to the covariance terms once per offset instead of to every window),
// and a node costs 25 multiply-adds.  The thread's 5 x 5 window slides in
// registers (its rows take turns in the array, so nothing is moved); its next
// row comes from the block's source rectangle in LDS (a load from memory inside
// the row loop would wait for the loop's stores, which the same counter
// covers), and lane r of a wave holds row r's offset.
//
// Bound by vector instruction issue (60 % of it at four waves per SIMD; half of
// the rest is the start of each block: source rectangle, then weights).  2048^2
// to 4096^2 on an MI355X: the other form 98.9 us, this one 54.9; 25 loads per
// window instead of sliding, or the window moved in registers, 71; 32 rows per
// block 59, 128 rows 83 (two waves per SIMD).  Error against 64 bits at ranges of
// 0.5 to 9000 spacings: largest 0.8e-7 relative (the other form: 2.3e-7).
constexpr int kPhaseRows = 64;     // destination rows per block, at most (a lane each)
constexpr int kPhaseStage = 9984;  // source values staged in LDS, at most

// Bilinear value of a node on its cell's corners.
__device__ __forceinline__ float krig_bilinear(const KrigArgs &p, const Axis &ax, int row)
{
    const Axis ay = axis_of(p.dy0, p.ddy, row, p.sy0, p.sdy, p.sny);
    const float *const r0 = p.src + (int64_t)ay.i0 * p.snx;
    const float *const r1 = p.src + (int64_t)ay.i1 * p.snx;
    const float q00 = r0[ax.i0], q10 = r0[ax.i1];
    const float q01 = r1[ax.i0], q11 = r1[ax.i1];
    const float top = q00 + ax.t * (q10 - q00);
    const float bot = q01 + ax.t * (q11 - q01);
    return top + ay.t * (bot - top);
}

template <bool kSeries>
__global__ __launch_bounds__(kKrigCols, 4) void k_kriging_phase(const KrigArgs p)
{
    extern __shared__ float s_src[];  // the rectangle (launch_kriging sizes it)
    const int row0 = blockIdx.y * p.rows;
    const int nrow = min(p.rows, p.dny - row0);
    // lane r of every wave holds row r's window start and y offset (bits)
    int wy_l, dv_l;
    {
        const Axis a = axis_of(p.dy0, p.ddy, row0 + min((int)threadIdx.x & 63, nrow - 1), p.sy0,
                               p.sdy, p.sny);
        wy_l = window_start(a.u, p.sny);
        dv_l = __float_as_int((float)(a.u - wy_l));
    }
    auto row_window = [&](int r) { return __builtin_amdgcn_readlane(wy_l, r); };
    auto row_offset = [&](int r) { return __builtin_amdgcn_readlane(dv_l, r); };
    const int col0 = blockIdx.x * kKrigCols, col = col0 + (int)threadIdx.x;
    const int last = min(col0 + kKrigCols, p.dnx) - 1;
    const Axis ax = axis_of(p.dx0, p.ddx, min(col, p.dnx - 1), p.sx0, p.sdx, p.snx);
    const int wx = window_start(ax.u, p.snx);
    const int il = window_start(axis_of(p.dx0, p.ddx, col0, p.sx0, p.sdx, p.snx).u, p.snx);
    const int ih = window_start(axis_of(p.dx0, p.ddx, last, p.sx0, p.sdx, p.snx).u, p.snx) + 4;
    const int jl = row_window(0), jh = row_window(nrow - 1) + 4;
    const int sw = ih - il + 1;
    stage_rect(p.src, p.snx, jl, il, sw, jh - jl + 1, s_src, kKrigCols);
    __syncthreads();
    // columns past the grid repeat the last one and store nothing (every lane
    // stays active: the row table is read across lanes)
    const bool on = col < p.dnx;
    float ex2[5];
    {
        const float du = (float)(ax.u - wx);
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const float e = ((float)i - du) * p.fdx;
            ex2[i] = e * e * p.c2;
        }
    }
    // weights of y offset dv
    auto weights = [&](float (&l)[25], float dv) {
        float g[25];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const float ey = ((float)k - dv) * p.fdy;
            const float ey2 = ey * ey * p.c2;
#pragma unroll
            for (int i = 0; i < 5; ++i)
                g[k * 5 + i] = one_minus_exp<kSeries>(__builtin_amdgcn_sqrtf(ex2[i] + ey2));
        }
        mirror(g);
        float one;
        inverse_blocks(g, true, one);
        mirror_back(g, l);
    };
    const float *const src = s_src + (wx - il);
    // Runs of rows that share two offsets.  Both weights are computed before
    // the window is loaded, so that the registers for that are free by then;
    // one run is the rule, edges have a few.
    int r = 0;
#pragma unroll 1
    while (r < nrow) {
        float la[25] = {}, lb[25] = {};
        const int da = row_offset(r);
        int rb = r + 1;
        while (rb < nrow && row_offset(rb) == da)
            ++rb;
        const int db = row_offset(min(rb, nrow - 1));
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int q = 0; q < 25; ++q)
                la[q] = lb[q];
            if (h == 0 || db != da)
                weights(lb, __int_as_float(h == 0 ? da : db));
        }

        int wy = row_window(r);
        float z[5][5];
        auto load_row = [&](int j, float (&to)[5]) {
            const float *const row = src + (min(j, jh) - jl) * sw;
#pragma unroll
            for (int i = 0; i < 5; ++i)
                to[i] = row[i];
        };
#pragma unroll
        for (int k = 0; k < 5; ++k)
            load_row(wy + k, z[k]);
        // The rows of the window whose first source row is z[kFirst], then one
        // source row down (into that row: the window turns in the array).
        // Rows that share a window mostly have one offset each, so both values
        // are computed together.  False after the run's last row.
        auto window = [&](auto first) -> bool {
            constexpr int kFirst = decltype(first)::value;
            const float zc = z[(kFirst + 2) % 5][2];
            float va = 0.0f, vb = 0.0f;
            if (db != da) {
#pragma unroll
                for (int q = 0; q < 25; ++q) {
                    const float d = z[(kFirst + q / 5) % 5][q % 5] - zc;
                    va = fmaf(la[q], d, va);
                    vb = fmaf(lb[q], d, vb);
                }
            } else {
#pragma unroll
                for (int q = 0; q < 25; ++q)
                    vb = fmaf(lb[q], z[(kFirst + q / 5) % 5][q % 5] - zc, vb);
            }
#pragma unroll 1
            for (; r < nrow && row_window(r) == wy; ++r) {
                const int dv = row_offset(r);
                if (dv != da && dv != db)
                    return false;
                float v = zc + (dv == db ? vb : va);
                if (!isfinite(v)) {
                    // a non-finite neighbour: bilinear on the node's cell corners
                    float t = 0.0f;  // NaN with any non-finite value
#pragma unroll
                    for (int q = 0; q < 25; ++q)
                        t = fmaf(z[q / 5][q % 5], 0.0f, t);
                    if (t != 0.0f)
                        v = krig_bilinear(p, ax, row0 + r);
                }
                if (on)
                    __builtin_nontemporal_store(v, p.dst + (int64_t)(row0 + r) * p.dnx + col);
            }
            ++wy;
            load_row(wy + 4, z[kFirst]);
            return r < nrow;
        };
        while (window(std::integral_constant<int, 0>{}) &&
               window(std::integral_constant<int, 1>{}) &&
               window(std::integral_constant<int, 2>{}) &&
               window(std::integral_constant<int, 3>{}) &&
               window(std::integral_constant<int, 4>{})) {
        }
    }
}

// Inverse of the 26 x 26 kriging matrix for node spacing (dx, dy) and range a,
// by Gauss-Jordan elimination with partial pivoting in FP64.
bool kriging_inverse(double dx, double dy, double range, double *out)
{
    constexpr int n = 26;
    double A[n][2 * n];
    for (int pi = 0; pi < 25; ++pi) {
        for (int qi = 0; qi < 25; ++qi) {
            const double h = std::hypot((pi % 5 - qi % 5) * dx, (pi / 5 - qi / 5) * dy);
            A[pi][qi] = -std::expm1(-h / range);
        }
        A[pi][25] = 1.0;
        A[25][pi] = 1.0;
    }
    A[25][25] = 0.0;
    for (int r = 0; r < n; ++r)
        for (int k = 0; k < n; ++k)
            A[r][n + k] = r == k ? 1.0 : 0.0;
    for (int col = 0; col < n; ++col) {
        int piv = col;
        for (int r = col + 1; r < n; ++r)
            if (std::fabs(A[r][col]) > std::fabs(A[piv][col]))
                piv = r;
        if (!(std::fabs(A[piv][col]) > 0.0))
            return false;
        if (piv != col)
            for (int k = 0; k < 2 * n; ++k)
                std::swap(A[piv][k], A[col][k]);
        const double d = A[col][col];
        for (int k = 0; k < 2 * n; ++k)
            A[col][k] /= d;
        for (int r = 0; r < n; ++r) {
            if (r == col || A[r][col] == 0.0)
                continue;
            const double f = A[r][col];
            for (int k = 0; k < 2 * n; ++k)
                A[r][k] -= f * A[col][k];
        }
    }
    for (int r = 0; r < n; ++r)
        for (int k = 0; k < n; ++k)
            out[r * n + k] = A[r][n + k];
    return true;
}

// M = D^-1 T K^-1 T' D^-1 for the mirror transform T (per axis: rows
// a0+a4, a1+a3, a2, a0-a4, a1-a3; the unbiasedness entry kept) and D = T T',
// so that K^-1 = T' M T.  M is block diagonal over the parity classes; its
// blocks are packed as the kernel reads them.  Fails if an entry outside the
// blocks is not negligible (it is zero in exact arithmetic).
bool mirror_blocks(const double *kinv, float *out)
{
    static const double ax[5][5] = {{1, 0, 0, 0, 1},
                                    {0, 1, 0, 1, 0},
                                    {0, 0, 1, 0, 0},
                                    {1, 0, 0, 0, -1},
                                    {0, 1, 0, -1, 0}};
    static const double dax[5] = {2, 2, 1, 2, 2};
    double T[26][26] = {}, Dinv[26];
    for (int ky = 0; ky < 5; ++ky)
        for (int kx = 0; kx < 5; ++kx) {
            for (int k = 0; k < 5; ++k)
                for (int i = 0; i < 5; ++i)
                    T[ky * 5 + kx][k * 5 + i] = ax[ky][k] * ax[kx][i];
            Dinv[ky * 5 + kx] = 1.0 / (dax[ky] * dax[kx]);
        }
    T[25][25] = 1.0;
    Dinv[25] = 1.0;
    double A[26][26], M[26][26];  // A = K^-1 T'
    for (int r = 0; r < 26; ++r)
        for (int c = 0; c < 26; ++c) {
            double acc = 0.0;
            for (int k = 0; k < 26; ++k)
                acc += kinv[r * 26 + k] * T[c][k];
            A[r][c] = acc;
        }
    double big = 0.0;
    for (int r = 0; r < 26; ++r)
        for (int c = 0; c < 26; ++c) {
            double acc = 0.0;
            for (int k = 0; k < 26; ++k)
                acc += T[r][k] * A[k][c];
            M[r][c] = Dinv[r] * acc * Dinv[c];
            big = std::max(big, std::fabs(M[r][c]));
        }
    // parity class of a mirror-basis index: 0 even-even, 1 even-odd,
    // 2 odd-even, 3 odd-odd (the unbiasedness entry is even-even)
    auto cls = [](int q) { return q == 25 ? 0 : 2 * (q / 5 >= 3) + (q % 5 >= 3); };
    for (int r = 0; r < 26; ++r)
        for (int c = 0; c < 26; ++c)
            if (cls(r) != cls(c) && !(std::fabs(M[r][c]) <= 1e-9 * big))
                return false;
    // members of each class in the kernel's order
    int ee[10], eo[6], oe[6], oo[4];
    for (int r = 0; r < 9; ++r)
        ee[r] = (r / 3) * 5 + r % 3;
    ee[9] = 25;
    for (int r = 0; r < 6; ++r) {
        eo[r] = (r / 2) * 5 + 3 + r % 2;
        oe[r] = (3 + r / 3) * 5 + r % 3;
    }
    for (int r = 0; r < 4; ++r)
        oo[r] = (3 + r / 2) * 5 + 3 + r % 2;
    int o = 0;
    for (int r = 0; r < 10; ++r)
        for (int c = 0; c < 9; ++c)
            out[o++] = (float)M[ee[r]][ee[c]];
    for (int r = 0; r < 6; ++r)
        for (int c = 0; c < 6; ++c)
            out[o++] = (float)M[eo[r]][eo[c]];
    for (int r = 0; r < 6; ++r)
        for (int c = 0; c < 6; ++c)
            out[o++] = (float)M[oe[r]][oe[c]];
    for (int r = 0; r < 4; ++r)
        for (int c = 0; c < 4; ++c)
            out[o++] = (float)M[oo[r]][oo[c]];
    return o == kBlockFloats;
}

// The last few inverses, keyed by (dx, dy, range): a resample loop over
// tiles of one survey pays the elimination once.
struct KrigCache {
    std::mutex mu;
    struct Entry {
        double dx, dy, range;
        double kinv[26 * 26];
    } e[8];
    int used = 0, next = 0;
};

bool cached_inverse(double dx, double dy, double range, double *out)
{
    static KrigCache cache;
    {
        std::lock_guard<std::mutex> lk(cache.mu);
        for (int i = 0; i < cache.used; ++i) {
            const KrigCache::Entry &e = cache.e[i];
            if (e.dx == dx && e.dy == dy && e.range == range) {
                std::memcpy(out, e.kinv, sizeof(e.kinv));
                return true;
            }
        }
    }
    if (!kriging_inverse(dx, dy, range, out))
        return false;
    std::lock_guard<std::mutex> lk(cache.mu);
    KrigCache::Entry &e = cache.e[cache.next];
    e.dx = dx;
    e.dy = dy;
    e.range = range;
    std::memcpy(e.kinv, out, sizeof(e.kinv));
    cache.next = (cache.next + 1) % 8;
    cache.used = std::min(cache.used + 1, 8);
    return true;
}

}  // namespace

auv_status launch_kriging(const float *src, const auv_grid_desc &s, float *dst,
                          const auv_grid_desc &d, double range, hipStream_t st)
{
    if (!(range > 0.0) || !std::isfinite(range))
        return fail(AUV_ERR_INVALID, "range must be positive and finite");
    if (s.nx < 5 || s.ny < 5)  // no 5 x 5 neighbourhood: every node is bilinear
        return launch_bilinear(src, s, dst, d, st);
    KrigArgs p;
    std::memset(&p, 0, sizeof(p));
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
    p.fdx = (float)s.dx;
    p.fdy = (float)s.dy;
    // a window node lies at most 4 spacings per axis from the destination
    // point (the point is clamped into the grid, the window moved in at edges)
    const double hmax = 4.0 * std::hypot(s.dx, s.dy);
    const bool series = hmax / range <= 0.25;
    if (range > kMaxRangeSpacings * std::max(s.dx, s.dy))
        return fail(AUV_ERR_RANGE, "kriging range above 1e4 source spacings");
    const double l = (series ? 1.0 : 1.4426950408889634) / range;
    p.c2 = (float)(l * l);
    double kinv[26 * 26];
    if (!cached_inverse(s.dx, s.dy, range, kinv))
        return fail(AUV_ERR_INVALID, "singular kriging system for this spacing and range");
    if (!mirror_blocks(kinv, p.mb))
        return fail(AUV_ERR_INVALID, "kriging inverse lost its mirror symmetry (range far outside the node spacing)");
    // Destination rows at the source's spacing or half of it have one or two y
    // offsets (and a few more at the edges): the form that keeps their weights.
    // Elsewhere every row would compute weights of its own, which costs it as
    // much as a window's product costs the other form, shared by its rows.
    bool phase = (std::fabs(d.dy - s.dy) <= 1e-9 * s.dy ||
                  std::fabs(2.0 * d.dy - s.dy) <= 1e-9 * s.dy) &&
                 axis_maps_fine(s, d);
    // more rows per block reuse more covariance terms or weights, but a small
    // grid needs the blocks: halve (down to 8) while under 1024 blocks
    const int64_t ncb = (d.nx + kKrigCols - 1) / kKrigCols;
    auto block_rows = [&](int rows) {
        while (rows > 8 && ncb * ((d.ny + rows - 1) / rows) < 1024)
            rows /= 2;
        return rows;
    };
    p.rows = block_rows(phase ? kPhaseRows : kKrigRows);
    // and the block's source rectangle has to fit kPhaseStage values, which
    // leave four blocks to a CU (two rows of slack for the rounding of the
    // axis maps); where eight rows do not, the other form takes its own rows
    const double sw = std::min((double)s.nx, std::ceil((kKrigCols - 1) * d.dx / s.dx) + 7.0);
    auto rect = [&](int rows) {
        return sw * std::min((double)s.ny, std::ceil((rows - 1) * d.dy / s.dy) + 7.0);
    };
    while (phase && p.rows > 8 && rect(p.rows) > kPhaseStage)
        p.rows /= 2;
    if (phase) {
        // Eight rows of half the source's spacing use each weight four times: with a
        // rectangle that would not let them be sixteen, that pays only while the
        // launch leaves CUs idle anyway (4000 x 1000 to 1333 x 2000, 1500 blocks, 33.5 us,
        // the other form 27.4; 8000 x 4000 to 2758 x 8000, 162 and 115; 2000 x 1000 to
        // 690 x 2000, 750 blocks, 16.9 and 17.4).  At the source's own spacing eight
        // rows pay: 4000 x 2000 to 2000 x 2000, 33.6 and 48.9.
        const int64_t blocks = ncb * ((d.ny + p.rows - 1) / p.rows);
        const bool few_rows =
            2.0 * d.dy < 1.5 * s.dy && rect(16) > kPhaseStage && blocks > 1024;
        if (rect(p.rows) > kPhaseStage || few_rows) {
            phase = false;
            p.rows = block_rows(kKrigRows);
        }
    }
    const size_t lds = phase ? sizeof(float) * (size_t)rect(p.rows) : 0;
    const dim3 grid((unsigned)ncb, (unsigned)((d.ny + p.rows - 1) / p.rows));
    if (phase && series)
        k_kriging_phase<true><<<grid, kKrigCols, lds, st>>>(p);
    else if (phase)
        k_kriging_phase<false><<<grid, kKrigCols, lds, st>>>(p);
    else if (series)
        k_kriging<true><<<grid, kKrigCols, 0, st>>>(p);
    else
        k_kriging<false><<<grid, kKrigCols, 0, st>>>(p);
    AUV_HIP(hipGetLastError());
    return AUV_OK;
}

}  // namespace auv
