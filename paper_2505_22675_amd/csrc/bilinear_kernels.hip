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
    int groups;  // k_bilinear: row groups per block (1 .. kBilGroups); k_bicubic: rows per block
};

constexpr int kBilThreads = 256;
constexpr int kBilCols = kBilThreads * 4;  // destination columns per block
constexpr int kBilRows = 8;                // destination rows per block
constexpr int kBilStage = 6144;            // source values staged in LDS

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

// One block owns a 1024-column band of p.groups row groups of 8 rows each:
// up to kBilGroups while the launch keeps at least 1024 blocks (at cfg2 2x, 2,
// 4, 8 and 16 groups gave 73, 70, 68 and 104 us), one when the rectangles
// are too large to stage (then there is nothing to prefetch).
// The FP64 axis maps of its columns are computed once into LDS, those of its
// rows likewise; each row group's source rectangle is staged into LDS when it
// fits (otherwise corners are gathered from global memory), and the next
// group's rectangle is loaded into registers while the current group is
// blended and stored, so the reads' latency hides behind the stores.  Every
// thread produces four consecutive nodes per row with one 16-byte streaming
// store.
constexpr int kBilGroups = 8;  // row groups per block, at most
constexpr int kBilPf = 12;     // prefetched values per thread (rectangles up to 3072 values)

__global__ __launch_bounds__(kBilThreads) void k_bilinear(BilArgs p)
{
    __shared__ int s_i0[kBilCols], s_i1[kBilCols];
    __shared__ float s_t[kBilCols];
    __shared__ int s_j0[kBilGroups * kBilRows], s_j1[kBilGroups * kBilRows];
    __shared__ float s_s[kBilGroups * kBilRows];
    __shared__ float s_src[kBilStage];
    const int ngroups = (p.dny + kBilRows - 1) / kBilRows;
    int pbx, pby;
    patch_of((p.dnx + kBilCols - 1) / kBilCols, (ngroups + p.groups - 1) / p.groups, &pbx,
             &pby);
    const int col0 = pbx * kBilCols;
    const int g0 = pby * p.groups;               // first row group of the block
    const int ng = min(p.groups, ngroups - g0);  // row groups of the block
    const int ncol = min(kBilCols, p.dnx - col0);
    for (int c = threadIdx.x; c < kBilCols; c += kBilThreads) {
        const Axis a = axis_of(p.dx0, p.ddx, min(col0 + c, p.dnx - 1), p.sx0, p.sdx, p.snx);
        s_i0[c] = a.i0;
        s_i1[c] = a.i1;
        s_t[c] = a.t;
    }
    if (threadIdx.x < p.groups * kBilRows) {
        const int row = min(g0 * kBilRows + (int)threadIdx.x, p.dny - 1);
        const Axis a = axis_of(p.dy0, p.ddy, row, p.sy0, p.sdy, p.sny);
        s_j0[threadIdx.x] = a.i0;
        s_j1[threadIdx.x] = a.i1;
        s_s[threadIdx.x] = a.t;
    }
    __syncthreads();
    // source columns read by the band (the maps are monotone)
    const int il = s_i0[0], ih = s_i1[ncol - 1];
    const int sw = ih - il + 1;
    // source rows (first, count) of row group g
    auto rows_of = [&](int g) {
        const int nrow = min(kBilRows, p.dny - (g0 + g) * kBilRows);
        const int jl = s_j0[g * kBilRows];
        return make_int2(jl, s_j1[g * kBilRows + nrow - 1] - jl + 1);
    };
    // this thread's share of a rectangle: element e = threadIdx.x + k
    // kBilThreads at (row e / sw, column e % sw), walked incrementally
    float pf[kBilPf];
    auto fetch = [&](int jl, int sh) {
        const int n = sw * sh;
        const int t = (int)threadIdx.x;
        if (t >= n)
            return;
        int r = t / sw, cc = t - r * sw;
        const int dr = kBilThreads / sw, dc = kBilThreads - dr * sw;
        const float *row = p.src + (int64_t)(jl + r) * p.snx + il;
#pragma unroll
        for (int k = 0; k < kBilPf; ++k) {
            if (t + k * kBilThreads < n)
                pf[k] = row[cc];
            cc += dc;
            int step = dr;
            if (cc >= sw) {
                cc -= sw;
                ++step;
            }
            row += (int64_t)step * p.snx;
        }
    };
    auto place = [&](int sh) {
        const int n = sw * sh;
#pragma unroll
        for (int k = 0; k < kBilPf; ++k) {
            const int e = (int)threadIdx.x + k * kBilThreads;
            if (e < n)
                s_src[e] = pf[k];
        }
    };
    const int c = threadIdx.x * 4;
    int i0[4], i1[4];
    float t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        i0[k] = s_i0[min(c + k, kBilCols - 1)];
        i1[k] = s_i1[min(c + k, kBilCols - 1)];
        t[k] = s_t[min(c + k, kBilCols - 1)];
    }
    const bool vec = c + 4 <= ncol && (p.dnx & 3) == 0 &&
                     (reinterpret_cast<uintptr_t>(p.dst) & 15) == 0;
    int2 rc = rows_of(0);
    bool staged = (long long)sw * rc.y <= kBilStage;
    if (staged)
        stage_rect(p.src, p.snx, rc.x, il, sw, rc.y, s_src, kBilThreads);
    __syncthreads();
    for (int g = 0; g < ng; ++g) {
        const int2 nx = g + 1 < ng ? rows_of(g + 1) : make_int2(0, 0);
        const bool nstaged = g + 1 < ng && (long long)sw * nx.y <= kBilStage;
        // small rectangles (2x upsampling: about 2600 values) are loaded into
        // registers now and land in LDS after this group's stores
        const bool pref = nstaged && sw * nx.y <= kBilThreads * kBilPf;
        if (pref)
            fetch(nx.x, nx.y);
        const int row0 = (g0 + g) * kBilRows;
        const int nrow = min(kBilRows, p.dny - row0);
        const int jl = rc.x;
        if (c < ncol) {
            for (int r = 0; r < nrow; ++r) {
                const int q = g * kBilRows + r;
                const float s = s_s[q];
                float v[4];
                if (staged) {
                    const float *r0 = s_src + (s_j0[q] - jl) * sw - il;
                    const float *r1 = s_src + (s_j1[q] - jl) * sw - il;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float q00 = r0[i0[k]], q10 = r0[i1[k]];
                        const float q01 = r1[i0[k]], q11 = r1[i1[k]];
                        const float top = q00 + t[k] * (q10 - q00);
                        const float bot = q01 + t[k] * (q11 - q01);
                        v[k] = top + s * (bot - top);
                    }
                } else {
                    const float *r0 = p.src + (int64_t)s_j0[q] * p.snx;
                    const float *r1 = p.src + (int64_t)s_j1[q] * p.snx;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float q00 = r0[i0[k]], q10 = r0[i1[k]];
                        const float q01 = r1[i0[k]], q11 = r1[i1[k]];
                        const float top = q00 + t[k] * (q10 - q00);
                        const float bot = q01 + t[k] * (q11 - q01);
                        v[k] = top + s * (bot - top);
                    }
                }
                float *out = p.dst + (int64_t)(row0 + r) * p.dnx + col0 + c;
                if (vec) {
                    // streaming store: the destination is not re-read by this kernel
                    typedef float f4v __attribute__((ext_vector_type(4)));
                    const f4v vv = {v[0], v[1], v[2], v[3]};
                    __builtin_nontemporal_store(vv, reinterpret_cast<f4v *>(out));
                } else {
                    for (int k = 0; k < 4 && c + k < ncol; ++k)
                        out[k] = v[k];
                }
            }
        }
        __syncthreads();  // every read of this group's rectangle is done
        if (pref)
            place(nx.y);
        else if (nstaged)
            stage_rect(p.src, p.snx, nx.x, il, sw, nx.y, s_src, kBilThreads);
        __syncthreads();
        rc = nx;
        staged = nstaged;
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

constexpr int kCubCols = 256;   // destination columns per block (one per thread)
constexpr int kCubRows = 32;    // destination rows per block, at most (a lane each)
constexpr int kCubStage = 5120; // source values staged in LDS, at most

// Catmull-Rom resample.  Taps are the source indices i0 - 1 .. i0 + 2 (clamped
// to the grid) around each node's cell; the cubic runs along x on the 4 tap
// rows, then along y.  The cubic is separable: walking down its column, a
// thread keeps the horizontal cubics of the 4 current tap rows in registers and
// computes a tap row's cubic only when the row enters the window, so each node
// costs one vertical cubic (7 operations; the rows' weights come from LDS).  A
// node with a non-finite tap takes the bilinear value of its 4 inner taps, NaN
// when one of them is NaN: a hole.
//
// One column per thread: the stores of a wave are whole lines whatever the row
// length (four columns per thread left a row length that is no multiple of four
// with stores of 4 bytes at a stride of 16), and the start of a block (FP64 axis
// maps, tap columns, the first four rows) is paid once per 32 rows instead of
// 8.  Bound by vector instruction issue and the stores.  Kernel times on an
// MI355X, four columns per thread and the cubic in Horner form / this form:
// 1501 x 1300 to 3199 x 2500 31.9 / 17.4 us, 2048^2 to 4096^2 29.4 / 24.0, 4096^2
// to 8192^2 114 / 77, 60^2 to 150^2 10.4 / 5.0; error against 64 bits (rms)
// 5.0e-8 / 3.8e-8.
template <bool kStaged>
__global__ __launch_bounds__(kCubCols) void k_bicubic(const BilArgs p)
{
    extern __shared__ float s_src[];
    __shared__ float4 s_row[kCubRows];  // weights and fraction of each row
    __shared__ int s_edge[2];
    const int nrb = (p.dny + p.groups - 1) / p.groups;  // groups: rows per block
    int pbx, pby;
    patch_of((p.dnx + kCubCols - 1) / kCubCols, nrb, &pbx, &pby);
    const int col = pbx * kCubCols + (int)threadIdx.x, row0 = pby * p.groups;
    const int nrow = min(p.groups, p.dny - row0);
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
    int il = 0, jl = 0, sw = 0;
    if constexpr (kStaged) {
        // source rectangle of every tap of the patch, clamped to the grid (the
        // maps are monotone), four rows of a wave in flight
        if (threadIdx.x == 0)
            s_edge[0] = ax.i0;
        if (threadIdx.x == kCubCols - 1)
            s_edge[1] = ax.i0;
        __syncthreads();
        il = max(s_edge[0] - 1, 0);
        sw = min(s_edge[1] + 2, p.snx - 1) - il + 1;
        jl = max(row_j0(0) - 1, 0);
        const int sh = min(row_j0(nrow - 1) + 2, p.sny - 1) - jl + 1;
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
    __syncthreads();
    int tc[4];  // tap columns (relative to the rectangle, or absolute)
#pragma unroll
    for (int q = 0; q < 4; ++q)
        tc[q] = min(max(ax.i0 - 1 + q, 0), p.snx - 1) - il;
    const CubW wx = cubic_weights(ax.t);
    auto clampr = [&](int j) { return min(max(j, 0), p.sny - 1); };
    auto at = [&](int j, int c) {
        if constexpr (kStaged)
            return s_src[(j - jl) * sw + c];
        else
            return p.src[(int64_t)j * p.snx + c];
    };
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

}  // namespace

auv_status launch_bicubic(const float *src, const auv_grid_desc &s, float *dst,
                          const auv_grid_desc &d, hipStream_t st)
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
    // rows per block: more of them share a block's start, but a small grid needs
    // the blocks (halved, down to 8, while under 2048, eight to a CU), and the source
    // rectangle has to fit kCubStage values, which leave eight blocks to a CU
    // (two rows and columns of slack for the rounding of the axis maps); a
    // rectangle too large at 8 rows is read from memory instead
    const int64_t ncb = (d.nx + kCubCols - 1) / kCubCols;
    int rows = kCubRows;
    while (rows > 8 && ncb * ((d.ny + rows - 1) / rows) < 2048)
        rows /= 2;
    const double sw = std::min((double)s.nx, std::ceil((kCubCols - 1) * d.dx / s.dx) + 6.0);
    auto rect = [&](int n) {
        return sw * std::min((double)s.ny, std::ceil((n - 1) * d.dy / s.dy) + 6.0);
    };
    while (rows > 8 && rect(rows) > kCubStage)
        rows /= 2;
    p.groups = rows;
    const unsigned grid = (unsigned)(ncb * ((d.ny + rows - 1) / rows));
    if (rect(rows) <= kCubStage)
        k_bicubic<true><<<grid, kCubCols, sizeof(float) * (size_t)rect(rows), st>>>(p);
    else
        k_bicubic<false><<<grid, kCubCols, 0, st>>>(p);
    AUV_HIP(hipGetLastError());
    return AUV_OK;
}

auv_status launch_bilinear(const float *src, const auv_grid_desc &s, float *dst,
                           const auv_grid_desc &d, hipStream_t st)
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
    const int ngroups = (d.ny + kBilRows - 1) / kBilRows;
    const int64_t ncb = (d.nx + kBilCols - 1) / kBilCols;
    // a row group's source rectangle, roughly: several groups per block only
    // pay when it is staged (the next one is prefetched meanwhile)
    const double rect = (kBilCols * d.dx / s.dx + 2.0) * (kBilRows * d.dy / s.dy + 2.0);
    p.groups = rect > kBilStage
                   ? 1
                   : (int)std::max<int64_t>(1, std::min<int64_t>(kBilGroups,
                                                                 ncb * ngroups / 1024));
    const unsigned grid = (unsigned)(ncb * ((ngroups + p.groups - 1) / p.groups));
    k_bilinear<<<grid, kBilThreads, 0, st>>>(p);
    AUV_HIP(hipGetLastError());
    return AUV_OK;
}

}  // namespace auv
