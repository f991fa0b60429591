// Empirical semivariogram of a grid along its axes, and the exponential
// variogram fit that gives kriging (Sec. III-C) its range.
//
//   k_vario_partial  one block per (axis, group of kVLags lags, band of rows or
//                    piece of one):
//                    FP64 sums of the squared differences of the pairs at
//                    those lags with both values finite, and their counts
//   k_vario_final    one block per (axis, lag): the bands' partials summed in
//                    band order
// Every sum runs in a fixed order (no atomics), so the result does not depend
// on timing.  The fit is host arithmetic on a few dozen points.
#include "auv_internal.hpp"

#include <algorithm>
#include <cmath>
#include <vector>

namespace auv {
namespace {

constexpr int kVThreads = 256;
constexpr int kMaxBands = 128;
constexpr int kMaxLags = 1024;

struct VPart {
    double sum;
    long long cnt;
};

__device__ inline void block_sum(double &s, long long &c, VPart *lds)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        s += __shfl_xor(s, d, 64);
        c += __shfl_xor(c, d, 64);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        lds[w] = VPart{s, c};
    __syncthreads();
    if (threadIdx.x == 0) {
        s = 0.0;
        c = 0;
        for (int i = 0; i < kVThreads / 64; ++i) {
            s += lds[i].sum;
            c += lds[i].cnt;
        }
    }
}

constexpr int kVLags = 8;               // lags per block
constexpr int kVRun = 8;                // consecutive values per thread
constexpr int kVWin = kVRun + kVLags - 1;  // their partners at the block's lags
constexpr int kVRowsMax = 16;           // rows a block stages at once (axis 0)

// A value, or NaN where it is not finite (inf * 0 is NaN; a finite value is
// unchanged), so that validity is one unordered test from here on.
__device__ inline float finite_or_nan(float z) { return fmaf(z, 0.0f, z); }

// |d|, or 0 where d is NaN: the maximum of a quiet NaN and a number is the number.
__device__ inline double abs_or_zero(double d)
{
    double r;
    asm("v_max_f64 %0, |%1|, 0" : "=v"(r) : "v"(d));
    return r;
}

// The pairs (za[i], zb[i + l]) of kVRun consecutive values at kVLags lags:
// their squared differences added to s[l], their number to c[l].  64 pairs
// take three FP64 operations each; the partners are converted once for all
// lags and the pairs counted from bit masks, eight to an instruction.
__device__ __forceinline__ void add_pairs(const float (&za)[kVRun], const float (&zb)[kVWin],
                                          double (&s)[kVLags], int (&c)[kVLags])
{
    double da[kVRun], db[kVWin];
    unsigned ma = 0, mb = 0;
#pragma unroll
    for (int i = 0; i < kVRun; ++i) {
        da[i] = (double)za[i];
        ma |= za[i] == za[i] ? 1u << i : 0u;
    }
#pragma unroll
    for (int i = 0; i < kVWin; ++i) {
        db[i] = (double)zb[i];
        mb |= zb[i] == zb[i] ? 1u << i : 0u;
    }
#pragma unroll
    for (int l = 0; l < kVLags; ++l) {
#pragma unroll
        for (int i = 0; i < kVRun; ++i) {
            const double t = abs_or_zero(da[i] - db[i + l]);
            s[l] = fma(t, t, s[l]);
        }
        c[l] += __popc(ma & (mb >> l));
    }
}

// Halves kH values per lane: each lane keeps the sums of one half with the
// lane kD across.
template <int kH, int kD, class T>
__device__ __forceinline__ void halve(T (&v)[kVLags])
{
    const bool up = (threadIdx.x & kD) != 0;
#pragma unroll
    for (int j = 0; j < kH; ++j) {
        const T keep = up ? v[j + kH] : v[j], send = up ? v[j] : v[j + kH];
        v[j] = keep + __shfl_xor(send, kD, 64);
    }
}

// Wave sums of kVLags values: the sum of value 4 b5 + 2 b4 + b3 (bits of the
// lane) is returned.
template <class T>
__device__ __forceinline__ T wave_sums(T (&v)[kVLags])
{
    static_assert(kVLags == 8, "three halvings");
    halve<4, 32>(v);
    halve<2, 16>(v);
    halve<1, 8>(v);
    T r = v[0];
#pragma unroll
    for (int d = 4; d >= 1; d >>= 1)
        r += __shfl_xor(r, d, 64);
    return r;
}

// grid: (bands * splits, ceil(nlags / kVLags), 2 axes).  Band b takes the pairs
// whose first value lies in rows [b * rows, (b + 1) * rows); block b * splits + i of
// them takes the first values of columns [i * cols, (i + 1) * cols) (see splits_for).
//
// Bound by FP64 instruction issue: about 4.8 instructions per pair (three of
// them FP64), each value read once per eight lags instead of once per pair.
// Along x a thread's run is consecutive in a row, read from LDS (padded to 9
// words per run, so that a wave's lanes meet different banks); along y it is
// consecutive in a column, so the lanes read consecutive addresses.  1024^2
// nodes, 64 lags, 134M pairs: 36 us, 3.7e12 pairs/s (one block per lag, one pair
// per two loads, counts by compare: 107 us).
__global__ __launch_bounds__(kVThreads, 4) void k_vario_partial(const float *__restrict__ src,
                                                             int nx, int ny, int nlags, int rows,
                                                             int cols, int splits,
                                                             VPart *__restrict__ part)
{
    __shared__ float s_a[kVThreads * 9], s_b[(kVThreads + kVRowsMax) * 9];
    __shared__ VPart s_sum[kVThreads / 64][kVLags];
    const int band = blockIdx.x / splits, axis = blockIdx.z;
    const int k0 = blockIdx.y * kVLags;  // lags k0 + 1 .. k0 + kVLags
    const int cb = ((int)blockIdx.x - band * splits) * cols, ce = min(nx, cb + cols);
    const int r0 = band * rows, r1 = min(ny, r0 + rows);
    double s[kVLags];
    int c[kVLags];
#pragma unroll
    for (int l = 0; l < kVLags; ++l) {
        s[l] = 0.0;
        c[l] = 0;
    }
    float za[kVRun], zb[kVWin];
    if (axis == 0) {
        // runs per row (at most a block's threads), rows per pass
        const int nch = min(kVThreads, (ce - cb + kVRun - 1) / kVRun);
        const int per = min(kVRowsMax, kVThreads / nch);
        const int rl = threadIdx.x / nch, ch = threadIdx.x - rl * nch;
        float *const pa = s_a + rl * nch * 9, *const pb = s_b + rl * (nch + 1) * 9;
        for (int c0 = cb; c0 < min(ce, nx - 1 - k0); c0 += nch * kVRun) {
            for (int a = r0; a < r1; a += per) {
                // loads beyond the grid read its last row or column instead
                const bool on = rl < per && a + rl < r1;
                const float *const row = src + (size_t)min(a + rl, ny - 1) * nx;
                auto load = [&](int b, int end) {
                    const float z = finite_or_nan(row[min(b, nx - 1)]);
                    return on && b < end ? z : NAN;
                };
                float va[kVRun], vb[kVRun];
#pragma unroll
                for (int j = 0; j < kVRun; ++j) {
                    va[j] = load(c0 + j * nch + ch, ce);
                    vb[j] = load(c0 + 1 + k0 + j * nch + ch, nx);
                }
                __syncthreads();  // the previous pass is read
                if (rl < per) {
#pragma unroll
                    for (int j = 0; j < kVRun; ++j) {
                        const int p = j * nch + ch;
                        pa[p + (p >> 3)] = va[j];
                        pb[p + (p >> 3)] = vb[j];
                    }
                    for (int p = nch * kVRun + ch; p < (nch + 1) * kVRun; p += nch)
                        pb[p + (p >> 3)] = load(c0 + 1 + k0 + p, nx);
                }
                __syncthreads();
                if (on) {
#pragma unroll
                    for (int i = 0; i < kVRun; ++i)
                        za[i] = pa[ch * 9 + i];
#pragma unroll
                    for (int i = 0; i < kVWin; ++i)
                        zb[i] = pb[ch * 9 + i + (i >> 3)];
                    add_pairs(za, zb, s, c);
                }
            }
        }
    } else {
        for (int b = cb + (int)threadIdx.x; b < ce; b += kVThreads) {
            for (int a0 = r0; a0 < min(r1, ny - 1 - k0); a0 += kVRun) {
                // opaque: the rows' addresses and tests are not worth the
                // registers it takes to keep them from one b to the next
                int a = a0;
                asm volatile("" : "+s"(a));
                auto load = [&](int r, int end) {
                    const float *const row = src + (size_t)min(r, ny - 1) * nx;
                    const float z = finite_or_nan(row[(uint32_t)b]);
                    return r < end ? z : NAN;
                };
#pragma unroll
                for (int i = 0; i < kVRun; ++i)
                    za[i] = load(a + i, r1);
#pragma unroll
                for (int i = 0; i < kVWin; ++i)
                    zb[i] = load(a + 1 + k0 + i, ny);
                add_pairs(za, zb, s, c);
            }
        }
    }
    // a thread's pairs fit 32 bits (a 256th of a block's columns times its rows),
    // a wave's of a grid of 1e9 columns do not
    long long cl[kVLags];
#pragma unroll
    for (int l = 0; l < kVLags; ++l)
        cl[l] = c[l];
    const double sum = wave_sums(s);
    const long long cnt = wave_sums(cl);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if ((lane & 7) == 0)
        s_sum[w][lane >> 3] = VPart{sum, cnt};
    __syncthreads();
    const int l = threadIdx.x;
    if (l < kVLags && k0 + l < nlags) {
        VPart t = s_sum[0][l];
        for (int i = 1; i < kVThreads / 64; ++i) {
            t.sum += s_sum[i][l].sum;
            t.cnt += s_sum[i][l].cnt;
        }
        part[((size_t)axis * nlags + k0 + l) * gridDim.x + blockIdx.x] = t;
    }
}

// grid: (nlags * 2): out[axis * nlags + lag] = sum over bands, in band order
// within each thread and in thread order across the block.
__global__ __launch_bounds__(kVThreads) void k_vario_final(const VPart *__restrict__ part,
                                                           int bands, VPart *__restrict__ out)
{
    __shared__ VPart lds[kVThreads / 64];
    const VPart *p = part + (size_t)blockIdx.x * bands;
    double s = 0.0;
    long long c = 0;
    for (int i = threadIdx.x; i < bands; i += kVThreads) {
        s += p[i].sum;
        c += p[i].cnt;
    }
    block_sum(s, c, lds);
    if (threadIdx.x == 0)
        out[blockIdx.x] = VPart{s, c};
}

// Rows per band: at most kMaxBands bands, of whole runs.
int band_rows(int ny)
{
    const int r = (ny + kMaxBands - 1) / kMaxBands;
    return (r + kVRun - 1) / kVRun * kVRun;
}
int bands_for(int ny) { return std::max(1, std::min(ny, kMaxBands)); }  // workspace

// Column pieces of a band: few bands leave CUs idle (one block of a wide grid of
// eight rows walked all its columns: 1e6 x 8 nodes, 64 lags, 6.97 ms, before the
// runs of eight 2.14 ms), so they are split while the launch has under 1024 blocks,
// into pieces of at least 64 columns and as far as the workspace holds partials.
int splits_for(int nx, int ny, int nlags, int bands)
{
    const int groups = (nlags + kVLags - 1) / kVLags;
    const int want = (1024 + 2 * groups * bands - 1) / (2 * groups * bands);
    return std::max(1, std::min({want, nx / 64, bands_for(ny) / bands}));
}

size_t vario_ws_bytes(int ny, int nlags)
{
    const size_t parts = (size_t)2 * nlags * bands_for(ny) * sizeof(VPart);
    return ((parts + 255) & ~size_t(255)) + (size_t)2 * nlags * sizeof(VPart);
}

auv_status check_vario_args(const auv_grid_desc *s, int32_t nlags)
{
    if (!s || s->nx < 1 || s->ny < 1)
        return fail(AUV_ERR_INVALID, "bad grid descriptor");
    if (!(s->dx > 0.0) || !(s->dy > 0.0) || !std::isfinite(s->dx) || !std::isfinite(s->dy))
        return fail(AUV_ERR_INVALID, "grid spacing must be finite and positive");
    if (nlags < 1 || nlags > kMaxLags)
        return fail(AUV_ERR_INVALID, "nlags must be in [1, 1024]");
    return AUV_OK;
}

// Weighted residual of the exponential model at range a, the sill at its
// least-squares value for that range.
double exp_residual(const double *h, const double *g, const double *w, int n, double a,
                    double *sill)
{
    double sgf = 0.0, sff = 0.0;
    for (int j = 0; j < n; ++j) {
        if (!(w[j] > 0.0) || !std::isfinite(g[j]) || !(h[j] > 0.0))
            continue;
        const double f = -std::expm1(-h[j] / a);
        sgf += w[j] * g[j] * f;
        sff += w[j] * f * f;
    }
    const double c = sff > 0.0 ? sgf / sff : 0.0;
    if (sill)
        *sill = c;
    // the residual summed term by term (the expanded form cancels near a
    // perfect fit and would blur the minimum)
    double r = 0.0;
    for (int j = 0; j < n; ++j) {
        if (!(w[j] > 0.0) || !std::isfinite(g[j]) || !(h[j] > 0.0))
            continue;
        const double e = g[j] + c * std::expm1(-h[j] / a);
        r += w[j] * e * e;
    }
    return r;
}

}  // namespace
}  // namespace auv

using namespace auv;

extern "C" {

auv_status auv_variogram_workspace_size(const auv_grid_desc *s, int32_t nlags, size_t *bytes)
{
    if (!bytes)
        return fail(AUV_ERR_INVALID, "bytes is null");
    const auv_status st = check_vario_args(s, nlags);
    if (st != AUV_OK)
        return st;
    *bytes = vario_ws_bytes(s->ny, nlags);
    return AUV_OK;
}

auv_status auv_variogram(const float *src, const auv_grid_desc *s, int32_t nlags, void *ws,
                         size_t ws_bytes, double *gamma_x, double *gamma_y, int64_t *pairs_x,
                         int64_t *pairs_y, auv_stream stream)
{
    auv_status st = check_vario_args(s, nlags);
    if (st != AUV_OK)
        return st;
    if (!src || !ws || !gamma_x || !gamma_y)
        return fail(AUV_ERR_INVALID, "null argument");
    if (ws_bytes < vario_ws_bytes(s->ny, nlags))
        return fail(AUV_ERR_BUDGET, "workspace smaller than auv_variogram_workspace_size");
    if ((reinterpret_cast<uintptr_t>(ws) & 255) != 0)
        return fail(AUV_ERR_INVALID, "workspace must be 256-byte aligned");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const int rows = band_rows(s->ny), bands = (s->ny + rows - 1) / rows;
    const int splits = splits_for(s->nx, s->ny, nlags, bands);
    const int cols = (s->nx + splits - 1) / splits;  // (every piece has some)
    const int pieces = bands * splits;
    VPart *part = static_cast<VPart *>(ws);
    const size_t parts = (size_t)2 * nlags * pieces * sizeof(VPart);
    VPart *out = reinterpret_cast<VPart *>(static_cast<char *>(ws) + ((parts + 255) & ~size_t(255)));
    const unsigned groups = (unsigned)((nlags + kVLags - 1) / kVLags);
    k_vario_partial<<<dim3((unsigned)pieces, groups, 2), kVThreads, 0, hs>>>(
        src, s->nx, s->ny, nlags, rows, cols, splits, part);
    k_vario_final<<<(unsigned)(2 * nlags), kVThreads, 0, hs>>>(part, pieces, out);
    AUV_HIP(hipGetLastError());
    std::vector<VPart> host(2 * (size_t)nlags);
    AUV_HIP(hipMemcpyAsync(host.data(), out, sizeof(VPart) * host.size(), hipMemcpyDeviceToHost,
                           hs));
    AUV_HIP(hipStreamSynchronize(hs));
    for (int k = 0; k < nlags; ++k) {
        const VPart px = host[k], py = host[nlags + k];
        gamma_x[k] = px.cnt > 0 ? px.sum / (2.0 * (double)px.cnt) : NAN;
        gamma_y[k] = py.cnt > 0 ? py.sum / (2.0 * (double)py.cnt) : NAN;
        if (pairs_x)
            pairs_x[k] = px.cnt;
        if (pairs_y)
            pairs_y[k] = py.cnt;
    }
    return AUV_OK;
}

auv_status auv_fit_exponential(const double *h, const double *gamma, const double *w, int32_t n,
                               double *range, double *sill)
{
    if (!h || !gamma || !w || !range || n < 1)
        return fail(AUV_ERR_INVALID, "null argument or no point");
    double hmin = INFINITY, hmax = 0.0;
    int used = 0;
    for (int j = 0; j < n; ++j) {
        if (!(w[j] > 0.0) || !std::isfinite(gamma[j]) || !(h[j] > 0.0))
            continue;
        hmin = std::min(hmin, h[j]);
        hmax = std::max(hmax, h[j]);
        ++used;
    }
    if (used < 2)
        return fail(AUV_ERR_INVALID, "fewer than two usable points");
    // log-spaced scan of the range, then golden-section search between the
    // neighbours of the best scanned value
    const int m = 4001;
    const double l0 = std::log(hmin / 100.0), l1 = std::log(1000.0 * hmax);
    auto at = [&](int i) { return l0 + (l1 - l0) * (double)i / (double)(m - 1); };
    int best = 0;
    double best_r = INFINITY;
    for (int i = 0; i < m; ++i) {
        const double r = exp_residual(h, gamma, w, n, std::exp(at(i)), nullptr);
        if (r < best_r) {
            best_r = r;
            best = i;
        }
    }
    double c = 0.0;
    if (best == 0 || best == m - 1) {
        *range = std::exp(at(best));
        exp_residual(h, gamma, w, n, *range, &c);
        if (sill)
            *sill = c;
        return fail(AUV_ERR_RANGE, "no sill inside [min lag / 100, 1000 max lag]");
    }
    const double phi = 0.5 * (std::sqrt(5.0) - 1.0);
    double lo = at(best - 1), hi = at(best + 1);
    double p = hi - phi * (hi - lo), q = lo + phi * (hi - lo);
    double rp = exp_residual(h, gamma, w, n, std::exp(p), nullptr);
    double rq = exp_residual(h, gamma, w, n, std::exp(q), nullptr);
    for (int it = 0; it < 120; ++it) {
        if (rp <= rq) {
            hi = q;
            q = p;
            rq = rp;
            p = hi - phi * (hi - lo);
            rp = exp_residual(h, gamma, w, n, std::exp(p), nullptr);
        } else {
            lo = p;
            p = q;
            rp = rq;
            q = lo + phi * (hi - lo);
            rq = exp_residual(h, gamma, w, n, std::exp(q), nullptr);
        }
    }
    *range = std::exp(0.5 * (lo + hi));
    exp_residual(h, gamma, w, n, *range, &c);
    if (sill)
        *sill = c;
    return AUV_OK;
}

}  // extern "C"
