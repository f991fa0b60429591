// Radius-limited IDW and nearest pick, gather form (gfx950): the sparse form of
// the exact path.
//
// One lane owns one node and keeps its accumulators (sums, count, depth
// bounds, nearest) in registers; a wave covers 8 x 8 nodes.  The binned
// soundings of the bin rows meeting the tile grown by the radius are read 64
// at a time, one per lane, and become records in LDS.  Every quarter of the
// tile (4 x 4 nodes, 16 lanes) has a list of the records whose disk meets the
// box of its nodes, and its lanes walk that list (a broadcast read per
// quarter): a wave's visits are the longest of its four lists, about 0.6 of
// the records that reach the whole tile.  Nodes above the cap are finished
// together, one lane each, by rounds of a sorted register list.
//
// Exactness: membership, ranking and hits on the exact lattice D^2 (FP64
// squares of integer offsets, exact below 2^53), FP32 weights from the exact
// offsets plus the residuals, FP64 final quotient, clamped to the members'
// depths.  Sums are relative to the depth of the tile's first record.  A node
// with coincident soundings (D^2 == 0) takes their mean depth.
//
// What bounds it: vector instruction issue on large grids (411 vector and 286
// scalar instructions per 64 nodes of the 2M-sounding swath; a SIMD issues a
// vector one in 4.2 clocks), the latency of one wave's chain of reads on small
// ones.  Against the window form it replaces (16 x 16 nodes per wave, LDS
// accumulators, over-cap nodes one at a time), on an MI355X, without binning: 20k
// soundings on 256^2 nodes, 121-node disks 53 -> 15.5 us; nearest only, 500k on 2048 x
// 1500, 64 -> 37 us; the 2M-sounding swath 214 -> 175 us; against the tile kernel, 120k
// on 701 x 650 at 3.3 m 61 -> 19 us.
#pragma once
#include "idw_dense_impl.hpp"
#include "idw_window_impl.hpp"

namespace auv {

namespace gather {

using dense::NodeL;
using dense::node_lat;

// A staged sounding.  p: lattice offset from the tile's first node (as FP32 where
// every offset stays below 2^24, else as integer bits), residuals.  q: depth,
// depth minus the tile's reference, original index (bits).
struct Rec {
    float4 p, q;
};

constexpr int kNull = 64;  // the record no node can reach

// LDS of one wave: the records of a batch, and per quarter the byte offsets of
// its records.
struct Smem {
    Rec rec[64 + 1];
    alignas(8) uint16_t list[4][64];
};
// Two and four list entries at once: types that may alias the entries' own (the
// lists are written an entry at a time).
typedef uint32_t __attribute__((may_alias)) Entries2;
typedef uint32_t __attribute__((ext_vector_type(2), may_alias)) Entries4;

// One instruction each, without the NaN quieting that the compiler adds to
// fminf / fmaxf of values it cannot prove canonical.
__device__ inline float min32(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline float max32(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
constexpr float kFar = 3e38f;

// Accumulators of one node.
struct Acc {
    float num = 0.0f, den = 0.0f, lo = INFINITY, hi = -INFINITY;
    int cnt = 0;
    double bd2 = 1e300;  // nearest: exact lattice D^2, original index, depth
    int bidx = INT_MAX;
    float bz = NAN;
    float emax = -kFar;  // running log2 weight maximum (general power)
};

// Adds a member at squared distance d2 with depth dz above the reference; a hit
// (coincident sounding) counts with the weight kHitW where kHits (integer powers).
template <int kPmode, bool kHits = false>
__device__ __forceinline__ void add_weight(const IdwArgs &a, float d2, float dz, float &num,
                                           float &den, float &emax, bool hit = false)
{
    if constexpr (kPmode != 0) {
        const float w = kHits && hit ? win::kHitW
                                     : win::weight_nonhit(d2, kPmode);
        num = fmaf(w, dz, num);
        den += w;
    } else {
        const float e = -0.5f * a.power * __builtin_amdgcn_logf(d2 * a.inv_r2);
        const float em = fmaxf(emax, e), sc = __builtin_amdgcn_exp2f(emax - em);
        const float w = __builtin_amdgcn_exp2f(e - em);
        num = fmaf(w, dz, num * sc);
        den = fmaf(den, sc, w);
        emax = em;
    }
}

// The binned positions of the bin rows and columns that meet a box, 64 at a
// time (one per lane): the rows' ranges are filled into the lanes one after
// the other, empty rows skipped by a mask (small radii have dozens of bin rows
// per tile, most of them empty).  Against a walk over every row: radius a tenth of
// the spacing, 100k soundings on 1000^2 nodes 44 -> 24 us (the window form 24); and
// with fewer branches between a row and the next, the 2M-sounding step 291 -> 270 us,
// the 256-tile batch 1740 -> 1628.
struct Batches {
    const auv_bin_view &bv;
    int by_lo, nrows, bx_lo, nbx_row;
    int rb, pos, lim;          // row block; the rest of the current row
    unsigned long long rows;   // non-empty rows of the block not yet begun
    int beg, end;              // this lane's row

    // lattice box [x0, x1] x [y0, y1] (nodes), grown by R
    __device__ __forceinline__ Batches(const auv_bin_view &v, int R, int x0, int x1, int y0, int y1)
        : bv(v)
    {
        const int s = v.bin_log2, hB = v.halo << s;
        bx_lo = max(0, (x0 - R + hB) >> s);
        nbx_row = min(v.nbx - 1, (x1 + R + hB) >> s) - bx_lo + 1;
        by_lo = max(0, (y0 - R + hB) >> s);
        nrows = min(v.nby - 1, (y1 + R + hB) >> s) - by_lo + 1;
        rb = 0;
        load();
    }
    __device__ __forceinline__ void load()
    {
        const int lane = threadIdx.x & 63;
        const auto cs = gmem(bv.cell_start);
        // lanes past the last row repeat it
        const int left = nrows - rb;
        const int id0 = (by_lo + rb + min(lane, left - 1)) * bv.nbx + bx_lo;
        beg = cs[id0];
        end = cs[id0 + nbx_row];
        rows = __ballot(end > beg) & (~0ull >> (64 - min(left, 64)));
        pos = lim = 0;
    }
    // The next batch: this lane's position k, valid for lanes below the
    // returned count (0: no batch is left).
    __device__ __forceinline__ int next(int *k)
    {
        const int lane = threadIdx.x & 63;
        int filled = 0, kk = 0;
        do {
            if (pos == lim) {
                while (rows == 0ull && filled == 0 && rb + 64 < nrows) {
                    rb += 64;
                    load();
                }
                if (rows == 0ull)
                    break;
                const int r = __ffsll((long long)rows) - 1;
                rows &= rows - 1ull;
                pos = __builtin_amdgcn_readlane(beg, r);
                lim = __builtin_amdgcn_readlane(end, r);
            }
            kk = lane >= filled ? pos + (lane - filled) : kk;
            const int take = min(64 - filled, lim - pos);
            filled += take;
            pos += take;
        } while (filled < 64);
        *k = kk;
        return filled;
    }
};

// kGen: any node lattice and any radius (nodes with residuals, offsets of any
// size); else the linear lattice of g with offsets below 2^24.
//
// Accumulate mode (kMode bit 2; integer powers, no cap): the wave takes every
// nparts-th batch of the tile's soundings, starting at batch `part`, and returns
// its nodes' sums in *acc_out and their reference depth in *zref_out; hits count
// with the weight kHitW.
//
// kTop > 0 (the dense form on bins of at least the radius): no sums, one pass that
// keeps every node's kTop nearest in a sorted register list, then the dense form's
// finish (max_pts <= kTop).
template <int kMode, int kPmode, bool kGen, int kTop = 0>
__device__ __forceinline__ void gather_tile(const auv_bin_view &bv, const IdwArgs &a,
                                            const WinGeom &g, int tx, int ty, Smem &sm,
                                            int part = 0, int nparts = 1, Acc *acc_out = nullptr,
                                            float *zref_out = nullptr)
{
    constexpr bool kIdw = (kMode & 1) != 0;
    constexpr bool kAccum = (kMode & 4) != 0;
    const int lane = threadIdx.x & 63;
    const int tb0 = tx * 8, ta0 = ty * 8;
    const int lb = lane & 7, la = lane >> 3;  // this lane's node in the tile
    const int quarter = ((la >> 2) << 1) | (lb >> 2);
    // last node of the tile inside the grid
    const int wl = min(7, a.nx - 1 - tb0), hl = min(7, a.ny - 1 - ta0);
    const bool act = lb <= wl && la <= hl;

    // this lane's node relative to the tile's first node (lanes past the grid
    // repeat the last node), and the node extents of the quarters
    int Xo, Yo;          // lattice coordinates of the tile's first node
    int xi, yi;          // offsets
    float rx = 0.0f, ry = 0.0f;  // residuals
    int xq[4], yq[4];    // first and last node of the two columns, the two rows
    if constexpr (kGen) {
        const NodeL nx = node_lat(tb0 + min(lb, wl), a.dx);
        const NodeL ny = node_lat(ta0 + min(la, hl), a.dy);
        Xo = __builtin_amdgcn_readlane(nx.X, 0);
        Yo = __builtin_amdgcn_readlane(ny.X, 0);
        xi = nx.X - Xo;
        yi = ny.X - Yo;
        rx = (float)nx.q * kResidualUnit;
        ry = (float)ny.q * kResidualUnit;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            xq[2 * c] = __builtin_amdgcn_readlane(xi, 4 * c);
            xq[2 * c + 1] = __builtin_amdgcn_readlane(xi, 4 * c + 3);
            yq[2 * c] = __builtin_amdgcn_readlane(yi, 32 * c);
            yq[2 * c + 1] = __builtin_amdgcn_readlane(yi, 32 * c + 24);
        }
    } else {
        Xo = g.X0 + tb0 * g.DXl;
        Yo = g.Y0 + ta0 * g.DYl;
        xi = min(lb, wl) * g.DXl;
        yi = min(la, hl) * g.DYl;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            xq[2 * c] = min(4 * c, wl) * g.DXl;
            xq[2 * c + 1] = min(4 * c + 3, wl) * g.DXl;
            yq[2 * c] = min(4 * c, hl) * g.DYl;
            yq[2 * c + 1] = min(4 * c + 3, hl) * g.DYl;
        }
    }
    const float xn = (float)xi, yn = (float)yi;
    const bool cx = wl >= 4, cy = hl >= 4;  // the second column / row of quarters exists
    const int R = a.R;
    const double R2 = (double)R * (double)R;
    // squared reach of the cull, widened against its FP32 rounding
    const float reach2 = (float)R * (float)R * (1.0f + 0x1p-20f);

    auto rec_at = [&](uint32_t off) {
        return reinterpret_cast<const Rec *>(reinterpret_cast<const char *>(sm.rec) + off);
    };
    // Offset of a record from this lane's node: an integer where kGen (offsets at
    // the largest radius, 2^24, exceed the integers that FP32 holds), else FP32
    // (exact: gather_linear keeps the offsets within reach below 2^24).
    auto off_x = [&](const float4 &p) {
        if constexpr (kGen)
            return __float_as_int(p.x) - xi;
        else
            return p.x - xn;
    };
    auto off_y = [&](const float4 &p) {
        if constexpr (kGen)
            return __float_as_int(p.y) - yi;
        else
            return p.y - yn;
    };
    auto d2_of = [](auto dx, auto dy) {  // exact where |dx|, |dy| <= 2^26
        return fma((double)dx, (double)dx, (double)dy * (double)dy);
    };
    constexpr uint32_t kNullOff = kNull * sizeof(Rec);
    if (lane == 0) {
        sm.rec[kNull].p = kGen ? make_float4(__int_as_float(1 << 30), __int_as_float(1 << 30), 0.0f, 0.0f)
                               : make_float4(1e19f, 1e19f, 0.0f, 0.0f);
        sm.rec[kNull].q = make_float4(0.0f, 0.0f, __int_as_float(INT_MAX), 0.0f);
    }
    float zref = 0.0f;
    bool have_ref = false;
    const uint16_t *const lst = sm.list[quarter];

    // Stages one batch (its records and the quarters' lists, filled up with
    // the null record); returns the length of the longest list.
    auto stage = [&](int k, int have) {
        const bool valid = lane < have;
        int xr = 0, yr = 0, idx = 0;
        uint32_t res = 0;
        float z = 0.0f;
        if (valid) {
            xr = dense::ld_at<int32_t>(gmem(bv.X), (uint32_t)k) - Xo;
            yr = dense::ld_at<int32_t>(gmem(bv.Y), (uint32_t)k) - Yo;
            res = dense::ld_at<uint32_t>(gmem(bv.res), (uint32_t)k);
            z = dense::ld_at<float>(gmem(bv.z), (uint32_t)k);
            idx = dense::ld_at<int32_t>(gmem(bv.idx), (uint32_t)k);
        }
        auto gap2 = [](int v, int lo, int hi) {
            const float e = (float)max(max(lo - v, v - hi), 0);
            return e * e;
        };
        const float ex0 = valid ? gap2(xr, xq[0], xq[1]) : INFINITY;
        const float ex1 = valid && cx ? gap2(xr, xq[2], xq[3]) : INFINITY;
        const float ey0 = reach2 - gap2(yr, yq[0], yq[1]);
        const float ey1 = (cy ? reach2 : -1.0f) - gap2(yr, yq[2], yq[3]);
        // this lane's record reaches the quarter (none reaches those past the grid)
        const bool in[4] = {ex0 <= ey0, ex1 <= ey0, ex0 <= ey1, ex1 <= ey1};
        unsigned long long m[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            m[q] = __ballot(in[q]);
        const unsigned long long any = m[0] | m[1] | m[2] | m[3];
        if (any == 0ull)
            return 0;
        if (!have_ref) {
            // the depth of the first kept sounding is the tile's reference
            zref = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z),
                                                            __ffsll((long long)any) - 1));
            have_ref = true;
        }
        __builtin_amdgcn_wave_barrier();
        const uint32_t nn = kNullOff | (kNullOff << 16);
        reinterpret_cast<Entries4 *>(sm.list)[lane] = Entries4{nn, nn};
        Rec &r = sm.rec[lane];
        r.p = make_float4(kGen ? __int_as_float(xr) : (float)xr, kGen ? __int_as_float(yr) : (float)yr,
                          (float)(int16_t)(res & 0xffffu) * kResidualUnit,
                          (float)(int16_t)(res >> 16) * kResidualUnit);
        r.q = make_float4(z, z - zref, __int_as_float(idx), 0.0f);
        int n = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int slot = __builtin_amdgcn_mbcnt_hi((unsigned)(m[q] >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((unsigned)m[q], 0u));
            if (in[q])
                sm.list[q][slot] = (uint16_t)(lane * sizeof(Rec));
            n = max(n, (int)__popcll(m[q]));
        }
        // the records and lists are read back by the same wave, in order
        __builtin_amdgcn_wave_barrier();
        return n;
    };
    // runs f(n) on every staged batch of the tile
    const int x_last = Xo + xq[3], y_last = Yo + yq[3];
    auto each = [&](auto &&f) {
        Batches it(bv, R, Xo, x_last, Yo, y_last);
        int k, have;
        for (int batch = 0; (have = it.next(&k)) > 0; ++batch) {
            if (kAccum && batch % nparts != part)
                continue;
            const int n = stage(k, have);
            f(n);
        }
    };

    // keys of the capped selection: D^2 << kb | index, as dense_node's list entries
    const int kb = max(bv.idx_bits, 12);
    // the entry of the record at `off` where it is a member above `last`, else +inf
    auto entry = [&](uint32_t off, double last) {
        const Rec *r = rec_at(off);
        const double D2 = d2_of(off_x(r->p), off_y(r->p));
        // bits of D2 + 2^52: the integer D2 under an exponent that the shift by at
        // least 12 drops; 2^52 added to the key makes it a normal number
        const unsigned long long key =
            (((unsigned long long)__double_as_longlong(D2 + 0x1p52)) << kb) | __float_as_uint(r->q.z);
        const double v = __longlong_as_double((long long)(key + (1ull << 52)));
        return (D2 <= R2) & (v > last) ? v : __builtin_huge_val();
    };
    if constexpr (kTop > 0) {
        double list[kTop];
#pragma unroll
        for (int u = 0; u < kTop; ++u)
            list[u] = __builtin_huge_val();
        each([&](int n) {
#pragma unroll 1
            for (int e = 0; e < n; e += 4) {
                const Entries4 o = *reinterpret_cast<const Entries4 *>(lst + e);
                dense::merge4(list, entry(o.x & 0xffffu, 0.0), entry(o.x >> 16, 0.0),
                              entry(o.y & 0xffffu, 0.0), entry(o.y >> 16, 0.0));
            }
        });
        if (act)
            dense::dense_finish<kMode, kTop>(bv, a, tb0 + lb, ta0 + la, list, kb, a.pmode);
        return;
    }

    Acc A;
    each([&](int n) {
        // two records at a time (their reads overlap)
#pragma unroll 1
        for (int e = 0; e < n; e += 2) {
            const uint32_t o2 = *reinterpret_cast<const Entries2 *>(lst + e);
            const Rec *const rp[2] = {rec_at(o2 & 0xffffu), rec_at(o2 >> 16)};
            float4 p[2], q[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                p[u] = rp[u]->p;
                q[u] = rp[u]->q;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const auto dx = off_x(p[u]), dy = off_y(p[u]);
                const double D2 = d2_of(dx, dy);
                if (D2 <= R2) {
                    if constexpr ((kMode & 2) != 0) {
                        const int id = __float_as_int(q[u].z);
                        const bool nearer = (D2 < A.bd2) | ((D2 == A.bd2) & (id < A.bidx));
                        A.bidx = nearer ? id : A.bidx;
                        A.bz = nearer ? q[u].x : A.bz;
                    }
                    if constexpr (!kAccum)
                        A.bd2 = dense::dmin(A.bd2, D2);
                    if constexpr (kIdw) {
                        const float fx = (float)dx + (kGen ? p[u].z - rx : p[u].z);
                        const float fy = (float)dy + (kGen ? p[u].w - ry : p[u].w);
                        const float d2 = fmaf(fx, fx, fy * fy);
                        add_weight<kPmode, kAccum>(a, kGen ? fmaxf(d2, 0x1p-40f) : d2, q[u].y,
                                                   A.num, A.den, A.emax, D2 == 0.0);
                        A.cnt += 1;
                        A.lo = min32(A.lo, q[u].x);
                        A.hi = max32(A.hi, q[u].x);
                    }
                }
            }
        }
    });

    if constexpr (kAccum) {
        *acc_out = A;
        *zref_out = zref;
        return;
    }
    // (64 bits: seven rows of 2^30 nodes are beyond any 32-bit offset)
    const int64_t o = (int64_t)(ta0 + la) * a.nx + (tb0 + lb);
    const bool hit = A.bd2 == 0.0;
    const bool over = kIdw && act && a.max_pts > 0 && A.cnt > a.max_pts;
    if (act && !over) {
        if constexpr ((kMode & 2) != 0) {
            if (a.nn_idx_out)
                gmem(a.nn_idx_out)[o] = A.bd2 < 1e300 ? A.bidx : -1;
            if (a.nn_z_out)
                gmem(a.nn_z_out)[o] = A.bz;
        }
        if constexpr (kIdw) {
            if (a.cnt_out)
                gmem(a.cnt_out)[o] = A.cnt;
            const bool hole = A.cnt == 0 || A.cnt < a.min_pts;
            const float v = (float)((double)zref + win::quotient64(A.num, A.den));
            gmem(a.z_out)[o] = hole ? NAN : fminf(fmaxf(v, A.lo), A.hi);
        }
    }
    if constexpr (kIdw) {
        // (both branches are marked rare: otherwise the registers of the rounds
        // below push the common path's values to scratch, 219 -> 203 us)
        if (__builtin_expect(__any(hit), 0)) {
            // coincident soundings: the node takes their mean depth
            double hsum = 0.0;
            int hcnt = 0;
            each([&](int n) {
#pragma unroll 1
                for (int e = 0; e < n; ++e) {
                    const Rec *r = rec_at(lst[e]);
                    const bool h = off_x(r->p) == 0 && off_y(r->p) == 0;
                    hsum += h ? (double)r->q.x : 0.0;
                    hcnt += h ? 1 : 0;
                }
            });
            if (hit && act && !over)
                gmem(a.z_out)[o] = (float)(hsum / (double)hcnt);
        }
        if (__builtin_expect(__any(over), 0)) {
            // The cap nearest of every node above the cap, in rounds of kRound:
            // each round keeps in a sorted register list the smallest keys above
            // the previous round's, and sums them in key order.
            constexpr int kRound = 8;
            const unsigned imask = (1u << bv.idx_bits) - 1u;
            double last = 0.0;  // key of the last member taken
            int bi = -1;
            float z0 = 0.0f, num = 0.0f, den = 0.0f, lo = INFINITY, hi = -INFINITY, em = -kFar;
            double hsum = 0.0;
            int hcnt = 0;
#pragma unroll 1
            for (int taken = 0; taken < a.max_pts; taken += kRound) {
                double list[kRound];
#pragma unroll
                for (int u = 0; u < kRound; ++u)
                    list[u] = __builtin_huge_val();
                each([&](int n) {
#pragma unroll 1
                    for (int e0 = 0; e0 < n; e0 += 4) {
                        dense::merge4(list, entry(lst[e0], last), entry(lst[e0 + 1], last),
                                      entry(lst[e0 + 2], last), entry(lst[e0 + 3], last));
                    }
                });
                last = list[kRound - 1];
                // one member at a time (a loop unrolled over the list would take
                // registers that cost the common path its waves)
#pragma unroll 1
                for (int u = 0; u < kRound && taken + u < a.max_pts; ++u) {
                    double v = list[0];
#pragma unroll
                    for (int j = 1; j < kRound; ++j)
                        v = u == j ? list[j] : v;
                    if (over) {
                        const unsigned long long key = dense::key_of(v);
                        const int id = (int)((unsigned)key & imask);
                        const int4 rec = bv.rec[id];
                        const float z = __int_as_float(rec.w);
                        if (taken + u == 0) {
                            bi = id;
                            z0 = z;
                        }
                        lo = fminf(lo, z);
                        hi = fmaxf(hi, z);
                        if ((key >> kb) == 0ull) {
                            hsum += (double)z;
                            hcnt += 1;
                        }
                        const float fx = (float)(rec.x - Xo - xi) +
                                         ((float)(int16_t)((uint32_t)rec.z & 0xffffu) * kResidualUnit - rx);
                        const float fy = (float)(rec.y - Yo - yi) +
                                         ((float)(int16_t)((uint32_t)rec.z >> 16) * kResidualUnit - ry);
                        add_weight<kPmode>(a, fmaxf(fmaf(fx, fx, fy * fy), 0x1p-40f), z - z0, num,
                                           den, em);
                    }
                }
            }
            if (over) {
                if constexpr ((kMode & 2) != 0) {
                    if (a.nn_idx_out)
                        gmem(a.nn_idx_out)[o] = bi;
                    if (a.nn_z_out)
                        gmem(a.nn_z_out)[o] = z0;
                }
                if (a.cnt_out)
                    gmem(a.cnt_out)[o] = a.max_pts;
                const float v = (float)((double)z0 + win::quotient64(num, den));
                gmem(a.z_out)[o] = hcnt > 0 ? (float)(hsum / (double)hcnt)
                                                     : a.max_pts < a.min_pts
                                                         ? NAN
                                                         : fminf(fmaxf(v, lo), hi);
            }
        }
    }
}

// Whether the gather form covers a call: 32-bit byte offsets into the binned
// arrays, and with a cap keys (D^2 << max(12, index bits) | index) below 2^62
// and at most eight rounds of the list (a round walks every candidate, so at
// caps of hundreds the window form's bisection over registers is cheaper).
__host__ __device__ inline bool gather_ok(int32_t R, int32_t idx_bits, int32_t max_pts)
{
    if (idx_bits > 30)
        return false;
    return max_pts == 0 ||
           (max_pts <= 64 && dense::dense_key_ok(R, idx_bits < 12 ? 12 : idx_bits));
}

// Whether the linear lattice's offsets within reach of a tile stay below 2^24.
__host__ __device__ inline bool gather_linear(const WinGeom &g, int32_t R)
{
    return (int64_t)R + 7ll * (g.DXl > g.DYl ? g.DXl : g.DYl) < (1ll << 24);
}

// tile0: first tile of the launch (a grid may take several, see launch_tiles)
template <int kMode, int kPmode, bool kGen>
__global__ __launch_bounds__(64, 8) void k_idw_gather(auv_bin_view bv, IdwArgs a, WinGeom g, int ntx,
                                                   int ntiles, int tile0)
{
    __shared__ Smem sm;
    const int tile = win::xcd_tile(tile0 + (int)blockIdx.x, ntiles);
    const int ty = tile / ntx;
    gather_tile<kMode, kPmode, kGen>(bv, a, g, tile - ty * ntx, ty, sm);
}

// Waves per SIMD that the list leaves room for.
constexpr int top_waves(int top) { return top == 8 ? 8 : 5; }

// The dense form on bins of at least the radius.  Its ring search reads nine
// such bins per node whatever the density, five times the disk; the quarters'
// lists hold about half of that, and every record is read once per tile instead
// of once per node.  Bound by vector instruction issue (the list merges) and, at
// one wave generation, by the chain of a tile's batches.  512^2 nodes, disks of
// (cap): 20 (16) 44 -> 39 us, 9 (16) 30 -> 23, 30 (16) 59 -> 54, 5 (8) 20 -> 12, 20 (8)
// 42 -> 28; finer bins, caps above 16 and dense disks keep the ring search
// (gather_top_pays).
template <int kMode, int kTop, bool kGen>
__global__ __launch_bounds__(64, top_waves(kTop)) void k_idw_gather_top(auv_bin_view bv, IdwArgs a,
                                                                      WinGeom g, int ntx,
                                                                      int ntiles, int tile0)
{
    __shared__ Smem sm;
    const int tile = win::xcd_tile(tile0 + (int)blockIdx.x, ntiles);
    const int ty = tile / ntx;
    gather_tile<kMode, 0, kGen, kTop>(bv, a, g, tile - ty * ntx, ty, sm);
}

}  // namespace gather
}  // namespace auv
