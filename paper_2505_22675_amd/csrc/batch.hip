// Batches of independent, uneven gridding problems.
//
//   auv_batch_plan      host: validate items, pick bin size and kernel form per
//                       item (autotune table or defaults), lay out a workspace
//   auv_batch_launch    first call: upload item tables, capture
//                         batched binning (4 launches for all items)
//                         -> one IDW launch per kernel form over the units of
//                         all its items (sparse gather, window, span / dense
//                         top-k, on two concurrent branches), + per-item
//                         launches for items they do not cover
//                       into a HIP graph; later calls replay the graph
//   auv_batch_launch_plain  the same items one after another, default sizes
//   auv_batch_autotune  time (bin size, form) candidates per item class
//
// A unit is one (item, node tile); block b of a form's launch takes one unit
// of the form's list (deal_unit), and the hardware's block scheduler balances
// units of uneven cost.  Items with the costliest tiles come first.
#include "idw_gather_impl.hpp"
#include "idw_span_impl.hpp"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <map>
#include <new>
#include <sstream>
#include <string>
#include <vector>

namespace auv {

namespace {

constexpr int kXcds = 8;
constexpr int kRun = 64;  // consecutive units of one XCD
constexpr int kForms = 6;
constexpr int kFewSortRows = 2560;  // ten bin rows per CU
constexpr int kBatchDenseK = 16;  // largest max_pts the batched dense kernel keeps

// gather form on linear lattices, dense ring search, span, dense by lists, gather form
// on any lattice, window form
enum { kSparse = 0, kDense = 1, kSpan = 2, kTop = 3, kWide = 4, kWindow = 5 };

struct IdwItem {
    auv_bin_view bv;
    IdwArgs a;
    WinGeom g;
    int32_t ntx, ntiles;
    int32_t form, pmode;
};

// The unit of block b out of n: blocks are dealt round-robin to the 8 XCDs,
// so each XCD gets runs of kRun consecutive units (neighbouring tiles of an
// item, whose halos overlap in its L2) and every XCD a share of every item.  Inside
// a run the order is transposed as 4 x 16: an XCD's blocks go to its four shader
// engines in turn, so units taken in order put every fourth tile on the same engine,
// and soundings in lines a multiple of four tiles apart (32 nodes) on a quarter of
// the chip (60 tiles of 256^2 nodes with all soundings in 5 % of the width at such a
// spacing, 60 per disk on average: in order 5.18 ms, transposed 2.99).
// (Queues with one head per XCD and guided grabs took longer: every grab is a
// device atomic on one of eight addresses, and the loop around a tile made the
// compiler keep its constants in scratch.)
__device__ inline int deal_unit(int b, int n)
{
    const int g = b / (kXcds * kRun), l = b - g * (kXcds * kRun);
    const int p = l / kXcds;
    return (g + 1) * (kXcds * kRun) <= n ? g * (kXcds * kRun) + (l & (kXcds - 1)) * kRun +
                                               (p >> 2) + (p & 3) * (kRun / 4)
                                         : b;
}

// One launch per form (their register and LDS budgets differ).  The work entry
// is wave-uniform: the item descriptor is read with scalar loads.

// Sparse: a unit is 16 nodes wide and 16 or 8 high, one 8 x 8-node gather tile
// per wave.  Bound by vector instruction issue like the gather form itself.
// Against the persistent window kernel it replaced (LDS accumulators, work from
// queues): 32 tiles of 512^2 nodes with 0.25 / 2 / 8 soundings per disk, binning
// included, 698 / 713 / 900 -> 108 / 138 / 417 us (cap 16), 864 -> 284 us
// (8 per disk, no cap).
template <bool kGeneral, bool kGen>
__global__ __launch_bounds__(256, 8) void k_idw_batch_sparse(const IdwItem *__restrict__ items,
                                                             const int2 *__restrict__ work, int n,
                                                             int b0)
{
    __shared__ gather::Smem sm[4];
    const int2 w = work[deal_unit(b0 + (int)blockIdx.x, n)];
    const IdwItem &it = items[w.x];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int uy = w.y / it.ntx, ux = w.y - uy * it.ntx;
    const int sub = win::tile_rows(it.a) / 8;  // gather tile rows of a unit
    const int tx = 2 * ux + (wave & 1), ty = sub * uy + (wave >> 1);
    if ((wave >> 1) >= sub || tx * 8 >= it.a.nx || ty * 8 >= it.a.ny)
        return;
    // an instantiation per integer power (a test of the power at every visit
    // costs a tenth) and one for a general power, with its rescaled sums
    if (it.pmode == 2) {
        gather::gather_tile<3, 2, kGen>(it.bv, it.a, it.g, tx, ty, sm[wave]);
    } else if (it.pmode == 1) {
        gather::gather_tile<3, 1, kGen>(it.bv, it.a, it.g, tx, ty, sm[wave]);
    } else if (it.pmode == 3) {
        gather::gather_tile<3, 3, kGen>(it.bv, it.a, it.g, tx, ty, sm[wave]);
    } else if constexpr (kGeneral) {
        gather::gather_tile<3, 0, kGen>(it.bv, it.a, it.g, tx, ty, sm[wave]);
    }
}

// Window: caps and keys beyond the gather form's, one 16 x 16 or 16 x 8 node tile per
// block.  Integer powers share one instantiation (the power at run time).  One launch
// per item instead, in series: 200 tiles of 64^2 nodes, cap 100, 2 / 12 / 40
// soundings per disk 2.1 / 8.1 / 24.5 ms.
template <bool kGeneral>
__global__ __launch_bounds__(64) void k_idw_batch_window(const IdwItem *__restrict__ items,
                                                         const int2 *__restrict__ work, int n,
                                                         int b0)
{
    __shared__ float2 s_nd[win::kAcc];
    __shared__ int s_cnt[win::kAcc];
    __shared__ float s_lo[win::kAcc], s_hi[win::kAcc];
    __shared__ unsigned long long s_key[win::kAcc];
    __shared__ float s_emax[kGeneral ? win::kAcc : 1];
    __shared__ int s_beg[win::kMaxRows], s_off[win::kMaxRows + 1];
    __shared__ int4 s_rec[win::kRecSlots];
    const win::WinSmem sm{s_nd, s_cnt, s_lo, s_hi, s_key, nullptr, nullptr, nullptr,
                          s_emax, s_beg, s_off, s_rec, s_rec + 1, nullptr};
    const int2 w = work[deal_unit(b0 + (int)blockIdx.x, n)];
    const IdwItem &it = items[w.x];
    if constexpr (kGeneral) {
        if (it.pmode == 0) {
            win::window_tile<3, 0, true, 1, AUV_P_FP32_REBASE>(it.bv, it.a, it.g, w.y, it.ntx, sm);
            return;
        }
    }
    win::window_tile<3, -1, true, 1, AUV_P_FP32_REBASE>(it.bv, it.a, it.g, w.y, it.ntx, sm);
}

// Dense: one node tile of 64 nodes per block.
__global__ __launch_bounds__(64) void k_idw_batch_dense(const IdwItem *__restrict__ items,
                                                        const int2 *__restrict__ work, int n,
                                                        int b0)
{
    const int2 w = work[deal_unit(b0 + (int)blockIdx.x, n)];
    const IdwItem &it = items[w.x];
    dense::dense_tile<3, kBatchDenseK>(it.bv, it.a, w.y, it.ntx, it.pmode);
}

// Dense by the gather form's lists: one tile of 8 x 8 nodes per block.
__global__ __launch_bounds__(64, gather::top_waves(kBatchDenseK)) void k_idw_batch_top(
    const IdwItem *__restrict__ items, const int2 *__restrict__ work, int n, int b0)
{
    __shared__ gather::Smem sm;
    const int2 w = work[deal_unit(b0 + (int)blockIdx.x, n)];
    const IdwItem &it = items[w.x];
    const int ty = w.y / it.ntx;
    gather::gather_tile<3, 0, false, kBatchDenseK>(it.bv, it.a, it.g, w.y - ty * it.ntx, ty, sm);
}

// Span: one 16 x 16 node tile per block.
__global__ __launch_bounds__(64) void k_idw_batch_span(const IdwItem *__restrict__ items,
                                                       const int2 *__restrict__ work, int n,
                                                       int b0)
{
    __shared__ span::Smem<win::kTW, win::kTH> sm;
    const int2 w = work[deal_unit(b0 + (int)blockIdx.x, n)];
    const IdwItem &it = items[w.x];
    span::span_tile<3, -1, win::kTW, win::kTH>(it.bv, it.a, it.g, w.y, it.ntx, sm);
}

void launch_form(int form, bool general, const IdwItem *items, const int2 *work, int n,
                 hipStream_t st)
{
    // HIP takes fewer than 2^32 threads per launch: the list goes in pieces (of
    // whole runs on every XCD)
    auto pieces = [&](auto *kernel, int threads) {
        constexpr int kPiece = 1 << 23;
        static_assert(kPiece % (kXcds * kRun) == 0, "pieces cut the dealt runs");
        for (int64_t b0 = 0; b0 < n; b0 += kPiece)
            kernel<<<(unsigned)std::min<int64_t>(kPiece, n - b0), threads, 0, st>>>(items, work, n,
                                                                                    (int)b0);
    };
    if (form == kDense)
        pieces(k_idw_batch_dense, 64);
    else if (form == kTop)
        pieces(k_idw_batch_top, 64);
    else if (form == kSpan)
        pieces(k_idw_batch_span, 64);
    else if (form == kWindow)
        pieces(general ? k_idw_batch_window<true> : k_idw_batch_window<false>, 64);
    else if (form == kWide)
        pieces(general ? k_idw_batch_sparse<true, true> : k_idw_batch_sparse<false, true>, 256);
    else
        pieces(general ? k_idw_batch_sparse<true, false> : k_idw_batch_sparse<false, false>, 256);
}

inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

int pmode_of(double p)
{
    if (p == 1.0)
        return 1;
    if (p == 2.0)
        return 2;
    if (p == 3.0)
        return 3;
    return 0;
}

// Expected soundings per disk: input count over the grid grown by r.
double disk_population(const auv_batch_item &it)
{
    const double r = it.params.radius;
    const double area = (it.grid.nx * it.grid.dx + 2 * r) * (it.grid.ny * it.grid.dy + 2 * r);
    return (double)it.n / area * 3.141592653589793 * r * r;
}

struct ClassKey {
    int dens, side;
    bool operator<(const ClassKey &o) const
    {
        return dens != o.dens ? dens < o.dens : side < o.side;
    }
};

ClassKey class_of(const auv_batch_item &it)
{
    ClassKey k;
    k.dens = (int)std::floor(std::log2(disk_population(it) + 1.0));
    k.side = (int)std::lround(std::log2((double)std::max(it.grid.nx, it.grid.ny)));
    return k;
}

bool dense_allowed(const auv_batch_item &it)
{
    int bits = 1;
    while (bits < 31 && (int64_t(1) << bits) < it.n)
        ++bits;
    const double Rd = std::rint(it.params.radius * kLatticePerMetre);
    return it.params.max_pts >= 1 && it.params.max_pts <= 32 &&
           it.params.precision == AUV_P_FP32_REBASE && Rd < 2147483648.0 &&
           dense::dense_key_ok((int32_t)Rd, bits);
}

// Bin side of the dense form's search for an item that no tuning table sets:
// the default side s (about R) halved until it is about 1.2 times the distance
// to the max_pts-th neighbour at the item's mean density (rounded to a power of
// two; caps under 8 count as 8, since a segment costs four candidates anyway).
// The ring search then ends after its first ring with about 3 max_pts
// candidates read, where default bins read nine bins of up to several hundred
// soundings each, and the sort's bins and rows are short.  256 uneven tiles of
// 1k-200k soundings, IDW and binning together: default side 4.95 ms, 0.7 / 1.0
// / 1.4 / 2.0 times the distance 2.33 / 2.25 / 2.26 / 2.51 ms.
//
// Up to kTopPop caps per disk the default side stays: the form by lists takes
// those items.  Limits of 1.0, 1.5 and 3 caps: the 256-tile batch 1738, 1738 and
// 1743 us (the ring search on small bins for all of them 1768); 4 tiles of which
// one holds 1.9 caps per disk 81 us at 1.5 and 66 at 3 (a small batch is the
// search's chain of bins), 6 such tiles 84 and 71.
constexpr double kTopPop = 3.0;

int32_t dense_cell_log2(const auv_batch_item &it, int32_t R, int32_t s)
{
    const double pop = disk_population(it);
    const double k = std::max(8, it.params.max_pts);
    if (!(pop > kTopPop * k))
        return s;
    const int32_t c = (int32_t)std::lround(std::log2(1.2 * R * std::sqrt(k / pop)));
    return std::max<int32_t>(12, std::min(s, c));
}

struct Choice {
    int32_t bin_log2;
    int32_t algo;                // AUV_ALGO_SPARSE or AUV_ALGO_DENSE
    int32_t tile_w = 0, tile_h = 0;  // node tile per wave (0: the form's default)
};

// Default node tile of a form.
Choice with_default_tile(Choice c)
{
    c.tile_w = c.algo == AUV_ALGO_DENSE ? dense::kDT : win::kTW;
    c.tile_h = c.algo == AUV_ALGO_DENSE ? dense::kDT : win::kTH;
    return c;
}

// The other node tiles the autotuner may try for a (bin size, form) choice.
std::vector<Choice> tile_variants(const Choice &c)
{
    std::vector<Choice> v;
    if (c.algo == AUV_ALGO_DENSE) {
        for (int tw : {16, 4}) {
            Choice d = c;
            d.tile_w = tw;
            d.tile_h = 64 / tw;
            v.push_back(d);
        }
    } else {
        Choice d = c;
        d.tile_w = win::kTW;
        d.tile_h = 8;
        v.push_back(d);
    }
    return v;
}

// Most work units an item can have, whatever its form and node tile (the dense
// form's tiles are any power-of-two shape of 64 nodes, the others larger than
// 8 x 8).
size_t most_units(const auv_batch_item &it)
{
    size_t most = 0;
    for (int w = 1; w <= 64; w *= 2) {
        const int h = 64 / w;
        most = std::max(most, (size_t)((it.grid.nx + w - 1) / w) *
                                  (size_t)((it.grid.ny + h - 1) / h));
    }
    return most;
}

// Candidate (bin size, form) pairs the autotuner may time for an item.
std::vector<Choice> candidates(const auv_batch_item &it, int32_t sR)
{
    std::vector<Choice> c;
    // the sparse form walks a tile's soundings again for every eight members of the
    // cap once a node is above it: at four caps per disk it takes twice the dense
    // form's time (512^2 nodes, cap 16: 245 and 108 us)
    const bool sparse_ok = !dense_allowed(it) || disk_population(it) < 4.0 * it.params.max_pts;
    for (int d = -1; d <= 1 && sparse_ok; ++d)
        if (sR + d >= 12 && sR + d <= 26)
            c.push_back({sR + d, AUV_ALGO_SPARSE});
    // dense: bins down to 1/64 of the default side (very dense tiles want bins
    // holding a few soundings, so the ring search stops after a few rings)
    if (dense_allowed(it) && disk_population(it) >= 0.5 * it.params.max_pts)
        for (int d = -6; d <= -1; ++d)
            if (sR + d >= 12)
                c.push_back({sR + d, AUV_ALGO_DENSE});
    return c;
}

}  // namespace

}  // namespace auv

// ------------------------------------------------------------- the batch --

struct auv_batch {
    std::vector<auv_batch_item> items;
    std::vector<auv_grid> grids;
    std::vector<auv::BinGeom> geom;        // batched form
    std::vector<int32_t> plan_bin;         // planned bin size (geom may subdivide it)
    std::vector<auv::BinGeom> geom_plain;  // plain form
    std::vector<int32_t> algo;             // batched form
    std::vector<auv::Choice> tile;         // batched form: node tile per wave
    std::vector<size_t> slice_off;         // per-item workspace slice
    std::vector<size_t> slice_size;
    std::vector<uint8_t> covered;          // by the forms' batched kernels
    size_t tables_bytes = 0, ws_bytes = 0;
    // host copies of the device tables (valid for `bound_ws`)
    std::vector<auv::RowItem> rows;
    std::vector<auv::IdwItem> idw;
    std::vector<int32_t> offs;  // hist, scatter, sort offsets
    std::vector<int2> work;
    int32_t hist_blocks = 0, scatter_blocks = 0, nrow_items = 0;
    auv::RowSortClass sort_class[auv::kRowSortClasses];
    int32_t work_off[auv::kForms + 1] = {0};  // each form's units in `work`
    bool any_general[auv::kForms] = {};  // the form has an item with a general power
    int32_t max_nbx = 0, max_nby = 0;  // largest bin domain of the row-binned items
    hipStream_t cap_stream2 = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    // graph
    void *bound_ws = nullptr;
    hipStream_t cap_stream = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

namespace auv {

namespace {

auv_status validate_item(const auv_batch_item &it, int i)
{
    const std::string tag = "item " + std::to_string(i) + ": ";
    if (it.n < 0 || it.n >= INT32_MAX)
        return fail(AUV_ERR_INVALID, tag + "n must be in [0, 2^31-1)");
    if (it.n > 0 && (!it.x || !it.y || !it.z))
        return fail(AUV_ERR_INVALID, tag + "null sounding pointer");
    if (!it.z_out)
        return fail(AUV_ERR_INVALID, tag + "z_out is null");
    const auv_idw_params &p = it.params;
    if (!(p.power > 0.0) || !(p.power <= 64.0) || p.min_pts < 0 || p.max_pts < 0)
        return fail(AUV_ERR_INVALID, tag + "bad power / min_pts / max_pts");
    if (p.precision != AUV_P_FP32_REBASE)
        return fail(AUV_ERR_INVALID, tag + "batches run the exact FP64-rebase form only");
    if (p.algo < AUV_ALGO_AUTO || p.algo > AUV_ALGO_SPAN)
        return fail(AUV_ERR_INVALID, tag + "unknown algo");
    return AUV_OK;
}

// Build the bin view and IDW arguments of item i with its workspace slice.
void item_views(const auv_batch *b, int i, char *ws, const BinGeom &geom, int32_t algo,
                BinWorkspace *w, auv_bin_view *bv, IdwArgs *a, Choice tile = Choice{0, 0})
{
    const auv_batch_item &it = b->items[i];
    bin_workspace_layout(it.n, geom, ws + b->slice_off[i], w);
    auv_bin_view v{};
    v.cell_start = w->cell_start;
    v.X = w->X;
    v.Y = w->Y;
    v.res = w->res;
    v.z = w->z;
    v.idx = w->idx;
    v.rec = w->rec;
    v.nbx = geom.nbx;
    v.nby = geom.nby;
    v.halo = geom.halo;
    v.bin_log2 = geom.s;
    v.R = geom.R;
    int bits = 1;
    while (bits < 31 && (int64_t(1) << bits) < it.n)
        ++bits;
    v.idx_bits = bits;
    *bv = v;
    IdwArgs x;
    std::memset(&x, 0, sizeof(x));
    x.dx = it.grid.dx;
    x.dy = it.grid.dy;
    x.nx = it.grid.nx;
    x.ny = it.grid.ny;
    x.R = geom.R;
    x.R_stage = geom.R;
    x.inv_r2 = (float)(1.0 / ((double)geom.R * geom.R));
    x.r2f = (float)(it.params.radius * it.params.radius);
    x.x0 = it.grid.x0;
    x.y0 = it.grid.y0;
    x.power = (float)it.params.power;
    x.min_pts = it.params.min_pts;
    x.max_pts = it.params.max_pts;
    x.precision = AUV_P_FP32_REBASE;
    x.mode = (it.nn_idx_out || it.nn_z_out) ? 3 : 1;
    x.z_out = it.z_out;
    x.cnt_out = it.cnt_out;
    x.nn_idx_out = it.nn_idx_out;
    x.nn_z_out = it.nn_z_out;
    x.population = (float)disk_population(it);
    x.dense = algo == AUV_ALGO_DENSE;
    x.span = algo == AUV_ALGO_SPAN;
    x.pmode = pmode_of(it.params.power);
    x.tile_w = tile.tile_w;
    x.tile_h = tile.tile_h;
    *a = x;
}

int32_t auto_algo(const auv_batch_item &it)
{
    if (it.params.algo != AUV_ALGO_AUTO)
        return it.params.algo;
    return dense_allowed(it) && disk_population(it) >= 0.5 * it.params.max_pts ? AUV_ALGO_DENSE
                                                                          : AUV_ALGO_SPARSE;
}

std::map<ClassKey, Choice> read_tune(const char *path)
{
    std::map<ClassKey, Choice> t;
    if (!path)
        return t;
    std::ifstream f(path);
    std::string line;
    while (std::getline(f, line)) {
        std::istringstream is(line);
        std::string tag, k1, k2;
        ClassKey key;
        Choice c;
        double ms;
        if (is >> tag >> key.dens >> key.side >> k1 >> c.bin_log2 >> k2 >> c.algo && tag == "class") {
            std::string k3;
            int tw = 0, th = 0;
            if (is >> k3 && k3 == "tile" && is >> tw >> th) {
                c.tile_w = tw;
                c.tile_h = th;
            }
            t[key] = c;
        }
        (void)ms;
    }
    return t;
}

// The batched kernels' descriptor of one item; false when they do not cover it
// (dense caps above 16; caps above 64 on lattices that are not linear or with windows
// of several chunks).
bool make_idw_item(const auv_batch_item &it, const auv_bin_view &bv, const IdwArgs &a,
                   int32_t algo, IdwItem *out)
{
    IdwItem d{};
    d.bv = bv;
    d.a = a;
    d.pmode = pmode_of(it.params.power);
    bool ok = true;
    if (algo == AUV_ALGO_DENSE) {
        d.form = kDense;
        ok = it.params.max_pts >= 1 && it.params.max_pts <= kBatchDenseK &&
             dense::dense_key_ok(a.R, bv.idx_bits);
        // on bins of at least the radius by the gather form's lists (8 x 8 nodes)
        if (ok && dense::dense_tile_w(a) == dense::kDT && gather_top_covers(bv, a) &&
            window_geometry(a, &d.g) && gather::gather_linear(d.g, a.R))
            d.form = kTop;
        const int tw = dense::dense_tile_w(a), th = 64 / tw;
        d.ntx = (it.grid.nx + tw - 1) / tw;
        d.ntiles = d.ntx * ((it.grid.ny + th - 1) / th);
    } else {
        const bool linear = window_geometry(a, &d.g);
        if (linear && a.span && span::span_ok(bv, a, d.g, d.pmode)) {
            d.form = kSpan;
        } else if (gather::gather_ok(a.R, bv.idx_bits, it.params.max_pts)) {
            d.form = linear && gather::gather_linear(d.g, a.R) ? kSparse : kWide;
        } else {
            // windows of one chunk, keys (D^2 << index bits | index) of 64 bits
            d.form = kWindow;
            ok = linear && d.g.nchunks == 1 && it.grid.nx <= 1 << 26 &&
                 ((unsigned __int128)((unsigned long long)a.R * a.R) << bv.idx_bits) <
                     ((unsigned __int128)1 << 64);
        }
        const int th = d.form == kSpan ? win::kTH : win::tile_rows(a);
        d.ntx = (it.grid.nx + win::kTW - 1) / win::kTW;
        d.ntiles = d.ntx * ((it.grid.ny + th - 1) / th);
    }
    *out = d;
    return ok;
}

// Build the device tables for workspace `ws` (host copies kept in the batch).
auv_status build_tables(auv_batch *b, char *ws)
{
    const int count = (int)b->items.size();
    b->rows.assign(count, RowItem{});
    b->max_nbx = b->max_nby = 0;
    b->idw.assign(count, IdwItem{});
    std::vector<int32_t> hist(1, 0), scat(1, 0), sort(1, 0);
    std::vector<double> tile_cost(count, 0.0);
    for (int i = 0; i < count; ++i) {
        const auv_batch_item &it = b->items[i];
        BinWorkspace w;
        auv_bin_view bv;
        IdwArgs a;
        item_views(b, i, ws, b->geom[i], b->algo[i], &w, &bv, &a, b->tile[i]);
        IdwItem &d = b->idw[i];
        const bool ok = make_idw_item(it, bv, a, b->algo[i], &d) && row_path_ok(b->geom[i]);
        b->covered[i] = ok ? 1 : 0;
        if (d.form == kDense || d.form == kTop) {
            tile_cost[i] = ((double)it.n + (double)it.grid.nx * it.grid.ny * 4.0) /
                           std::max(1, d.ntiles);
        } else {
            // a tile costs a fixed part plus one visit per sounding
            // within reach of its box (uniform density over the grid grown
            // by the radius)
            const double r = it.params.radius;
            const double rho = (double)it.n / ((it.grid.nx * it.grid.dx + 2.0 * r) *
                                               (it.grid.ny * it.grid.dy + 2.0 * r));
            const double bw = win::kTW * it.grid.dx + 2.0 * r;
            const double bh = win::tile_rows(a) * it.grid.dy + 2.0 * r;
            tile_cost[i] = 20.0 + rho * bw * bh;
        }
    }
    // row-binned items by the class of their rows' sort; a batch of few rows takes
    // one launch of the largest class instead (a launch costs more than the
    // smaller key areas save there: 7 tiles 93 -> 86 us, 16 tiles 107 -> 103)
    int64_t all_rows = 0;
    int top_class = 0;
    for (int i = 0; i < count; ++i) {
        const BinGeom &g = b->geom[i];
        if (!row_path_ok(g))
            continue;
        all_rows += g.nby;
        top_class = std::max(top_class,
                             row_sort_class((double)b->items[i].n / std::max(1, g.nby)));
    }
    const bool one_class = all_rows <= kFewSortRows;
    b->nrow_items = 0;
    for (int sc = 0; sc < kRowSortClasses; ++sc) {
        RowSortClass &c = b->sort_class[sc];
        c = RowSortClass{};
        c.block0 = sort.back();
        for (int i = 0; i < count; ++i) {
            const auv_batch_item &it = b->items[i];
            const BinGeom &g = b->geom[i];
            if (!row_path_ok(g))
                continue;
            if (sc != (one_class ? top_class
                                 : row_sort_class((double)it.n / std::max(1, g.nby))))
                continue;
            BinWorkspace w;
            bin_workspace_layout(it.n, g, ws + b->slice_off[i], &w);
            b->rows[b->nrow_items++] =
                make_row_item(&b->grids[i], g, it.x, it.y, it.z, it.n, w);
            hist.push_back(hist.back() + row_hist_blocks(it.n));
            scat.push_back(scat.back() + row_scatter_blocks(it.n));
            sort.push_back(sort.back() + g.nby);
            c.max_nbx = std::max(c.max_nbx, g.nbx);
            b->max_nbx = std::max(b->max_nbx, g.nbx);
            b->max_nby = std::max(b->max_nby, g.nby);
        }
        c.block1 = sort.back();
    }
    b->hist_blocks = hist.back();
    b->scatter_blocks = scat.back();
    // units by form, items with the costliest tiles first (a wave takes a tile
    // alone, so a long tile late in the launch would end it late)
    std::vector<int> order(count);
    for (int i = 0; i < count; ++i)
        order[i] = i;
    std::stable_sort(order.begin(), order.end(),
                     [&](int x, int y) { return tile_cost[x] > tile_cost[y]; });
    b->work.clear();
    for (int form = 0; form < kForms; ++form) {
        b->any_general[form] = false;
        for (int i : order) {
            if (!b->covered[i] || b->idw[i].form != form)
                continue;
            for (int t = 0; t < b->idw[i].ntiles; ++t)
                b->work.push_back(make_int2(i, t));
            b->any_general[form] = b->any_general[form] || b->idw[i].pmode == 0;
        }
        b->work_off[form + 1] = (int32_t)b->work.size();
    }
    b->offs.clear();
    b->offs.insert(b->offs.end(), hist.begin(), hist.end());
    b->offs.insert(b->offs.end(), scat.begin(), scat.end());
    b->offs.insert(b->offs.end(), sort.begin(), sort.end());
    return AUV_OK;
}

// Table region at the start of the workspace.
struct Tables {
    RowItem *rows;
    IdwItem *idw;
    int32_t *offs;
    int2 *work;
};

Tables table_ptrs(const auv_batch *b, char *ws)
{
    const size_t count = b->items.size();
    size_t off = 0;
    Tables t;
    t.rows = reinterpret_cast<RowItem *>(ws + off);
    off += align256(sizeof(RowItem) * count);
    t.idw = reinterpret_cast<IdwItem *>(ws + off);
    off += align256(sizeof(IdwItem) * count);
    t.offs = reinterpret_cast<int32_t *>(ws + off);
    off += align256(sizeof(int32_t) * 3 * (count + 1));
    t.work = reinterpret_cast<int2 *>(ws + off);
    return t;
}

size_t tables_size(size_t count, size_t max_tiles)
{
    return align256(sizeof(RowItem) * count) + align256(sizeof(IdwItem) * count) +
           align256(sizeof(int32_t) * 3 * (count + 1)) +
           align256(sizeof(int2) * std::max<size_t>(max_tiles, 1));
}

// Enqueue the whole batched form on `st` (captured by the caller).
auv_status enqueue_batched(auv_batch *b, char *ws, hipStream_t st)
{
    const Tables t = table_ptrs(b, ws);
    const int count = (int)b->items.size();
    const int nr = b->nrow_items;
    AUV_TRY_S(launch_binning_batch(t.rows, t.offs, t.offs + (nr + 1), t.offs + 2 * (nr + 1), nr,
                                   b->hist_blocks, b->scatter_blocks, b->sort_class, b->max_nbx,
                                   b->max_nby, false, st));
    for (int i = 0; i < count; ++i) {
        if (row_path_ok(b->geom[i]))
            continue;
        BinWorkspace w;
        auv_bin_view bv;
        IdwArgs a;
        item_views(b, i, ws, b->geom[i], b->algo[i], &w, &bv, &a, b->tile[i]);
        const auv_batch_item &it = b->items[i];
        AUV_TRY_S(launch_binning(&b->grids[i], b->geom[i], it.x, it.y, it.z, it.n, w, st));
    }
    auto units = [&](int form) { return b->work_off[form + 1] - b->work_off[form]; };
    auto launch = [&](int form, hipStream_t s) -> auv_status {
        if (units(form) > 0) {
            launch_form(form, b->any_general[form], t.idw, t.work + b->work_off[form], units(form), s);
            AUV_HIP(hipGetLastError());
        }
        return AUV_OK;
    };
    // the dense forms run on a forked branch of the graph, concurrently
    const bool fork = units(kDense) > 0 || units(kTop) > 0;
    if (fork) {
        AUV_HIP(hipEventRecord(b->ev_fork, st));
        AUV_HIP(hipStreamWaitEvent(b->cap_stream2, b->ev_fork, 0));
        AUV_TRY_S(launch(kDense, b->cap_stream2));
        AUV_TRY_S(launch(kTop, b->cap_stream2));
        AUV_HIP(hipEventRecord(b->ev_join, b->cap_stream2));
    }
    for (int form : {kSparse, kWide, kWindow, kSpan})
        AUV_TRY_S(launch(form, st));
    if (fork)
        AUV_HIP(hipStreamWaitEvent(st, b->ev_join, 0));
    for (int i = 0; i < count; ++i) {
        if (b->covered[i])
            continue;
        AUV_TRY_S(launch_idw(b->idw[i].bv, b->idw[i].a, st));
    }
    return AUV_OK;
}

}  // namespace
}  // namespace auv

using namespace auv;

extern "C" {

auv_status auv_batch_plan(const auv_batch_item *items, int32_t count, const char *tune_path,
                          auv_batch **out)
{
    if (!out)
        return fail(AUV_ERR_INVALID, "out is null");
    *out = nullptr;
    if (!items || count < 1)
        return fail(AUV_ERR_INVALID, "need at least one item");
    auv_batch *b = new (std::nothrow) auv_batch;
    if (!b)
        return fail(AUV_ERR_INVALID, "out of host memory");
    b->items.assign(items, items + count);
    b->grids.resize(count);
    b->geom.resize(count);
    b->plan_bin.resize(count);
    b->geom_plain.resize(count);
    b->algo.resize(count);
    b->tile.resize(count);
    b->slice_off.resize(count);
    b->slice_size.resize(count);
    b->covered.assign(count, 0);
    const std::map<ClassKey, Choice> tune = read_tune(tune_path);
    size_t off = 0, max_tiles = 0;
    for (int i = 0; i < count; ++i) {
        const auv_batch_item &it = b->items[i];
        auv_status st = validate_item(it, i);
        if (st == AUV_OK) {
            auv_grid *g = nullptr;
            st = auv_grid_create(&it.grid, &g);
            if (st == AUV_OK) {
                b->grids[i] = *g;
                auv_grid_destroy(g);
            }
        }
        if (st == AUV_OK)
            st = bin_geometry(&b->grids[i], it.params.radius, 0, &b->geom_plain[i]);
        if (st != AUV_OK) {
            delete b;
            return st;
        }
        Choice c{b->geom_plain[i].s, auto_algo(it)};
        const auto f = tune.find(class_of(it));
        const bool tuned = f != tune.end() && it.params.algo == AUV_ALGO_AUTO &&
                           (f->second.algo == AUV_ALGO_SPARSE || dense_allowed(it));
        if (tuned)
            c = f->second;
        b->algo[i] = c.algo;
        b->tile[i] = c.tile_w > 0 ? c : with_default_tile(c);
        st = bin_geometry(&b->grids[i], it.params.radius, c.bin_log2, &b->geom[i]);
        if (st != AUV_OK) {
            b->geom[i] = b->geom_plain[i];
            b->algo[i] = auto_algo(it);
            b->tile[i] = with_default_tile(Choice{0, b->algo[i]});
        }
        b->plan_bin[i] = b->geom[i].s;
        if (!tuned && b->algo[i] == AUV_ALGO_DENSE) {
            // the dense form's own subdivision of the planned bins, where the
            // row binning covers it (at most 8192 bins across and down)
            BinGeom gg;
            if (bin_geometry(&b->grids[i], it.params.radius,
                             dense_cell_log2(it, b->geom[i].R, b->geom[i].s), &gg) == AUV_OK &&
                row_path_ok(gg) && (int64_t)gg.nbx * gg.nby <= (int64_t)1 << 24)
                b->geom[i] = gg;
        }
        // slice: the largest layout any form or autotune candidate may use
        size_t need = std::max(bin_workspace_layout(it.n, b->geom[i], nullptr, nullptr),
                               bin_workspace_layout(it.n, b->geom_plain[i], nullptr, nullptr));
        for (const Choice &cc : candidates(it, b->geom_plain[i].s)) {
            BinGeom gg;
            if (bin_geometry(&b->grids[i], it.params.radius, cc.bin_log2, &gg) == AUV_OK &&
                (int64_t)gg.nbx * gg.nby <= (int64_t)1 << 24)
                need = std::max(need, bin_workspace_layout(it.n, gg, nullptr, nullptr));
        }
        b->slice_size[i] = align256(need);
        max_tiles += most_units(it);
    }
    b->tables_bytes = align256(tables_size(count, max_tiles));
    off = b->tables_bytes;
    for (int i = 0; i < count; ++i) {
        b->slice_off[i] = off;
        off += b->slice_size[i];
    }
    b->ws_bytes = off;
    *out = b;
    return AUV_OK;
}

auv_status auv_batch_workspace_size(const auv_batch *batch, size_t *bytes)
{
    if (!batch || !bytes)
        return fail(AUV_ERR_INVALID, "null argument");
    *bytes = batch->ws_bytes;
    return AUV_OK;
}

auv_status auv_batch_item_plan(const auv_batch *batch, int32_t item, int32_t *bin_log2,
                               int32_t *algo, int32_t *tile_w, int32_t *tile_h)
{
    if (!batch || item < 0 || item >= (int32_t)batch->items.size())
        return fail(AUV_ERR_INVALID, "bad batch or item");
    if (bin_log2)
        *bin_log2 = batch->plan_bin[item];
    if (algo)
        *algo = batch->algo[item];
    if (tile_w)
        *tile_w = batch->tile[item].tile_w;
    if (tile_h)
        *tile_h = batch->tile[item].tile_h;
    return AUV_OK;
}

static auv_status check_ws(const auv_batch *b, void *ws, size_t ws_bytes)
{
    if (!b)
        return fail(AUV_ERR_INVALID, "batch is null");
    if (!ws || ws_bytes < b->ws_bytes)
        return fail(AUV_ERR_BUDGET, "workspace smaller than auv_batch_workspace_size");
    if ((reinterpret_cast<uintptr_t>(ws) & 255) != 0)
        return fail(AUV_ERR_INVALID, "workspace must be 256-byte aligned");
    return AUV_OK;
}

auv_status auv_batch_launch(auv_batch *b, void *ws, size_t ws_bytes, auv_stream stream)
{
    AUV_TRY_S(check_ws(b, ws, ws_bytes));
    hipStream_t st = static_cast<hipStream_t>(stream);
    char *base = static_cast<char *>(ws);
    if (b->exec && b->bound_ws == ws) {
        AUV_HIP(hipGraphLaunch(b->exec, st));
        return AUV_OK;
    }
    // (re)bind: tables for this workspace, then capture
    if (b->exec) {
        (void)hipGraphExecDestroy(b->exec);
        b->exec = nullptr;
    }
    if (b->graph) {
        (void)hipGraphDestroy(b->graph);
        b->graph = nullptr;
    }
    AUV_TRY_S(build_tables(b, base));
    const Tables t = table_ptrs(b, base);
    AUV_HIP(hipMemcpyAsync(t.rows, b->rows.data(), sizeof(RowItem) * b->rows.size(),
                           hipMemcpyHostToDevice, st));
    AUV_HIP(hipMemcpyAsync(t.idw, b->idw.data(), sizeof(IdwItem) * b->idw.size(),
                           hipMemcpyHostToDevice, st));
    AUV_HIP(hipMemcpyAsync(t.offs, b->offs.data(), sizeof(int32_t) * b->offs.size(),
                           hipMemcpyHostToDevice, st));
    if (!b->work.empty())
        AUV_HIP(hipMemcpyAsync(t.work, b->work.data(), sizeof(int2) * b->work.size(),
                               hipMemcpyHostToDevice, st));
    // the tables must be in place before any replay reads them
    AUV_HIP(hipStreamSynchronize(st));
    if (!b->cap_stream) {
        AUV_HIP(hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking));
        AUV_HIP(hipStreamCreateWithFlags(&b->cap_stream2, hipStreamNonBlocking));
        AUV_HIP(hipEventCreateWithFlags(&b->ev_fork, hipEventDisableTiming));
        AUV_HIP(hipEventCreateWithFlags(&b->ev_join, hipEventDisableTiming));
    }
    AUV_HIP(hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal));
    const auv_status es = enqueue_batched(b, base, b->cap_stream);
    hipGraph_t g = nullptr;
    const hipError_t ce = hipStreamEndCapture(b->cap_stream, &g);
    if (es != AUV_OK) {
        if (g)
            (void)hipGraphDestroy(g);
        return es;
    }
    if (ce != hipSuccess)
        return hip_fail(ce, "hipStreamEndCapture");
    b->graph = g;
    AUV_HIP(hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0));
    b->bound_ws = ws;
    AUV_HIP(hipGraphLaunch(b->exec, st));
    return AUV_OK;
}

auv_status auv_batch_launch_plain(auv_batch *b, void *ws, size_t ws_bytes, auv_stream stream)
{
    AUV_TRY_S(check_ws(b, ws, ws_bytes));
    hipStream_t st = static_cast<hipStream_t>(stream);
    char *base = static_cast<char *>(ws);
    for (int i = 0; i < (int)b->items.size(); ++i) {
        const auv_batch_item &it = b->items[i];
        BinWorkspace w;
        auv_bin_view bv;
        IdwArgs a;
        item_views(b, i, base, b->geom_plain[i], auto_algo(it), &w, &bv, &a);
        AUV_TRY_S(launch_binning(&b->grids[i], b->geom_plain[i], it.x, it.y, it.z, it.n, w, st));
        AUV_TRY_S(launch_idw(bv, a, st));
    }
    return AUV_OK;
}

auv_status auv_batch_autotune(const auv_batch_item *items, int32_t count, void *ws,
                              size_t ws_bytes, auv_stream stream, const char *tune_path)
{
    if (!tune_path)
        return fail(AUV_ERR_INVALID, "tune_path is null");
    auv_batch *b = nullptr;
    AUV_TRY_S(auv_batch_plan(items, count, nullptr, &b));
    struct Guard {
        auv_batch *b;
        ~Guard() { auv_batch_destroy(b); }
    } guard{b};
    AUV_TRY_S(check_ws(b, ws, ws_bytes));
    hipStream_t st = static_cast<hipStream_t>(stream);
    char *base = static_cast<char *>(ws);
    // one representative per class: the item with the most soundings
    std::map<ClassKey, int> rep;
    for (int i = 0; i < count; ++i) {
        const ClassKey k = class_of(b->items[i]);
        const auto f = rep.find(k);
        if (f == rep.end() || b->items[i].n > b->items[f->second].n)
            rep[k] = i;
    }
    hipEvent_t e0, e1;
    AUV_HIP(hipEventCreate(&e0));
    AUV_HIP(hipEventCreate(&e1));
    int dev = 0, cus = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    // the tables region of the workspace holds the throughput runs' work list
    size_t work_cap = 0;
    for (int k = 0; k < count; ++k)
        work_cap += most_units(b->items[k]);
    std::ostringstream table;
    table << "# auvgrid autotune table: class <log2 disk population> <log2 grid side> "
             "bin_log2 <s> algo <1 sparse | 2 dense> tile <nodes across> <nodes down> "
             "ms <time>\n";
    auv_status result = AUV_OK;
    for (const auto &kv : rep) {
        const int i = kv.second;
        const auv_batch_item &it = b->items[i];
        Choice best = with_default_tile(Choice{b->geom_plain[i].s, auto_algo(it)});
        float best_ms = 1e30f;
        // Time of a candidate in the setting it will run in: binning the item
        // (min of three rows of runs after one untimed), plus the batched kernel of
        // its form over enough repetitions of the item's tiles to fill the
        // chip (all reading the same bins), per repetition, and over the
        // item's tiles alone, by the item's share of the batch (a small batch
        // is its longest item's chain); items the
        // batched kernels do not cover get their own IDW launch instead.
        auto time_choice = [&](const Choice &c, float *out_ms) -> auv_status {
            *out_ms = 1e30f;
            BinGeom gg;
            if (bin_geometry(&b->grids[i], it.params.radius, c.bin_log2, &gg) != AUV_OK ||
                (int64_t)gg.nbx * gg.nby > (int64_t)1 << 24 ||
                bin_workspace_layout(it.n, gg, nullptr, nullptr) > b->slice_size[i])
                return AUV_OK;
            BinWorkspace w;
            auv_bin_view bv;
            IdwArgs a;
            item_views(b, i, base, gg, c.algo, &w, &bv, &a, c);
            auto min_of_runs = [&](auto &&enqueue, float *best) -> auv_status {
                *best = 1e30f;
                for (int rep_i = 0; rep_i < 4; ++rep_i) {
                    AUV_HIP(hipEventRecord(e0, st));
                    AUV_TRY_S(enqueue());
                    AUV_HIP(hipEventRecord(e1, st));
                    AUV_HIP(hipEventSynchronize(e1));
                    float ms = 0.0f;
                    AUV_HIP(hipEventElapsedTime(&ms, e0, e1));
                    if (rep_i > 0)
                        *best = std::min(*best, ms);
                }
                return AUV_OK;
            };
            float bin_ms, idw_ms;
            // (several in a row: one alone is launches and waits, whose scatter of a
            // microsecond exceeds what a small item's IDW takes in the batch)
            constexpr int kBinRuns = 16;
            AUV_TRY_S(min_of_runs(
                [&]() -> auv_status {
                    for (int r = 0; r < kBinRuns; ++r)
                        AUV_TRY_S(
                            launch_binning(&b->grids[i], gg, it.x, it.y, it.z, it.n, w, st));
                    return AUV_OK;
                },
                &bin_ms));
            // an item's binning leaves most of the chip to the other items of its batch
            // and is waited for with theirs: it counts by the share of the chip's blocks
            // (eight to a CU) that its largest launch takes, and by the item's share of
            // the batch.  Counted in full, the choice was that of the bins whose lone
            // binning is fastest: 64 tiles up to 256^2 139 us untuned, 151 tuned, now 130;
            // 150 tiles up to 128^2 240, 269, 226; 256 tiles 1626, 1780, 1582.
            const double bin_blocks = std::max<double>(gg.nby, row_scatter_blocks(it.n));
            bin_ms *= (float)(std::min(1.0, bin_blocks / (24.0 * cus) + 1.0 / count) / kBinRuns);
            IdwItem d;
            if (!make_idw_item(it, bv, a, c.algo, &d) || !row_path_ok(gg) || d.ntiles < 1) {
                AUV_TRY_S(min_of_runs([&] { return launch_idw(bv, a, st); }, &idw_ms));
                *out_ms = bin_ms + idw_ms;
                return AUV_OK;
            }
            const int64_t target = (int64_t)cus * 16 * 8;  // tiles: ~8 per resident wave
            const int copies = (int)std::max<int64_t>(
                1, std::min<int64_t>((target + d.ntiles - 1) / d.ntiles,
                                     (int64_t)work_cap / d.ntiles));
            const int nwork = copies * d.ntiles;
            std::vector<int2> work(nwork);
            for (int t = 0; t < nwork; ++t)
                work[t] = make_int2(0, t % d.ntiles);
            const Tables t = table_ptrs(b, base);
            AUV_HIP(hipMemcpyAsync(t.idw, &d, sizeof(d), hipMemcpyHostToDevice, st));
            AUV_HIP(hipMemcpyAsync(t.work, work.data(), sizeof(int2) * nwork,
                                   hipMemcpyHostToDevice, st));
            auto idw_time = [&](int units, float *ms) {
                return min_of_runs(
                    [&]() -> auv_status {
                        launch_form(d.form, d.pmode == 0, t.idw, t.work, units, st);
                        AUV_HIP(hipGetLastError());
                        return AUV_OK;
                    },
                    ms);
            };
            float alone_ms;
            AUV_TRY_S(idw_time(nwork, &idw_ms));
            AUV_TRY_S(idw_time(d.ntiles, &alone_ms));
            *out_ms = bin_ms + idw_ms / (float)copies + alone_ms / (float)count;
            return AUV_OK;
        };
        // bin size and form at the form's default tile, the untuned plan's choice among
        // them (the list form's bins of at least the radius are in no dense candidate),
        // then the other node tiles of the winner
        std::vector<Choice> cand = candidates(it, b->geom_plain[i].s);
        const Choice untuned{b->geom[i].s, b->algo[i]};
        if (untuned.algo != AUV_ALGO_SPAN &&
            std::none_of(cand.begin(), cand.end(), [&](const Choice &c) {
                return c.bin_log2 == untuned.bin_log2 && c.algo == untuned.algo;
            }))
            cand.push_back(untuned);
        for (const Choice &c0 : cand) {
            const Choice c = with_default_tile(c0);
            float ms;
            result = time_choice(c, &ms);
            if (result != AUV_OK)
                break;
            if (ms < best_ms) {
                best_ms = ms;
                best = c;
            }
        }
        if (result == AUV_OK && best_ms < 1e30f) {
            for (const Choice &c : tile_variants(best)) {
                float ms;
                result = time_choice(c, &ms);
                if (result != AUV_OK)
                    break;
                if (ms < best_ms) {
                    best_ms = ms;
                    best = c;
                }
            }
        }
        if (result != AUV_OK)
            break;
        table << "class " << kv.first.dens << " " << kv.first.side << " bin_log2 "
              << best.bin_log2 << " algo " << best.algo << " tile " << best.tile_w << " "
              << best.tile_h << " ms " << best_ms << "\n";
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (result != AUV_OK)
        return result;
    std::ofstream f(tune_path);
    if (!f)
        return fail(AUV_ERR_INVALID, std::string("cannot write ") + tune_path);
    f << table.str();
    return AUV_OK;
}

void auv_batch_destroy(auv_batch *b)
{
    if (!b)
        return;
    if (b->exec)
        (void)hipGraphExecDestroy(b->exec);
    if (b->graph)
        (void)hipGraphDestroy(b->graph);
    if (b->cap_stream)
        (void)hipStreamDestroy(b->cap_stream);
    if (b->cap_stream2)
        (void)hipStreamDestroy(b->cap_stream2);
    if (b->ev_fork)
        (void)hipEventDestroy(b->ev_fork);
    if (b->ev_join)
        (void)hipEventDestroy(b->ev_join);
    delete b;
}

}  // extern "C"
