// Gather IDW form: launcher.  The per-tile code is in idw_gather_impl.hpp.
#include "idw_gather_impl.hpp"

#include <algorithm>

namespace auv {

using namespace gather;

namespace {

// One wave per tile.  HIP takes fewer than 2^32 threads per launch, so a grid of
// 2^26 tiles or more (2^32 nodes) goes in pieces.
template <class K>
void launch_tiles(K *kernel, const auv_bin_view &bv, const IdwArgs &a, const WinGeom &g,
                  hipStream_t st)
{
    constexpr int64_t kPiece = int64_t(1) << 25;
    const int ntx = (a.nx + 7) / 8;
    const int64_t nt = (int64_t)ntx * ((a.ny + 7) / 8);
    for (int64_t t0 = 0; t0 < nt; t0 += kPiece)
        kernel<<<(unsigned)std::min(kPiece, nt - t0), 64, 0, st>>>(bv, a, g, ntx, (int)nt, (int)t0);
}

template <int kMode, bool kGen>
void launch_pmode(const auv_bin_view &bv, const IdwArgs &a, const WinGeom &g, hipStream_t st)
{
    if (kMode == 2 || a.pmode == 2)
        launch_tiles(k_idw_gather<kMode, 2, kGen>, bv, a, g, st);
    else if (a.pmode == 1)
        launch_tiles(k_idw_gather<kMode, 1, kGen>, bv, a, g, st);
    else if (a.pmode == 3)
        launch_tiles(k_idw_gather<kMode, 3, kGen>, bv, a, g, st);
    else
        launch_tiles(k_idw_gather<kMode, 0, kGen>, bv, a, g, st);
}

template <int kMode>
void launch_lattice(const auv_bin_view &bv, const IdwArgs &a, const WinGeom *g, hipStream_t st)
{
    if (g && gather_linear(*g, a.R))
        launch_pmode<kMode, false>(bv, a, *g, st);
    else
        launch_pmode<kMode, true>(bv, a, WinGeom{}, st);
}

template <int kMode>
void launch_top(const auv_bin_view &bv, const IdwArgs &a, const WinGeom *g, hipStream_t st)
{
    auto launch = [&](auto *linear, auto *general) {
        if (g && gather_linear(*g, a.R))
            launch_tiles(linear, bv, a, *g, st);
        else
            launch_tiles(general, bv, a, WinGeom{}, st);
    };
    if (a.max_pts <= 8)
        launch(k_idw_gather_top<kMode, 8, false>, k_idw_gather_top<kMode, 8, true>);
    else
        launch(k_idw_gather_top<kMode, 16, false>, k_idw_gather_top<kMode, 16, true>);
}

}  // namespace

bool gather_top_covers(const auv_bin_view &bv, const IdwArgs &a)
{
    return a.precision == AUV_P_FP32_REBASE && a.mode >= 1 && a.mode <= 3 && a.max_pts >= 1 &&
           a.max_pts <= 16 && gather_ok(a.R, bv.idx_bits, a.max_pts) &&
           (int64_t(1) << bv.bin_log2) >= a.R &&
           (int64_t)((a.nx + 7) / 8) * ((a.ny + 7) / 8) < (int64_t(1) << 31);
}

// The lists merge every candidate of a quarter, the ring search stops when the
// nearest bins have filled a node's list, so the search wins from some density on:
// later for lists of 8 (their merges cost half) and on grids of several waves per
// SIMD, where the lists' chain of batches is hidden.  Lists / search, whole IDW
// calls at 8, 20, 32, 48, 128, 256, 512 soundings per disk: 512^2 nodes, cap 8 0.68,
// 0.71, 0.74, 0.81, 0.86, 0.91, 0.71, cap 4 0.65, 0.71, 0.73, 0.80, 0.88, 0.79, 1.57,
// cap 16 (from 12 per disk) 0.89, 0.91, 0.94, 1.02, 1.14, 1.17, 1.21; 128^2 nodes,
// cap 8 0.86, 0.91, 0.97, 1.13, 1.15, 1.06, 1.10, cap 16 0.90, 1.00, 1.05, 1.20,
// 1.33, 1.39, 1.19; 64^2 and 256^2 as 128^2, 1024^2 as 512^2 or better.  Lists of 32
// lost throughout (1.03 to 1.3): caps above 16 take the search.
bool gather_top_pays(const IdwArgs &a)
{
    const bool large = (int64_t)a.nx * a.ny >= 4096 * 64;
    const float most = a.max_pts <= 8 ? (large ? 256.0f : 32.0f) : (large ? 40.0f : 20.0f);
    return a.population <= most;
}

auv_status launch_idw_gather_top(const auv_bin_view &bv, const IdwArgs &a, const WinGeom *g,
                                 hipStream_t st)
{
    switch (a.mode) {
    case 1: launch_top<1>(bv, a, g, st); break;
    case 2: launch_top<2>(bv, a, g, st); break;
    default: launch_top<3>(bv, a, g, st); break;
    }
    AUV_HIP(hipGetLastError());
    return AUV_OK;
}

bool gather_covers(const auv_bin_view &bv, const IdwArgs &a)
{
    return a.precision == AUV_P_FP32_REBASE && a.mode >= 1 && a.mode <= 3 &&
           gather_ok(a.R, bv.idx_bits, a.max_pts) &&
           (int64_t)((a.nx + 7) / 8) * ((a.ny + 7) / 8) < (int64_t(1) << 31);
}

auv_status launch_idw_gather(const auv_bin_view &bv, const IdwArgs &a, const WinGeom *g,
                             hipStream_t st)
{
    switch (a.mode) {
    case 1: launch_lattice<1>(bv, a, g, st); break;
    case 2: launch_lattice<2>(bv, a, g, st); break;
    default: launch_lattice<3>(bv, a, g, st); break;
    }
    AUV_HIP(hipGetLastError());
    return AUV_OK;
}

}  // namespace auv
