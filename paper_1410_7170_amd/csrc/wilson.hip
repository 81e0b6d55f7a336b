// Launch of the Wilson stencil kernels (wilson.h, wilson_tile.h): blocks of 64 or
// 256 sites (192 or 256 for the streaming form, up to 512 for the tile form),
// ordered (site block, RHS) and spread over the XCDs by the kernel itself.
#include <algorithm>

#include "internal.h"

namespace ovl {

template <int PREC, int WPE, bool STAGE, int NT = kBlock, bool TILED = false>
static void wilson_ts_dispatch_s(int mode, bool g5, dim3 grid, const WArgs &a, hipStream_t st, hipEvent_t e0,
                                 hipEvent_t e1)
{
    const dim3 b(NT);
    if (g5) {
        switch (mode) {
        case W_PLAIN: launch_k(k_wilson_ts<PREC, W_PLAIN, true, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a); break;
        case W_NORM: launch_k(k_wilson_ts<PREC, W_NORM, true, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a); break;
        case W_SHIFT: launch_k(k_wilson_ts<PREC, W_SHIFT, true, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a); break;
        case W_RUPDATE:
            launch_k(k_wilson_ts<PREC, W_RUPDATE, true, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a);
            break;
        case W_RUPDATE0:
            launch_k(k_wilson_ts<PREC, W_RUPDATE0, true, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a);
            break;
        case W_SNORM: launch_k(k_wilson_ts<PREC, W_SNORM, true, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a); break;
        case W_LZ1:
        case W_LZ2:
        case W_LZ3:
            if constexpr (PREC == P_F64) {
                if (mode == W_LZ1) launch_k(k_wilson_ts<PREC, W_LZ1, true, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a);
                else if (mode == W_LZ2) launch_k(k_wilson_ts<PREC, W_LZ2, true, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a);
                else launch_k(k_wilson_ts<PREC, W_LZ3, true, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a);
            }
            break;
        default: launch_k(k_wilson_ts<PREC, W_RESNORM, true, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a); break;
        }
    } else {
        launch_k(k_wilson_ts<PREC, W_PLAIN, false, WPE, STAGE, NT, TILED>, grid, b, st, e0, e1, a);
    }
}

// Blocks of whole x3 rows of consecutive x2 at one x1 take the one-wave build
// that stages each slice in LDS, at any grid size (at 32^3x64 it beats the
// two-wave build for one field, 411 against 456 us in FP64, and for batches
// of 7 fields, 2.7 against 2.9 ms); 48-bit fields, whose loaded words need
// fewer registers, take the staged two-wave build on grids of more than 256
// blocks (stencil_shape sizes them for it); blocks of 192 threads (nt, from
// stream_threads) exist only for that build.  Otherwise launches of at most
// 512 blocks take the one-wave build without staging, larger grids the
// two-wave build.  A block holds nt >> kr sites (K = 2^kr lanes per site).
static bool staged_rows(const Geom &g, int sites)
{
    return sites % g.L[3] == 0 && (g.L[2] * g.L[3]) % sites == 0;
}

template <int PREC>
static void wilson_ts_dispatch(int mode, bool g5, dim3 grid, int nt, const WArgs &a, hipStream_t st, hipEvent_t e0,
                               hipEvent_t e1)
{
    // 192-thread blocks (three waves) in FP64 take the build capped at two
    // waves per SIMD: the one-wave build needs more than 256 registers, so a
    // block holds three of a CU's four SIMDs and the fourth idles (24^3x48,
    // 12 RHS: 1489 -> 1252 us, with a few spilled registers); FP32 measured the
    // same either way
    constexpr int W192 = PREC == P_F64 || PREC == P_F48 ? 2 : 1;
    if (a.kr > 0) {
        // RHS tiles: staged builds only (stencil_shape guarantees whole rows)
        if (nt == 192) wilson_ts_dispatch_s<PREC, W192, true, 192, true>(mode, g5, grid, a, st, e0, e1);
        else wilson_ts_dispatch_s<PREC, 1, true, kBlock, true>(mode, g5, grid, a, st, e0, e1);
        return;
    }
    if (nt == 192) {
        wilson_ts_dispatch_s<PREC, W192, true, 192>(mode, g5, grid, a, st, e0, e1);
        return;
    }
    if (staged_rows(a.g, nt)) {
        if (PREC == P_F48 && grid.x > 256) wilson_ts_dispatch_s<PREC, 2, true>(mode, g5, grid, a, st, e0, e1);
        else wilson_ts_dispatch_s<PREC, 1, true>(mode, g5, grid, a, st, e0, e1);
    } else if (grid.x <= 512) {
        wilson_ts_dispatch_s<PREC, 1, false>(mode, g5, grid, a, st, e0, e1);
    } else {
        wilson_ts_dispatch_s<PREC, 2, false>(mode, g5, grid, a, st, e0, e1);
    }
}

// The streaming form's shape.  The RHS tile K is the lattice's rhs_tile,
// capped at the next power of two of nrhs, and halved until the block's
// sites times the stream length cover at least 256 site-slices (so the
// blocks of one tile fit the 2 nb partial-sum slots per RHS) and the block's
// sites are whole x3 rows (tiles run in the LDS-staged build only).
static StencilShape stencil_shape_ts(const Lat &L, int ts, int nrhs)
{
    StencilShape sh{};
    const int nt = stream_threads(L.g, ts);
    int kr = L.g.Kr;
    while (kr > 0 && (1 << (kr - 1)) >= nrhs) kr--;   // K <= next power of two of nrhs
    while (kr > 0 && ((nt >> kr) * ts < 256 || !staged_rows(L.g, nt >> kr))) kr--;
    sh.ts = ts;
    sh.nt = nt;
    sh.kr = kr;
    sh.blocks_per_tile = (int)(L.V / ((int64_t)(nt >> kr) * ts));
    sh.ntile = (nrhs + (1 << kr) - 1) >> kr;
    return sh;
}

// Blocks of the one-site form: one wave each where a launch leaves no partial
// sums and has no more than kWaveWork sites on all its fields, so that they spread
// evenly over the CUs (a wave reads 70 to 150 KB through its CU's L1: D_W at 12^3x20
// with 4 RHS FP64 26.8 us with four waves a block, 22.5 with one, FP32 13.0 and
// 10.0; at 140000 sites 1.24 times as fast in FP32, 1.13 in FP64; from 280000 on
// 0.97 to 1.01; on 48-bit fields 1.03 to 1.08 at 105000 sites, 0.91 to 1.10 from
// 131072 on).  With partial sums up to kWaveSites sites, whose sums are then at
// most one slot to each of the 256 strided sums; beyond, every wave of a carried
// stage adds up more (four waves a block / one, FP64 and mixed overlap apply, ms:
// 8x12^3 3.77 / 3.42, 3.55 / 3.57; 10x12^3 4.06 / 3.90, 3.79 / 3.94;
// 12^4 4.15 / 4.12, 3.95 / 4.23; 20x12^3 5.25 / 6.05, 4.70 / 5.80).  The two waves
// per parity of 4^4 gain nothing apart, those of anything larger do (Q^2 in us:
// 4^4 12.95 / 13.1, 6x4^3 13.8 / 12.8, 8x4^3 15.3 / 13.7, 6^4 17.2 / 14.3); FP16
// fields gain from 2000 sites on (6^4 12.8 / 13.3, 10x6^3 1.05 times as fast).
constexpr int64_t kWaveSites = 64 * 256;
constexpr int64_t kWaveWork = 1 << 18, kWaveWork48 = (1 << 17) - 1;
constexpr int64_t kTwoWaves = 256, kFew16 = 2047;

static int site_threads(const Lat &L, bool sums, int prec = P_F64, int nrhs = 1)
{
    const bool many = sums ? L.V > kWaveSites : L.V * nrhs > (prec == P_F48 ? kWaveWork48 : kWaveWork);
    return L.V <= (prec == P_F16S ? kFew16 : kTwoWaves) || many ? kBlock : 64;
}

static bool mode_sums(int mode)
{
    return mode == W_NORM || mode == W_RUPDATE || mode == W_RUPDATE0 || mode == W_RESNORM || mode == W_SNORM ||
           mode == W_LZ1;
}

static int blocks_of(const Lat &L, int nt) { return 2 * ((L.Vh + nt - 1) / nt); }

// Every block of a carrying launch adds up all of the previous one's partial
// sums, and their reads grow with the square of the lattice; up to two slots for
// each of the 256 strided sums a launch that carries is faster everywhere (stages
// in kernels of their own / carried, FP64 and mixed overlap apply, ms: 16x10^3
// 4.53 / 3.94, 4.69 / 4.01; 20x16^3 10.4 / 9.23, 8.61 / 7.34; 32x16^3 13.3 / 12.1,
// 11.0 / 9.81; 24x18^3, 432 slots, 16.6 / 15.4, 13.8 / 13.3).  Beyond, several RHS
// can lose (26x22^2x20, tiles, 1573 slots, mixed: 21.7 / 21.1, 3 RHS 51.9 / 52.8).
constexpr int kCarrySlots = 512;

// 48-bit fields take the FP64 length, halved while the launch has fewer than
// 512 blocks: their staged build runs two waves per SIMD (wilson_ts_dispatch),
// which needs two blocks per CU (at 32^3x64: 16 slices and 512 blocks, the mixed
// solver's 48-bit stencils 381 -> 367 us (t update) and 382 -> 353 us (residual
// update) against one wave at 32 slices; FP64 itself spills at two waves and
// keeps one)
StencilShape stencil_shape(const Lat &L, int prec, int nrhs, bool sums)
{
    const int ts = (prec == P_F64 || prec == P_F48) && L.g.Ts64 > 0 ? L.g.Ts64 : L.g.Ts;
    if (ts <= 0 || prec == P_F16S) {
        StencilShape sh{};
        if ((prec == P_F64 || prec == P_F48) &&
            tile_pays(L.tile, prec == P_F64, nrhs, sums, tile_count(L.tile) <= kCarrySlots))
            sh.tile = L.tile;
        sh.nt = site_threads(L, true);
        return sh;
    }
    StencilShape sh = stencil_shape_ts(L, ts, nrhs);
    while (prec == P_F48 && sh.ts % 2 == 0 && (int64_t)sh.blocks_per_tile * sh.ntile < 512)
        sh = stencil_shape_ts(L, sh.ts / 2, nrhs);
    return sh;
}

int stencil_partials(const Lat &L, int prec, int nrhs)
{
    const StencilShape sh = stencil_shape(L, prec, nrhs);
    return sh.ts > 0 ? sh.blocks_per_tile : sh.tile.nt ? tile_count(sh.tile) : blocks_of(L, sh.nt);
}

int part_stride(const Lat &L)
{
    return std::max(blocks_of(L, site_threads(L, true)), L.tile.nt ? tile_count(L.tile) : 0);
}

bool carries_scalars(const Lat &L, int prec, int nrhs)
{
    return stencil_shape(L, prec, nrhs).ts == 0 && stencil_partials(L, prec, nrhs) <= kCarrySlots;
}

template <int PREC, int MODE, bool G5>
static void launch_site(dim3 grid, int nt, const WArgs &a, const ProArgs &pro, hipStream_t st, hipEvent_t e0,
                        hipEvent_t e1)
{
    if (nt == kBlock) launch_k(k_wilson<PREC, MODE, G5, kBlock>, grid, dim3(kBlock), st, e0, e1, a, pro);
    else launch_k(k_wilson<PREC, MODE, G5, 64>, grid, dim3(64), st, e0, e1, a, pro);
}

template <int PREC>
static void wilson_dispatch(int mode, bool g5, dim3 grid, int nt, const WArgs &a, const ProArgs &pro, hipStream_t st,
                            hipEvent_t e0, hipEvent_t e1)
{
    if (!g5) {
        launch_site<PREC, W_PLAIN, false>(grid, nt, a, pro, st, e0, e1);
        return;
    }
    switch (mode) {
    case W_PLAIN: launch_site<PREC, W_PLAIN, true>(grid, nt, a, pro, st, e0, e1); break;
    case W_NORM: launch_site<PREC, W_NORM, true>(grid, nt, a, pro, st, e0, e1); break;
    case W_SHIFT: launch_site<PREC, W_SHIFT, true>(grid, nt, a, pro, st, e0, e1); break;
    case W_RUPDATE: launch_site<PREC, W_RUPDATE, true>(grid, nt, a, pro, st, e0, e1); break;
    case W_RUPDATE0: launch_site<PREC, W_RUPDATE0, true>(grid, nt, a, pro, st, e0, e1); break;
    case W_SNORM: launch_site<PREC, W_SNORM, true>(grid, nt, a, pro, st, e0, e1); break;
    case W_LZ1:
    case W_LZ2:
    case W_LZ3:
        if constexpr (PREC == P_F64) {
            if (mode == W_LZ1) launch_site<PREC, W_LZ1, true>(grid, nt, a, pro, st, e0, e1);
            else if (mode == W_LZ2) launch_site<PREC, W_LZ2, true>(grid, nt, a, pro, st, e0, e1);
            else launch_site<PREC, W_LZ3, true>(grid, nt, a, pro, st, e0, e1);
        }
        break;
    default: launch_site<PREC, W_RESNORM, true>(grid, nt, a, pro, st, e0, e1); break;
    }
}

// RHS tiles in a group of the streaming form: all, or at most three where that
// pays, the groups alike.  A die holds 32 (48-bit: 64) of its blocks at a time;
// with every RHS of a block of sites side by side these span 8192 / nrhs sites, and
// where that is little more than an x1 plane the x1 neighbours miss L2; with one
// RHS after the other the links do (D_W, 12 FP32 RHS at 24^3x48: 2.92 GB fetched
// side by side, 2.41 in groups).  From 2^20 sites on fewer RHS gain too, FP32
// apart; FP32 and 48-bit fields lose where the last group is not full (7 RHS: 0.97
// at 32^4 and 16^2x64x32).  Rates of groups of three over all side by side, D_W
// (FP32, 48-bit, FP64):
//                       plane  4 RHS           6 RHS           12 RHS
//   8x32^3     2^18     1024                                   0.96 0.95 1.00
//   32x64x16x32 2^20     512   0.99 0.97 0.98  0.99 0.99 1.00  0.99 1.03 1.03
//   48x24^3    0.7 M     576   0.98 1.00 1.00  1.01 1.00 1.01  1.01 0.99 1.02
//   20x32^2x24 0.5 M     768   0.97 0.97 0.96  0.98 0.97 0.99  1.00 0.99 1.01
//   36x24^2x32 0.7 M     768   0.98 0.98 0.99  0.99 0.98 1.01  1.01 1.01 1.07
//   16x32^3    2^19     1024   1.00 0.99 1.02  1.00 1.00 1.03  0.99 1.00 1.06
//   32^4       2^20     1024   0.99 1.01 1.03  1.00 1.04 1.05  1.07 1.11 1.15
//   48x32^3    1.6 M    1024   0.98 1.00 1.04  1.01 1.05 1.11  1.11 1.22 1.27
//   40^2x24x32 1.2 M     768   0.98 1.00 1.00  1.00 1.02 1.04  1.04 1.11 1.20
//   16x48x32x48 1.2 M   1536   1.01 1.04 1.09  1.02 1.05 1.11  1.12 1.13 1.19
//   16^2x64x32 2^19     2048   1.02 1.02 1.03  1.01 1.01 1.09  1.00 1.07 1.10
// (Three: 12 RHS at 32^4 in groups of 12 / 1 / 2 / 3 / 4 / 6, FP64 us 2416 / 2161 / 2093
// / 2103 / 2126 / 2128.)
static int group_tiles(const Lat &L, int prec, int nrhs, int ntile)
{
    const int64_t plane = (int64_t)L.g.L[2] * L.g.L[3];
    const bool large = prec != P_F32 && L.V >= 1 << 20 && plane >= 768;
    const bool wide = L.V >= 1 << 19 && nrhs * plane > 6144 && (prec == P_F64 || ntile % 3 == 0);
    if (!large && !wide) return ntile;
    const int groups = (ntile + 2) / 3;
    return (ntile + groups - 1) / groups;
}

hipError_t launch_wilson(const Lat &L, int prec, int mode, bool g5, WArgs a, hipStream_t st, hipEvent_t e0,
                         hipEvent_t e1, const ProArgs *pro)
{
    const ProArgs pa = pro ? *pro : ProArgs{};
    if (mode >= W_LZ1 && prec != P_F64) return hipErrorInvalidValue;
    a.g = L.g;
    a.nblk = part_stride(L);
    a.kr = 0;
    if (prec == P_F32 && mode == W_PLAIN && L.g.Mfma && a.nrhs >= 2) {
        // the matrix-core form: events as markers around its launch
        if (e0) {
            const hipError_t h0 = hipEventRecord(e0, st);
            if (h0 != hipSuccess) return h0;
        }
        const hipError_t h = launch_wilson_mfma(L, g5, a, st);
        if (h == hipSuccess && e1) return hipEventRecord(e1, st);
        return h;
    }
    const StencilShape sh = stencil_shape(L, prec, a.nrhs, mode_sums(mode) || mode >= W_LZ1);
    if (sh.ts > 0) {
        // time-streaming form (FP64, 48-bit, FP32): blocks_per_tile blocks per RHS
        // tile; the FP16 stencil keeps one site per thread, which measured
        // faster
        if (sh.blocks_per_tile > a.nblk || pa.kind) return hipErrorInvalidConfiguration;
        a.kr = sh.kr;
        a.grp = group_tiles(L, prec, a.nrhs, sh.ntile);
        if (prec == P_F48) a.g.Ts64 = sh.ts;   // the kernel reads its length from there
        dim3 grid((unsigned)sh.blocks_per_tile * sh.ntile);
        if (prec == P_F64) wilson_ts_dispatch<P_F64>(mode, g5, grid, sh.nt, a, st, e0, e1);
        else if (prec == P_F48) wilson_ts_dispatch<P_F48>(mode, g5, grid, sh.nt, a, st, e0, e1);
        else wilson_ts_dispatch<P_F32>(mode, g5, grid, sh.nt, a, st, e0, e1);
        return hipGetLastError();
    }
    const int extra = pa.kind ? a.nrhs : 0;   // blocks of the scalar stage
    if (sh.tile.nt) {
        dim3 grid((unsigned)tile_count(sh.tile) * a.nrhs + extra);
        return launch_wilson_tile(prec, mode, g5, grid, a, sh.tile, pa, st, e0, e1);
    }
    const int nt = mode_sums(mode) ? sh.nt : site_threads(L, false, prec, a.nrhs);
    dim3 grid(blocks_of(L, nt) * a.nrhs + extra);
    if (prec == P_F64) wilson_dispatch<P_F64>(mode, g5, grid, nt, a, pa, st, e0, e1);
    else if (prec == P_F48) wilson_dispatch<P_F48>(mode, g5, grid, nt, a, pa, st, e0, e1);
    else if (prec == P_F32) wilson_dispatch<P_F32>(mode, g5, grid, nt, a, pa, st, e0, e1);
    else wilson_dispatch<P_F16S>(mode, g5, grid, nt, a, pa, st, e0, e1);
    return hipGetLastError();
}

}  // namespace ovl
