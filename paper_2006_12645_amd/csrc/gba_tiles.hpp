// gba_tiles.hpp -- the tile configurations compiled into the library and the
// launch-table types shared by the per-layout instantiation units and the
// host entry points.
//
// The paper generated one kernel per block/warp tile choice and kept the
// best per problem size (Experimental Evaluation section); this table is the
// MI355X counterpart of that tile space.  Block tiles are sized for the
// 160 KB LDS of a gfx950 compute unit (two stages of (BM + BN) x 64 fp16)
// and warp tiles for its 512 registers per lane.
#pragma once

#include <hip/hip_runtime.h>

#include "gba_kernel.hpp"
#include "gba_kernel16.hpp"
#include "gba_kernel_generic.hpp"
#include "gba_kernel_ragged.hpp"
#include "gba_kernel_thin.hpp"

namespace gba {

struct TileCfg {
    int bm, bn, wm, wn, sk, nstg;
};

// X(id, BM, BN, WM, WN, SK, NSTG): BM output rows x BN output columns per
// workgroup, WM x WN waves, each owning a (BM/WM) x (BN/WN) warp tile
// (multiples of 32 x 32, the MFMA block), times SK k-groups of waves that
// split each reduction step (intra-workgroup split-K; fp32 accumulation
// only); NSTG LDS stages.  32x128 and 128x32 have four waves of 32x32 (two of
// 64x32 before): one to a SIMD, fp16 accumulation 1.3-1.55x faster (its
// rounding chain is split over all four), fp32 0-8% (128 x 3968 x 6208 RR
// 24.9 -> 24.0 us, fp16 49.0 -> 31.9; 1024^3 CC 7.7 -> 7.4, fp16 11.4 -> 8.6).
#define GBA_TILE_LIST(X)         \
    X(0, 256, 256, 2, 2, 1, 2)   \
    X(1, 256, 256, 2, 4, 1, 2)   \
    X(2, 256, 128, 2, 2, 1, 2)   \
    X(3, 128, 256, 2, 2, 1, 2)   \
    X(4, 128, 128, 2, 2, 1, 2)   \
    X(5, 128, 64, 2, 2, 1, 2)    \
    X(6, 64, 64, 2, 2, 1, 2)     \
    X(7, 64, 128, 2, 2, 1, 2)    \
    X(8, 32, 64, 1, 2, 1, 2)     \
    X(9, 32, 32, 1, 1, 1, 2)     \
    X(10, 64, 64, 1, 1, 4, 2)    \
    X(11, 64, 64, 2, 2, 2, 4)    \
    X(12, 32, 64, 1, 1, 4, 2)    \
    X(13, 32, 32, 1, 1, 4, 4)    \
    X(14, 128, 128, 2, 2, 2, 2)  \
    X(15, 64, 128, 1, 2, 2, 2)   \
    X(16, 256, 128, 2, 4, 1, 2)  \
    X(17, 128, 256, 4, 2, 1, 2)  \
    X(18, 128, 128, 2, 4, 1, 2)  \
    X(19, 128, 64, 4, 2, 1, 2)   \
    X(20, 64, 128, 2, 4, 1, 2)   \
    X(21, 32, 64, 1, 2, 1, 4)    \
    X(22, 64, 64, 2, 2, 1, 4)    \
    X(23, 32, 32, 1, 1, 1, 4)    \
    X(24, 32, 128, 1, 4, 1, 4)   \
    X(25, 128, 32, 4, 1, 1, 4)

constexpr int NUM_TILES = 26;

#define GBA_TILE_CFG(id, BM, BN, WM, WN, SK, NSTG) TileCfg{BM, BN, WM, WN, SK, NSTG},
constexpr TileCfg TILES[NUM_TILES] = {GBA_TILE_LIST(GBA_TILE_CFG)};
#undef GBA_TILE_CFG

// Block tile of the general path (any size, leading dimension, alignment).
constexpr TileCfg GENERIC_TILE = {64, 64, 2, 2, 1, 2};

typedef hipError_t (*LaunchFn)(const GemmArgs &, hipStream_t);

// Tiles whose reduction can also be split across workgroups (fp32
// accumulation): one k-group and at most 128x128 outputs.  Larger tiles
// already fill the GPU with few output tiles.
constexpr bool tile_splits(const TileCfg &c) { return c.sk == 1 && c.bm * c.bn <= 128 * 128; }

// Deep variants of a tile: four computing and four copy-only waves on the
// 16x16x32 kernel, with as many LDS stages as fit one workgroup per compute
// unit (fp32 accumulation).  The library takes them where one round of
// workgroups covers the output (deep_choice in gba_api.hip); they answer to
// the id of the tile of the same shape and waves.  Sides of 128 or more are
// needed along an M- or N-contiguous operand, and with both operands
// M-contiguous the wide tile is wider in N (68.6 against 67.4 us on 8192 x
// 1024 x 4096; 39.0 / 36.6 on 4096 x 2048 x 2048).
enum { DEEP_WIDE, DEEP_SQUARE, DEEP_HALF, NUM_DEEP };

constexpr TileCfg deep_cfg(int la, int lb, int deep)
{
    if (deep == DEEP_SQUARE) return TileCfg{128, 128, 2, 2, 1, 4};
    if (deep == DEEP_WIDE) return la == COL && lb == COL ? TileCfg{128, 256, 2, 2, 1, 3} : TileCfg{256, 128, 2, 2, 1, 3};
    if (la == COL && lb == ROW) return TileCfg{0, 0, 0, 0, 0, 0};   // no half tile
    return la == ROW && lb == ROW ? TileCfg{64, 128, 2, 2, 1, 4} : TileCfg{128, 64, 2, 2, 1, 4};
}

constexpr int deep_tile(int la, int lb, int deep)
{
    const TileCfg c = deep_cfg(la, lb, deep);
    return deep == DEEP_SQUARE ? 4 : deep == DEEP_WIDE ? (c.bm > c.bn ? 2 : 3) : (c.bm > c.bn ? 5 : 7);
}

// Per operand-layout pair and kernel variant: fast[tile][acc16] for the
// aligned fast path (null for fp16 accumulation with split-K), split[tile]
// for its reduction split across workgroups (null where tile_splits is
// false), deep[variant] for its deep variants (null where there is none),
// generic[acc16] otherwise.
struct LayoutTable {
    LaunchFn fast[NUM_TILES][2];
    LaunchFn split[NUM_TILES];
    LaunchFn deep[NUM_DEEP];
    LaunchFn generic[2];
};

// Which tiles run the 16x16x32 kernel (gemm_bias_act_fast16): the ones
// with eight waves of one k-group, in every layout where an M- or
// N-contiguous operand tile has 128 or more elements per row (its
// conflict-free group permutation needs eight 16-element groups); the deep
// variants (deep_cfg); and,
// without prologue, the four-stage small tiles (21-25) under the same layout condition (all
// of them in the layout where both operand tiles are reduction-contiguous,
// 32x128 with row-major B, 128x32 with column-major A), where the 16x16x32
// kernel adds waves that only issue copies (with fp16 accumulation its
// fp16 running sum also breaks the chain of dependent MFMAs).  With fp32
// accumulation that is 6-10% faster than these tiles on 32x32x16 without
// copy-only waves, and than the k-group tiles on 1024^3 in RC (6.66 against
// 7.33 us) and 1000^3 (6.99 against 7.75); in RR, 32x128 takes 1024^3 in
// 7.84 us against 8.78 on the k-group 64x64 tile.
constexpr bool use_fast16(int la, int lb, int bm, int bn, int wm, int wn, int sk, int nstg, bool acc16, bool pro,
                          bool split = false)
{
    const bool layouts = (bm >= 128 || la == ROW) && (bn >= 128 || lb == COL);
    if (wm * wn == 8) return layouts;
    if (bm * bn >= 128 * 64 && nstg >= 3) return layouts && !acc16 && !split;   // deep variants
    return !pro && sk == 1 && nstg == 4 && layouts;
}

// Threads of a workgroup of a tile's kernel.
constexpr int tile_threads(int la, int lb, const TileCfg &c, bool acc16, bool pro, bool split)
{
    const bool fast16 = use_fast16(la, lb, c.bm, c.bn, c.wm, c.wn, c.sk, c.nstg, acc16, pro, split);
    return 64 * (c.wm * c.wn * c.sk + (fast16 ? copy_only_waves(c.wm, c.wn, c.sk) : 0));
}

// hipGetLastError reports the last failure of any runtime call on the
// calling thread, not only of the launch before it: the launchers clear it
// first, so that an earlier, unrelated failure does not turn a kernel that
// was enqueued (and will run) into an error return.
inline void clear_last_error() { (void)hipGetLastError(); }

template <int BM, int BN, int WM, int WN, int SK, int NSTG, int LA, int LB, bool ACC16, bool PRO, bool DUAL,
          bool SPLIT = false>
hipError_t launch_fast(const GemmArgs &a, hipStream_t s)
{
    // one workgroup per output tile, times the splits of its reduction
    constexpr int NT = tile_threads(LA, LB, TileCfg{BM, BN, WM, WN, SK, NSTG}, ACC16, PRO, SPLIT);
    dim3 grid((unsigned)(a.tiles_m * a.tiles_n * (SPLIT ? a.splits : 1))), block(NT);
    // The 8-wave tiles (one k-group) run on 16x16x32 MFMAs, and so do the
    // four-stage small tiles where use_fast16 allows them;
    // everything else on 32x32x16 (measured per tile: the 16x16x32 kernels
    // of the 4-wave tiles were up to 20% slower with fp32 accumulation, and
    // the 4-wave 256x256 one does not fit its 64 accumulator blocks per wave
    // in registers)
    clear_last_error();
    if constexpr (use_fast16(LA, LB, BM, BN, WM, WN, SK, NSTG, ACC16, PRO, SPLIT))
        hipLaunchKernelGGL((gemm_bias_act_fast16<BM, BN, WM, WN, SK, NSTG, LA, LB, ACC16, PRO, DUAL, SPLIT>), grid,
                           block, 0, s, a);
    else
        hipLaunchKernelGGL((gemm_bias_act_fast<BM, BN, WM, WN, SK, NSTG, LA, LB, ACC16, PRO, DUAL, SPLIT>), grid,
                           block, 0, s, a);
    return hipGetLastError();
}

// Launch-table entry for fp16 accumulation: none with split-K.
template <int BM, int BN, int WM, int WN, int SK, int NSTG, int LA, int LB, bool PRO, bool DUAL>
constexpr LaunchFn fast_acc16()
{
    if constexpr (SK == 1) return &launch_fast<BM, BN, WM, WN, SK, NSTG, LA, LB, true, PRO, DUAL>;
    else return nullptr;
}

// Launch-table entry for a reduction split across workgroups.
template <int BM, int BN, int WM, int WN, int SK, int NSTG, int LA, int LB, bool PRO, bool DUAL>
constexpr LaunchFn fast_split()
{
    if constexpr (tile_splits(TileCfg{BM, BN, WM, WN, SK, NSTG}))
        return &launch_fast<BM, BN, WM, WN, SK, NSTG, LA, LB, false, PRO, DUAL, true>;
    else return nullptr;
}

// Launch-table entry for a deep variant.
template <int LA, int LB, bool PRO, bool DUAL, int DEEP>
constexpr LaunchFn fast_deep()
{
    constexpr TileCfg c = deep_cfg(LA, LB, DEEP);
    if constexpr (c.bm > 0) return &launch_fast<c.bm, c.bn, c.wm, c.wn, c.sk, c.nstg, LA, LB, false, PRO, DUAL>;
    else return nullptr;
}

template <int LA, int LB, bool ACC16, bool PRO, bool DUAL>
hipError_t launch_generic(const GemmArgs &a, hipStream_t s)
{
    constexpr TileCfg c = GENERIC_TILE;
    dim3 grid((unsigned)(a.tiles_m * a.tiles_n)), block(64 * c.wm * c.wn);
    clear_last_error();
    hipLaunchKernelGGL((gemm_bias_act_generic<c.bm, c.bn, c.wm, c.wn, LA, LB, ACC16, PRO, DUAL>),
                       grid, block, 0, s, a);
    return hipGetLastError();
}

// The few-row kernel, for one layout pair (the prologue and the second
// product are run-time options there): thin_launcher(LA, LB, TM, TN), TM row
// blocks of 16 by TN column blocks of 16: 1x1, 1x2 or 2x2 with column-major
// B, 1x2, 1x4 or 2x4 with row-major B.
template <int LA, int LB, int TM, int TN>
hipError_t launch_thin(const GemmArgs &a, hipStream_t s)
{
    dim3 grid((unsigned)(a.tiles_m * a.tiles_n)), block(64 * a.waves);
    clear_last_error();
    hipLaunchKernelGGL((gemm_bias_act_thin<LA, LB, TM, TN>), grid, block, 0, s, a);
    return hipGetLastError();
}

LaunchFn thin_launcher(int la, int lb, int tm, int tn);

// Block tiles of the kernel for large requests outside the fast path
// (gba_kernel_ragged.hpp): BM, BN, WM, WN.
#define GBA_RAGGED_LIST(X) \
    X(0, 256, 256, 2, 4)   \
    X(1, 128, 128, 2, 4)   \
    X(2, 64, 64, 2, 2)

constexpr int NUM_RAGGED = 3;

#define GBA_RAGGED_CFG(id, BM, BN, WM, WN) TileCfg{BM, BN, WM, WN, 1, 2},
constexpr TileCfg RAGGED_TILES[NUM_RAGGED] = {GBA_RAGGED_LIST(GBA_RAGGED_CFG)};
#undef GBA_RAGGED_CFG

template <int BM, int BN, int WM, int WN, int LA, int LB, bool ACC16>
hipError_t launch_ragged(const GemmArgs &a, hipStream_t s)
{
    dim3 grid((unsigned)(a.tiles_m * a.tiles_n)), block(64 * WM * WN);
    clear_last_error();
    hipLaunchKernelGGL((gemm_bias_act_ragged<BM, BN, WM, WN, LA, LB, ACC16>), grid, block, 0, s, a);
    return hipGetLastError();
}

// Launch-table entry for fp16 accumulation: none on the 256x256 tile.
template <int BM, int BN, int WM, int WN, int LA, int LB>
constexpr LaunchFn ragged_acc16()
{
    if constexpr (BM * BN <= 128 * 128) return &launch_ragged<BM, BN, WM, WN, LA, LB, true>;
    else return nullptr;
}

template <int LA, int LB>
LaunchFn ragged_entry(int acc16, int tile);

// Host-side launch table of one layout pair (LA, LB) and variant: PRO = ReLU
// prologue on the left operands, DUAL = a second product.  Each
// specialisation is defined in its own instantiation unit
// (gba_gemm_unit.hip compiled once per combination).
template <int LA, int LB, bool PRO, bool DUAL>
const LayoutTable &layout_table();

}  // namespace gba
