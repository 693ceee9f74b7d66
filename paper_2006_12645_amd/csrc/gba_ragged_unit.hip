// Instantiations of the kernel for large requests outside the fast path
// (gba_kernel_ragged.hpp) with one operand-layout pair: compiled once per
// pair with GBA_LA, GBA_LB (0 = row-major, 1 = column-major).
#include "gba_tiles.hpp"

#if !defined(GBA_LA) || !defined(GBA_LB)
#error "gba_ragged_unit.hip needs GBA_LA and GBA_LB"
#endif

namespace gba {

#define GBA_RAGGED_ENTRY(id, BM, BN, WM, WN) \
    {&launch_ragged<BM, BN, WM, WN, GBA_LA, GBA_LB, false>, ragged_acc16<BM, BN, WM, WN, GBA_LA, GBA_LB>()},

template <>
LaunchFn ragged_entry<GBA_LA, GBA_LB>(int acc16, int tile)
{
    static const LaunchFn t[NUM_RAGGED][2] = {GBA_RAGGED_LIST(GBA_RAGGED_ENTRY)};
    return t[tile][acc16];
}

#undef GBA_RAGGED_ENTRY

}  // namespace gba
