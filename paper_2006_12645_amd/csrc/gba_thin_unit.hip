// Instantiations of the few-row kernel (gba_kernel_thin.hpp) in every
// operand layout.
#include "gba_tiles.hpp"

namespace gba {
namespace {

template <int LA, int LB>
LaunchFn pick(int tm, int tn)
{
    constexpr int T = LB == COL ? 1 : 2;   // the smallest blocks' columns, in 16s
    if (tm == 2) return &launch_thin<LA, LB, 2, 2 * T>;
    return tn == T ? &launch_thin<LA, LB, 1, T> : &launch_thin<LA, LB, 1, 2 * T>;
}

}  // namespace

LaunchFn thin_launcher(int la, int lb, int tm, int tn)
{
    if (la == ROW) return lb == ROW ? pick<ROW, ROW>(tm, tn) : pick<ROW, COL>(tm, tn);
    return lb == ROW ? pick<COL, ROW>(tm, tn) : pick<COL, COL>(tm, tn);
}

}  // namespace gba
