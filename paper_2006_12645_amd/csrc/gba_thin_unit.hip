// Instantiations of the few-row kernel (gba_kernel_thin.hpp) in every
// operand layout.
#include "gba_tiles.hpp"

namespace gba {
namespace {

template <int LA, int LB, int TN>
LaunchFn pick(int tm)
{
    return tm == 1 ? &launch_thin<LA, LB, 1, TN> : &launch_thin<LA, LB, 2, TN>;
}

template <int LA, int LB>
LaunchFn pick(int tm, int tn)
{
    if constexpr (LB == COL) {
        if (tn == 1) return pick<LA, LB, 1>(tm);
        return pick<LA, LB, 2>(tm);
    } else {
        if (tn == 2) return pick<LA, LB, 2>(tm);
        return pick<LA, LB, 4>(tm);
    }
}

}  // namespace

LaunchFn thin_launcher(int la, int lb, int tm, int tn)
{
    if (la == ROW) return lb == ROW ? pick<ROW, ROW>(tm, tn) : pick<ROW, COL>(tm, tn);
    return lb == ROW ? pick<COL, ROW>(tm, tn) : pick<COL, COL>(tm, tn);
}

}  // namespace gba
