// Launches of the one-map kernel (z3_multipoles_device.h) over window lists.
#include "z3_multipoles_device.h"

namespace z3 {

template <int M, bool PLANAR>
static void launch_mp(bool f32out, bool self, const MultArgs &a, hipStream_t s)
{
    dim3 grid(a.nblocks, a.groups.n), block(kBlock);
    if (f32out) {
        if (self) hipLaunchKernelGGL((k_multipoles<M, true, false, true, PLANAR, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_multipoles<M, true, false, false, PLANAR, true>), grid, block, 0, s, a);
    } else {
        if (self) hipLaunchKernelGGL((k_multipoles<M, false, false, true, PLANAR, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_multipoles<M, false, false, false, PLANAR, true>), grid, block, 0, s, a);
    }
}

z3_status launch_multipoles_list(int m_max, bool planar, bool mixed, bool self, const MultArgs &a, hipStream_t s)
{
    switch (m_max) {
#define Z3_CASE(MM) \
    case MM: planar ? launch_mp<MM, true>(mixed, self, a, s) : launch_mp<MM, false>(mixed, self, a, s); break;
        Z3_CASE(0) Z3_CASE(1) Z3_CASE(2) Z3_CASE(3) Z3_CASE(4) Z3_CASE(5) Z3_CASE(6) Z3_CASE(7)
        Z3_CASE(8) Z3_CASE(9) Z3_CASE(10) Z3_CASE(11) Z3_CASE(12) Z3_CASE(13) Z3_CASE(14)
        Z3_CASE(15) Z3_CASE(16)
#undef Z3_CASE
    default: return fail(Z3_ERR_UNSUPPORTED, "m_max=%d not compiled", m_max);
    }
    return check_launch("k_multipoles (window lists)");
}

}  // namespace z3
