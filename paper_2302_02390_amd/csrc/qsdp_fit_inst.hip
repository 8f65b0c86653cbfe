// Instantiations of the level fit for one shape; compiled with -DQSDP_FIT_V=<values per lane> and
// -DQSDP_FIT_W=<waves per batch>: buckets of up to 64 * V * W values.
#include "qsdp_launch.hpp"

#if !defined(QSDP_FIT_V) || !defined(QSDP_FIT_W)
#error "define QSDP_FIT_V and QSDP_FIT_W"
#endif

#define QSDP_CAT2(a, b, c, d) a##b##c##d
#define QSDP_CAT(a, b, c, d) QSDP_CAT2(a, b, c, d)

namespace qsdp {

hipError_t QSDP_CAT(launch_fit_, QSDP_FIT_V, _, QSDP_FIT_W)(const FitParams& p, unsigned grid, hipStream_t s) {
    const dim3 block(FitShape<1, QSDP_FIT_V, QSDP_FIT_W>::kThreads);
    switch (p.bits) {
        case 1: hipLaunchKernelGGL((fit_levels_kernel<1, QSDP_FIT_V, QSDP_FIT_W>), dim3(grid), block, 0, s, p); break;
        case 2: hipLaunchKernelGGL((fit_levels_kernel<2, QSDP_FIT_V, QSDP_FIT_W>), dim3(grid), block, 0, s, p); break;
        case 3: hipLaunchKernelGGL((fit_levels_kernel<3, QSDP_FIT_V, QSDP_FIT_W>), dim3(grid), block, 0, s, p); break;
        case 4: hipLaunchKernelGGL((fit_levels_kernel<4, QSDP_FIT_V, QSDP_FIT_W>), dim3(grid), block, 0, s, p); break;
        case 5: hipLaunchKernelGGL((fit_levels_kernel<5, QSDP_FIT_V, QSDP_FIT_W>), dim3(grid), block, 0, s, p); break;
        case 6: hipLaunchKernelGGL((fit_levels_kernel<6, QSDP_FIT_V, QSDP_FIT_W>), dim3(grid), block, 0, s, p); break;
        case 7: hipLaunchKernelGGL((fit_levels_kernel<7, QSDP_FIT_V, QSDP_FIT_W>), dim3(grid), block, 0, s, p); break;
        case 8: hipLaunchKernelGGL((fit_levels_kernel<8, QSDP_FIT_V, QSDP_FIT_W>), dim3(grid), block, 0, s, p); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace qsdp
