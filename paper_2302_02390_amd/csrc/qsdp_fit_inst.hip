// Instantiations of the level fit for one shape; compiled with -DQSDP_FIT_V=<values per lane> and
// -DQSDP_FIT_W=<waves per batch>: buckets of up to 64 * V * W values; W = 1
// (qsdp_fit_kernel.hpp) or more (qsdp_fit_rounds.hpp).
#include "qsdp_launch.hpp"

#if !defined(QSDP_FIT_V) || !defined(QSDP_FIT_W)
#error "define QSDP_FIT_V and QSDP_FIT_W"
#endif

#if QSDP_FIT_W > 1
#include "qsdp_fit_rounds.hpp"
#else
#include "qsdp_fit_kernel.hpp"
#endif

#define QSDP_CAT2(a, b, c, d) a##b##c##d
#define QSDP_CAT(a, b, c, d) QSDP_CAT2(a, b, c, d)

namespace qsdp {

#if QSDP_FIT_W > 1
namespace kernels = fit_rounds;
#else
namespace kernels = qsdp;
#endif

namespace {

template <int BITS>
hipError_t go(const FitParams& p, unsigned grid, hipStream_t s) {
    hipLaunchKernelGGL((kernels::fit_levels_kernel<BITS, QSDP_FIT_V, QSDP_FIT_W>), dim3(grid),
                       dim3(kernels::FitShape<BITS, QSDP_FIT_V, QSDP_FIT_W>::kThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace

hipError_t QSDP_CAT(launch_fit_, QSDP_FIT_V, _, QSDP_FIT_W)(const FitParams& p, unsigned grid, hipStream_t s) {
    switch (p.bits) {
        case 1: return go<1>(p, grid, s);
        case 2: return go<2>(p, grid, s);
        case 3: return go<3>(p, grid, s);
        case 4: return go<4>(p, grid, s);
        case 5: return go<5>(p, grid, s);
        case 6: return go<6>(p, grid, s);
        case 7: return go<7>(p, grid, s);
        case 8: return go<8>(p, grid, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace qsdp
