// Instantiations of the tile kernel for one team shape; compiled with -DQSDP_TILE_W=<waves> -DQSDP_TILE_R=<rows>.
#include "qsdp_launch.hpp"

#if !defined(QSDP_TILE_W) || !defined(QSDP_TILE_R)
#error "define QSDP_TILE_W and QSDP_TILE_R"
#endif

#define QSDP_CAT4(a, b, c, d) a##b##c##d
#define QSDP_CAT(a, b, c, d) QSDP_CAT4(a, b, c, d)

namespace qsdp {
namespace {

template <int MODE>
hipError_t go(const Params& p, const TileArgs& a, unsigned grid, hipStream_t s) {
    const bool three = MODE == MODE_FUSED &&
                       three_workgroups_stream(p.bucket, a.buckets, QSDP_TILE_W, QSDP_TILE_R, p.n, p.segs != nullptr,
                                               p.g_half != 0u, p.codes != nullptr ? p.wbits : 0, p.delta > 0.0f);
    const unsigned unused_lds = three ? 32000u : 0u;
    hipLaunchKernelGGL((tile_kernel<MODE, QSDP_TILE_R, QSDP_TILE_W>), dim3(grid), dim3(256), unused_lds, s, p,
                       p.segs, a);
    return hipGetLastError();
}

}  // namespace

hipError_t QSDP_CAT(launch_tile_, QSDP_TILE_W, _, QSDP_TILE_R)(int mode, const Params& p, const TileArgs& a,
                                                               unsigned grid, hipStream_t s) {
    switch (mode) {
        case MODE_GRAD: return go<MODE_GRAD>(p, a, grid, s);
        case MODE_WEIGHT: return go<MODE_WEIGHT>(p, a, grid, s);
        case MODE_FUSED: return go<MODE_FUSED>(p, a, grid, s);
        case MODE_FUSED_CODES: return go<MODE_FUSED_CODES>(p, a, grid, s);
        case MODE_LEVELS: return go<MODE_LEVELS>(p, a, grid, s);
        case MODE_LEVELS_COIN: return go<MODE_LEVELS_COIN>(p, a, grid, s);
        case MODE_ADAMW: return go<MODE_ADAMW>(p, a, grid, s);
        case MODE_ADAMW_CODES: return go<MODE_ADAMW_CODES>(p, a, grid, s);
        case MODE_RECV: return go<MODE_RECV>(p, a, grid, s);
        case MODE_RECV_ADAMW: return go<MODE_RECV_ADAMW>(p, a, grid, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace qsdp
