// Host-side launch interface between the C ABI (qsdp_api.hip) and the kernel translation
// units. Wave kernels are instantiated per bucket shape in qsdp_wave_inst.hip, compiled
// once per (G, P) pair, tile kernels per team shape in qsdp_tile_inst.hip, the level fit per shape in qsdp_fit_inst.hip.
#pragma once

#include <hip/hip_runtime.h>

#include "qsdp_kernels.hpp"

namespace qsdp {

// One launcher per instantiated bucket size. `bits` is the width of the codes stored.
#define QSDP_DECLARE_WAVE(B) \
    hipError_t launch_wave_##B(int mode, int bits, const Params& p, unsigned grid, hipStream_t s);
QSDP_DECLARE_WAVE(128)
QSDP_DECLARE_WAVE(256)
QSDP_DECLARE_WAVE(512)
QSDP_DECLARE_WAVE(1024)
QSDP_DECLARE_WAVE(2048)
QSDP_DECLARE_WAVE(4096)
QSDP_DECLARE_WAVE(1024w2)  // weight quantizer only: two waves per 1024-bucket
#undef QSDP_DECLARE_WAVE

// One launcher per tile shape (waves, rows), see tile_plan.
#define QSDP_DECLARE_TILE(W, R) \
    hipError_t launch_tile_##W##_##R(int mode, const Params& p, const TileArgs& a, unsigned grid, hipStream_t s);
QSDP_DECLARE_TILE(1, 2)
QSDP_DECLARE_TILE(4, 2)
QSDP_DECLARE_TILE(1, 4)
QSDP_DECLARE_TILE(1, 6)
QSDP_DECLARE_TILE(1, 8)
QSDP_DECLARE_TILE(4, 4)
QSDP_DECLARE_TILE(4, 6)
QSDP_DECLARE_TILE(4, 8)
#undef QSDP_DECLARE_TILE

// One launcher per shape (values per lane, waves per batch) of the level fit.
#define QSDP_DECLARE_FIT(V, W) hipError_t launch_fit_##V##_##W(const FitParams& p, unsigned grid, hipStream_t s);
QSDP_DECLARE_FIT(2, 1)
QSDP_DECLARE_FIT(4, 1)
QSDP_DECLARE_FIT(8, 1)
QSDP_DECLARE_FIT(16, 1)
QSDP_DECLARE_FIT(32, 1)
QSDP_DECLARE_FIT(16, 4)
QSDP_DECLARE_FIT(16, 8)
#undef QSDP_DECLARE_FIT

hipError_t launch_dequant(int bits, bool bf16, const DequantParams& p, dim3 grid, hipStream_t s);
hipError_t launch_dequant_add(int bits, const DequantAddParams& p, unsigned grid, hipStream_t s);

}  // namespace qsdp
