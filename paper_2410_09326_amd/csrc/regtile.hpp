// Launches of one register tile variant (defined in the variant's own object,
// see regtile.hip), and the variants that are built.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "devprog.hpp"

namespace qops {

// (R, W): register and wave bits; the build script compiles each for both
// precisions.
#define QOPS_TILE_VARIANTS(X) X(3, 2) X(3, 3) X(4, 0) X(4, 2) X(4, 3)

template <typename T, int R, int W>
hipError_t launch_tile_t(void* state, const PassHdr* hdr, const DevOp* ops, const void* coef, uint64_t ntiles,
                         int lds_bytes, int grid_cap, hipStream_t s);

template <typename T, int R, int W>
hipError_t launch_batch_reg_t(const BatchItem* items, int nitems, const BatchCirc* circs, const PassHdr* hdrs,
                              const DevOp* ops, const void* coef, int pass, int lds_bytes, int grid, hipStream_t s);

}  // namespace qops
