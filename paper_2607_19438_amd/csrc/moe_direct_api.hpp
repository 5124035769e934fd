// Host interface of moe_direct.hip: the grouped MoE GEMM for few rows per expert.
#pragma once

#include "qgemm_kernels.hpp"

namespace qg {

// Whether a launch of M rows over E experts is one for the direct kernel.
__attribute__((visibility("hidden"))) bool moe_direct_takes(int fmt, long M, int E);

// Launches it for the plain grouped GEMM or (swi) the fused gate/up + SiLU one; false, with nothing
// launched, if the grid would be too large. The caller checks for launch errors.
__attribute__((visibility("hidden"))) bool moe_direct_launch(int fmt, bool swi, TileArgs a, const void* const* wq,
                                                             const void* const* sc, int E, hipStream_t s);

}  // namespace qg
