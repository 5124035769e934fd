// Host interface of moe_direct.hip: the grouped MoE GEMM for few rows per expert.
#pragma once

#include "qgemm_kernels.hpp"

namespace qg {

// Launches the direct kernel with groups of `rows` rows, what moe_direct_rows gives for the call, for the
// plain grouped GEMM or (swi) the fused gate/up + SiLU one. The caller checks for launch errors.
__attribute__((visibility("hidden"))) void moe_direct_launch(int rows, int fmt, bool swi, const TileArgs& a,
                                                             const void* const* wq, const void* const* sc, int E,
                                                             hipStream_t s);

}  // namespace qg
