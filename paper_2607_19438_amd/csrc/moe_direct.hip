// Launches of the direct MoE kernel (moe_direct.hpp). A source of its own, and so a code object of its
// own: it compiles beside the rest, and the staged kernels' code stays as compact as without it.
#include <hip/hip_runtime.h>

#include "moe_direct.hpp"
#include "moe_direct_api.hpp"
#include "tile_rules.hpp"

namespace qg {
namespace {

static_assert(kMoeSlice == kMaxExpertsPerLaunch, "experts per launch");

// RB 32-row blocks per group, KS K sub-steps per stage, WV waves per workgroup, WPE waves per SIMD
// the register allocation leaves room for (moe_direct.hpp)
template <int FMT, int RB, int KS, int WV, bool SWI, int WPE>
void launch(TileArgs a, const void* const* wq, const void* const* sc, int E, hipStream_t s) {
  constexpr int BM = RB * 32;
  const long nt = moe_direct_tiles(BM, SWI, SWI ? a.swi_inter : a.N);
  for (int e0 = 0; e0 < E; e0 += kMaxExpertsPerLaunch) {
    const int ne = (E - e0) < kMaxExpertsPerLaunch ? (E - e0) : kMaxExpertsPerLaunch;
    ExpertPtrs ep;
    for (int i = 0; i < kMaxExpertsPerLaunch; ++i) {
      ep.wq[i] = i < ne ? static_cast<const uint8_t*>(wq[e0 + i]) : nullptr;
      ep.sc[i] = i < ne ? static_cast<const uint16_t*>(sc[e0 + i]) : nullptr;
    }
    a.e_begin = e0;
    a.n_experts = ne;
    const long grid = moe_direct_groups(BM, a.M, ne) * nt;   // moe_direct_rows has seen that it fits
    hipLaunchKernelGGL((moe_direct_kernel<FMT, RB, KS, WV, SWI, WPE>), dim3((unsigned)grid),
                       dim3(WV * 64), 0, s, a, ep);
  }
}

template <int FMT, bool SWI>
void pick(int rows, const TileArgs& a, const void* const* wq, const void* const* sc, int E, hipStream_t s) {
  if (rows == 32) return launch<FMT, 1, 4, 4, SWI, 4>(a, wq, sc, E, s);
  if constexpr (FMT == kQ4) {
    if (rows == 64) return launch<FMT, 2, 4, 8, SWI, 4>(a, wq, sc, E, s);
  }
  launch<FMT, 4, 2, 4, SWI, 2>(a, wq, sc, E, s);
}

}  // namespace

void moe_direct_launch(int rows, int fmt, bool swi, const TileArgs& a, const void* const* wq, const void* const* sc,
                       int E, hipStream_t s) {
  if (fmt == kQ8) return swi ? pick<kQ8, true>(rows, a, wq, sc, E, s) : pick<kQ8, false>(rows, a, wq, sc, E, s);
  return swi ? pick<kQ4, true>(rows, a, wq, sc, E, s) : pick<kQ4, false>(rows, a, wq, sc, E, s);
}

}  // namespace qg
