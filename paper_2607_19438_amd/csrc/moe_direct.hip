// Launches of the direct MoE kernel (moe_direct.hpp). A source of its own, and so a code object of its
// own: it compiles beside the rest, and the staged kernels' code stays as compact as without it.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "moe_direct.hpp"
#include "moe_direct_api.hpp"

namespace qg {
namespace {

// RB 32-row blocks per group, KS K sub-steps per stage, WV waves per workgroup, WPE waves per SIMD
// the register allocation leaves room for (moe_direct.hpp)
template <int FMT, int RB, int KS, int WV, bool SWI, int WPE>
bool launch(TileArgs a, const void* const* wq, const void* const* sc, int E, hipStream_t s) {
  constexpr int BM = RB * 32;
  constexpr int BN = (SWI ? 16 : 32) * WV;   // output columns per workgroup
  const int nt = ((SWI ? a.swi_inter : a.N) + BN - 1) / BN;
  for (int e0 = 0; e0 < E; e0 += kMaxExpertsPerLaunch) {
    const int ne = (E - e0) < kMaxExpertsPerLaunch ? (E - e0) : kMaxExpertsPerLaunch;
    ExpertPtrs ep;
    for (int i = 0; i < kMaxExpertsPerLaunch; ++i) {
      ep.wq[i] = i < ne ? static_cast<const uint8_t*>(wq[e0 + i]) : nullptr;
      ep.sc[i] = i < ne ? static_cast<const uint16_t*>(sc[e0 + i]) : nullptr;
    }
    a.e_begin = e0;
    a.n_experts = ne;
    // upper bound of sum_e ceil(c_e / BM): every active expert (at most one per row) adds one group
    // and its further rows whole groups
    const long active = std::min<long>(ne, a.M);
    const long groups = (a.M - active) / BM + active;
    const long grid = groups * nt;
    if (grid > 0x7fffffffL) return false;
    hipLaunchKernelGGL((moe_direct_kernel<FMT, RB, KS, WV, SWI, WPE>), dim3((unsigned)grid),
                       dim3(WV * 64), 0, s, a, ep);
  }
  return true;
}

// Rows per group, from the mean rows per expert (the host does not see the routing); above the last
// limit the staged tiles take the call.
// Taller groups dequantise a large expert's weights fewer times, shorter ones leave more workgroups
// and registers for loads in flight; four waves per workgroup spread few items over more CUs.
// Measured on E=128 top-8 hidden 2048 inter 768 Q4 (gate/up + SiLU, down; us), against the staged
// tiles that took these calls before (64x128 / 128x128 up to 32 rows, 192x256 above):
//   T=4    32-row 19.6, 9.8     64-row 20.8, 10.4    staged 27.5, 17.0
//   T=128  32-row 66.9, 34.2    64-row 67.9, 35.4    128-row 77.5, 42.6   staged 96.0, 57.4
//   T=500  32-row 94.6, 54.7    64-row 86.3, 50.5    128-row 93.7, 59.4   staged 114, 75.4
//   T=1024 64-row 119, 73.5     128-row 114, 77.4    staged 124, 81.6
//   T=1536 64-row 149, 93.2     128-row 135, 96.4    staged 137, 95.1
// and E=64 top-6 hidden 2048 inter 1056 Q8 (its 64-row form spills; 32-row up to a mean of 32):
//   T=300 (mean 28)   32-row 83.8, 51.6   128-row 87.5, 48.5   staged 105, 57.2
//   T=777 (mean 73)   32-row 166, 88.6    128-row 106, 65.4    staged 160, 78.7
//   T=1200 (mean 112) 128-row 127, 90.6   staged 167, 86.1
constexpr long rows32(int fmt) { return fmt == kQ4 ? 16 : 32; }
constexpr long kRows64Q4 = 48;
constexpr long rows128(int fmt) { return fmt == kQ4 ? 80 : 96; }

template <int FMT, bool SWI>
bool pick(const TileArgs& a, const void* const* wq, const void* const* sc, int E, hipStream_t s) {
  const long mean_rows = (long)a.M / E;
  if (mean_rows <= rows32(FMT)) return launch<FMT, 1, 4, 4, SWI, 4>(a, wq, sc, E, s);
  if constexpr (FMT == kQ4) {
    if (mean_rows <= kRows64Q4) return launch<FMT, 2, 4, 8, SWI, 4>(a, wq, sc, E, s);
  }
  return launch<FMT, 4, 2, 4, SWI, 2>(a, wq, sc, E, s);
}

}  // namespace

bool moe_direct_takes(int fmt, long M, int E) { return M / E <= rows128(fmt); }

bool moe_direct_launch(int fmt, bool swi, TileArgs a, const void* const* wq, const void* const* sc, int E,
                       hipStream_t s) {
  if (fmt == kQ8) return swi ? pick<kQ8, true>(a, wq, sc, E, s) : pick<kQ8, false>(a, wq, sc, E, s);
  return swi ? pick<kQ4, true>(a, wq, sc, E, s) : pick<kQ4, false>(a, wq, sc, E, s);
}

}  // namespace qg
