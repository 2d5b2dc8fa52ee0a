// Launch of the list-free or list-driven pair kernels for every cluster size
// and set of outputs (included by the files that compile one part each).
#pragma once
#include "pair_kernels.h"

namespace gcme {
namespace {

template <typename T, int CI, bool ELEC, bool EV, bool ADJ, bool COUNT>
void launch_one(hipStream_t s, const PairLaunch& a) {
  dim3 g(a.ntiles), b(NL_WAVES * 64);
  if (a.direct)
    hipLaunchKernelGGL((k_pair_fused<T, CI, ELEC, EV, ADJ, COUNT>), g, b, 0, s, a);
  else
    hipLaunchKernelGGL((k_nl_force<T, CI, ELEC, EV, ADJ, COUNT>), g, b, 0, s, a);
}

template <typename T, int CI, bool ELEC>
void dispatch_mode(hipStream_t s, const PairLaunch& a, bool ev, bool adj, bool count) {
  if (count)
    launch_one<T, CI, ELEC, false, false, true>(s, a);
  else if (adj)
    launch_one<T, CI, ELEC, true, true, false>(s, a);
  else if (ev)
    launch_one<T, CI, ELEC, true, false, false>(s, a);
  else
    launch_one<T, CI, ELEC, false, false, false>(s, a);
}

}  // namespace

template <typename T, bool ELEC>
void dispatch_ci(hipStream_t s, const PairLaunch& a, bool ev, bool adj, bool count) {
  switch (a.ci) {
    case 2: dispatch_mode<T, 2, ELEC>(s, a, ev, adj, count); break;
    case 8: dispatch_mode<T, 8, ELEC>(s, a, ev, adj, count); break;
    default: dispatch_mode<T, 4, ELEC>(s, a, ev, adj, count); break;
  }
}

}  // namespace gcme
