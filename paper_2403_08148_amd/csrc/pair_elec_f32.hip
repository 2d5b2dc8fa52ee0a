// Real-space electrostatics of the charged pairs in single precision.
#include "pair_dispatch.h"

namespace gcme {
template void dispatch_ci<float, true>(hipStream_t s, const PairLaunch& a, bool ev, bool adj, bool count);
}  // namespace gcme
