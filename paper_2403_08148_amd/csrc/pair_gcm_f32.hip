// Excluded-volume pairs in single precision.
#include "pair_dispatch.h"

namespace gcme {
template void dispatch_ci<float, false>(hipStream_t s, const PairLaunch& a, bool ev, bool adj, bool count);
}  // namespace gcme
