// Weight-stationary short-K kernel with its rows in an LDS ring: forms for 8-bit weights, K <= 128.
#include "shortk_ring_launch.h"

namespace qnn {

bool launch_ring_int8_low(ShortKRingArgs &a, int ks, bool always, hipStream_t s) { return launch_ring_low<false>(a, ks, always, s); }

} // namespace qnn
