// Weight-stationary short-K kernel with its rows in an LDS ring: forms for 4-bit weights, K > 128.
#include "shortk_ring_launch.h"

namespace qnn {

bool launch_ring_int4_high(ShortKRingArgs &a, int ks, bool always, hipStream_t s) { return launch_ring_high<true>(a, ks, always, s); }

} // namespace qnn
