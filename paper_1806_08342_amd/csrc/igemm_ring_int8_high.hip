// Weight-stationary short-K kernel with its rows in an LDS ring: forms for 8-bit weights, K > 128.
#include "shortk_ring_launch.h"

namespace qnn {

void launch_ring_int8_high(ShortKRingArgs &a, int ks, hipStream_t s) { launch_ring_high<false>(a, ks, s); }

} // namespace qnn
