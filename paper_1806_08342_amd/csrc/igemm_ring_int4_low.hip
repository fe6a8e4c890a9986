// Weight-stationary short-K kernel with its rows in an LDS ring: forms for 4-bit weights, K <= 128.
#include "shortk_ring_launch.h"

namespace qnn {

void launch_ring_int4_low(ShortKRingArgs &a, int ks, hipStream_t s) { launch_ring_low<true>(a, ks, s); }

} // namespace qnn
