// The weight-stationary short-K kernel of shortk.h for 4-bit weights.
#include "shortk_launch.h"

namespace qnn {

void launch_shortk_int4(const ShortKArgs &a, int ks, bool v16, int64_t waves, hipStream_t s) { launch_shortk_ks<true>(a, ks, v16, waves, s); }

} // namespace qnn
