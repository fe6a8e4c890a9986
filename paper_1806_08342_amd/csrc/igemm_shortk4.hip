// The weight-stationary short-K kernel for 4-bit weights.
#include "shortk_launch.h"

namespace qnn {

void launch_shortk_int4(const ShortKArgs &a, int ks, int64_t waves, hipStream_t s, bool v16, bool alds)
{
    if (v16) launch_shortk_ks<true, 16>(a, ks, waves, s, alds);
    else launch_shortk_ks<true, 8>(a, ks, waves, s, false);
}

} // namespace qnn
