// Launch templates of the weight-stationary short-K kernel, for the two files that instantiate them (8- and 4-bit weights).
#pragma once

#include "igemm_launch.h"
#include "shortk.h"

namespace qnn {

template <int KS, bool INT4> inline void launch_shortk_one(const ShortKArgs &a, bool v16, int64_t waves, hipStream_t s)
{
    constexpr int NB = KS <= 4 ? 4 : 2;
    const dim3 blocks((unsigned)((waves + 3) / 4));
    if (a.g.zw) {
        if (v16) hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, 16, true>), blocks, dim3(256), 0, s, a);
        else hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, 8, true>), blocks, dim3(256), 0, s, a);
    } else {
        if (v16) hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, 16>), blocks, dim3(256), 0, s, a);
        else hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, 8>), blocks, dim3(256), 0, s, a);
    }
}

// Sub-steps beyond K are loaded like any other, so a form for nearly every number of them
template <bool INT4> inline void launch_shortk_ks(const ShortKArgs &a, int ks, bool v16, int64_t waves, hipStream_t s)
{
    switch (ks) {
    case 1: return launch_shortk_one<1, INT4>(a, v16, waves, s);
    case 2: return launch_shortk_one<2, INT4>(a, v16, waves, s);
    case 3: return launch_shortk_one<3, INT4>(a, v16, waves, s);
    case 4: return launch_shortk_one<4, INT4>(a, v16, waves, s);
    case 5:
    case 6: return launch_shortk_one<6, INT4>(a, v16, waves, s);
    case 7: return launch_shortk_one<7, INT4>(a, v16, waves, s);
    default: return launch_shortk_one<8, INT4>(a, v16, waves, s);
    }
}

void launch_shortk_int8(const ShortKArgs &a, int ks, bool v16, int64_t waves, hipStream_t s);
void launch_shortk_int4(const ShortKArgs &a, int ks, bool v16, int64_t waves, hipStream_t s);

} // namespace qnn
