// Launch templates of the weight-stationary short-K kernel, for the two files that instantiate them (8- and 4-bit weights).
#pragma once

#include "igemm_launch.h"
#include "shortk.h"

namespace qnn {

template <int NB, int KS, bool INT4, int ADD> inline void launch_shortk_add(const ShortKArgs &a, int64_t waves, hipStream_t s)
{
    // the waves of a workgroup (8 with the 64 KB table of code pairs, else 4) share the table(s); their tiles behind
    constexpr int kWaves = ADD == 2 ? 8 : 4;
    constexpr int kLds = (ADD == 2 ? 65536 : 2048) + kWaves * 32 * (32 * NB + 32);
    auto kernel = shortk_kernel<NB, KS, INT4, 16, ADD>;
    static LdsOptIn opt_in; // per instantiation
    if (opt_in.ensure(reinterpret_cast<const void *>(kernel), kLds) != hipSuccess) return; // the error stays pending for the caller
    hipLaunchKernelGGL(kernel, dim3((unsigned)((waves + kWaves - 1) / kWaves)), dim3(kWaves * 64), kLds, s, a);
}

template <int KS, bool INT4> inline void launch_shortk_one(const ShortKArgs &a, bool v16, int64_t waves, hipStream_t s)
{
    constexpr int NB = KS <= 4 ? 4 : 2;
    if (a.g.R) { // residual add in the store phase (the launcher only leaves R set for pieces of 16)
        if (shortk_pairs(a.g)) launch_shortk_add<NB, KS, INT4, 2>(a, waves, s);
        else launch_shortk_add<NB, KS, INT4, 1>(a, waves, s);
        return;
    }
    const dim3 blocks((unsigned)((waves + 3) / 4));
    if (a.g.zw) {
        if (v16) hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, 16, 0, true>), blocks, dim3(256), 0, s, a);
        else hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, 8, 0, true>), blocks, dim3(256), 0, s, a);
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
