// Launch templates of the weight-stationary short-K kernel, for the two files that instantiate them (8- and 4-bit weights).
#pragma once

#include "igemm_launch.h"
#include "shortk.h"

namespace qnn {

template <int NB, int KS, bool INT4, int VEC, int BVEC, int ADD>
inline void launch_shortk_add(const ShortKArgs &a, int64_t waves, hipStream_t s)
{
    // the waves of a workgroup (8 with the 64 KB table of code pairs, else 4) share the table(s); their tiles behind
    constexpr int kWaves = ADD == 2 ? 8 : 4;
    constexpr int kLds = (ADD == 2 ? 65536 : 2048) + kWaves * 32 * (32 * NB + 32);
    auto kernel = shortk_kernel<NB, KS, INT4, VEC, BVEC, ADD>;
    static LdsOptIn opt_in; // per instantiation
    if (opt_in.ensure(reinterpret_cast<const void *>(kernel), kLds) != hipSuccess) return; // the error stays pending for the caller
    hipLaunchKernelGGL(kernel, dim3((unsigned)((waves + kWaves - 1) / kWaves)), dim3(kWaves * 64), kLds, s, a);
}

template <int KS, bool INT4, int VEC> inline void launch_shortk_one(const ShortKArgs &a, int64_t waves, hipStream_t s, bool alds)
{
    constexpr int NB = KS <= 4 ? 4 : 2;
    // weights: 16-byte loads when every 16-element piece of a column is 16-byte aligned, else dwords
    constexpr int W16 = INT4 ? 4 : 16;
    const bool b16 = !INT4 && aligned_to(a.g.B, 16) && (a.g.ldb % 16) == 0 && (a.g.K % 16) == 0;
    if constexpr (VEC == 16 && (KS == 4 || KS == 8)) {
        if (alds) { // A rows through LDS, shared by the waves of a workgroup (the caller sized `waves` in workgroups)
            if (b16) hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, VEC, W16, 0, true>), dim3((unsigned)waves), dim3(256), 0, s, a);
            else hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, VEC, 4, 0, true>), dim3((unsigned)waves), dim3(256), 0, s, a);
            return;
        }
    }
    if constexpr (VEC == 16) {
        if (a.g.R) { // residual add in the store phase (the launcher only leaves R set for VEC == 16)
            // from 2^24 outputs on the 65536-entry pair table pays for itself; below, two 256-entry tables
            const bool pairs = a.g.M * (int64_t)a.g.N >= ((int64_t)1 << 24);
            if (b16) pairs ? launch_shortk_add<NB, KS, INT4, VEC, W16, 2>(a, waves, s) : launch_shortk_add<NB, KS, INT4, VEC, W16, 1>(a, waves, s);
            else pairs ? launch_shortk_add<NB, KS, INT4, VEC, 4, 2>(a, waves, s) : launch_shortk_add<NB, KS, INT4, VEC, 4, 1>(a, waves, s);
            return;
        }
    }
    const unsigned blocks = (unsigned)((waves + 3) / 4);
    if (a.g.zw) {
        if (b16) hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, VEC, W16, 0, false, true>), dim3(blocks), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, VEC, 4, 0, false, true>), dim3(blocks), dim3(256), 0, s, a);
        return;
    }
    if (b16) hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, VEC, W16>), dim3(blocks), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((shortk_kernel<NB, KS, INT4, VEC, 4>), dim3(blocks), dim3(256), 0, s, a);
}

// Sub-steps beyond K are loaded like any other (clamped, see shortk_load16), so a form for nearly every number of them:
// 4800 x 464 x 160 6.0 us with 6, 6.6 with 8; 20000 x 144 x 224 6.7 with 7, 7.0 with 8; 20000 x 144 x 80 with the add 10.7
// with 3, 11.7 with 4.
template <bool INT4, int VEC> inline void launch_shortk_ks(const ShortKArgs &a, int ks, int64_t waves, hipStream_t s, bool alds)
{
    switch (ks) {
    case 1: return launch_shortk_one<1, INT4, VEC>(a, waves, s, false);
    case 2: return launch_shortk_one<2, INT4, VEC>(a, waves, s, false);
    case 3: return launch_shortk_one<3, INT4, VEC>(a, waves, s, false);
    case 4: return launch_shortk_one<4, INT4, VEC>(a, waves, s, alds);
    case 5:
    case 6: return launch_shortk_one<6, INT4, VEC>(a, waves, s, false);
    case 7: return launch_shortk_one<7, INT4, VEC>(a, waves, s, false);
    default: return launch_shortk_one<8, INT4, VEC>(a, waves, s, alds);
    }
}

void launch_shortk_int8(const ShortKArgs &a, int ks, int64_t waves, hipStream_t s, bool v16, bool alds);
void launch_shortk_int4(const ShortKArgs &a, int ks, int64_t waves, hipStream_t s, bool v16, bool alds);

} // namespace qnn
