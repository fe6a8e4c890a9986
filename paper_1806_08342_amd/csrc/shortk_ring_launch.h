// Launch templates of shortk_ring.h, for the files that instantiate them.
#pragma once

#include "igemm_launch.h"
#include "ring_grid.h"
#include "shortk_ring.h"

namespace qnn {

template <int NB, int KS, bool INT4, int ADD, bool WIDE, bool ZW, bool STRIDED> inline void launch_ring_form(ShortKRingArgs &a, hipStream_t s)
{
    using G = RingGeometry<NB, KS, ADD, WIDE, ZW>;
    if constexpr (!G::kFits) {
        launch_ring_form<NB, KS, INT4, ADD, true, ZW, STRIDED>(a, s);
    } else {
        auto kernel = shortk_ring_kernel<NB, KS, INT4, ADD, WIDE, ZW, STRIDED>;
        static LdsOptIn opt_in; // per instantiation
        if (opt_in.ensure(reinterpret_cast<const void *>(kernel), G::kLds) != hipSuccess) return; // the error stays pending for the caller
        const int steps = (int)((a.s.g.M + 32 * G::kRw - 1) / (32 * G::kRw));
        a.s.col_groups = (a.s.g.N + 32 * NB - 1) / (32 * NB);
        const int sets = (a.s.col_groups + G::kCw - 1) / G::kCw;
        const int walkers = ring_walkers(G::kResident, sets, steps);
        a.s.walkers = walkers, a.steps = steps / walkers, a.more = steps % walkers;
        hipLaunchKernelGGL(kernel, dim3(8, (unsigned)sets, (unsigned)((walkers + 7) / 8)), dim3(G::kWaves * 64), G::kLds, s, a);
    }
}

template <int KS, bool INT4, int ADD, bool ZW, bool STRIDED> inline void launch_ring_width(ShortKRingArgs &a, hipStream_t s)
{
    constexpr int NB = KS > 4 || ADD == 3 ? 2 : 4;
    const int N = a.s.g.N;
    // few columns: one wave's, no wider than they are (not with the pair table, which is for large outputs)
    if constexpr (ADD < 2) {
        if (N <= 32) return launch_ring_form<1, KS, INT4, ADD, false, ZW, STRIDED>(a, s);
        if (NB == 4 && N <= 64) return launch_ring_form<2, KS, INT4, ADD, false, ZW, STRIDED>(a, s);
    }
    // four waves side by side on the same rows, unless more than an eighth of them had no columns (ADD == 3: eight, or four)
    constexpr int W = RingGeometry<NB, KS, ADD, true, ZW>::kCw;
    const int groups = (N + 32 * NB - 1) / (32 * NB), idle = (groups + W - 1) / W * W - groups;
    if (idle * 8 <= groups + idle) launch_ring_form<NB, KS, INT4, ADD, true, ZW, STRIDED>(a, s);
    else launch_ring_form<NB, KS, INT4, ADD, false, ZW, STRIDED>(a, s);
}

template <int KS, bool INT4> inline void launch_ring_ks(ShortKRingArgs &a, hipStream_t s)
{
    if (a.s.g.R) {
        // from 2^24 outputs on the 65536-entry pair table pays for itself; below, two 256-entry tables
        if (a.s.g.M * (int64_t)a.s.g.N >= ((int64_t)1 << 24)) {
            if constexpr (KS == 3 || KS == 4) // 16 waves where they have columns
                if (a.s.g.N >= 192) return launch_ring_width<KS, INT4, 3, false, false>(a, s);
            launch_ring_width<KS, INT4, 2, false, false>(a, s);
        } else launch_ring_width<KS, INT4, 1, false, false>(a, s);
    } else if (a.s.g.zw) {
        launch_ring_width<KS, INT4, 0, true, false>(a, s);
    } else if (a.s.strided) {
        launch_ring_width<KS, INT4, 0, false, true>(a, s);
    } else {
        launch_ring_width<KS, INT4, 0, false, false>(a, s);
    }
}

// the forms for ks sub-steps of 32 k (igemm_ring*.hip: 8- and 4-bit weights, up to 4 and more)
void launch_ring_int8_low(ShortKRingArgs &a, int ks, hipStream_t s);
void launch_ring_int8_high(ShortKRingArgs &a, int ks, hipStream_t s);
void launch_ring_int4_low(ShortKRingArgs &a, int ks, hipStream_t s);
void launch_ring_int4_high(ShortKRingArgs &a, int ks, hipStream_t s);

// Sub-steps beyond K cost like any other, so a form for nearly every number of them
template <bool INT4> inline void launch_ring_low(ShortKRingArgs &a, int ks, hipStream_t s)
{
    switch (ks) {
    case 1: return launch_ring_ks<1, INT4>(a, s);
    case 2: return launch_ring_ks<2, INT4>(a, s);
    case 3: return launch_ring_ks<3, INT4>(a, s);
    default: return launch_ring_ks<4, INT4>(a, s);
    }
}
template <bool INT4> inline void launch_ring_high(ShortKRingArgs &a, int ks, hipStream_t s)
{
    switch (ks) {
    case 5:
    case 6: return launch_ring_ks<6, INT4>(a, s);
    default: return launch_ring_ks<8, INT4>(a, s);
    }
}

} // namespace qnn
