// Launch templates of shortk_ring.h, for the files that instantiate them.
#pragma once

#include "igemm_launch.h"
#include "ring_grid.h"
#include "shortk_ring.h"

namespace qnn {

// Whether a launch without the add is ahead of shortk.h, whose lanes load their fragments straight from global memory (us there and
// here; 8-bit weights unless said).
//  - up to 32 columns, or 64 with K <= 128: always (a form as wide as the columns; 25088 x 24 x 144 5.2 and 4.6), but for strided
//    launches of one step with K > 128 (28800 x 32 x 176 5.7 and 6.0).
//  - one step per walker: the launch is its set-up, and the weight exchange and its barriers lose (4-bit weights, 6272 x 576 x 96
//    5.1 and 5.9, 1568 x 960 x 160 4.3 and 4.9; 2000 x 1000 x 208 6.3 and 6.8, 2000 x 1000 x 64 6.1 and 6.4), unless the weight
//    rows are a multiple of 128 bytes apart, where fragment loads meet in the same channels (2000 x 1000 x 256 7.1 and 6.7,
//    55614 x 128 x 128 10.0 and 7.3), with weight zero-points 96 < K <= 128 altogether, or K <= 128 fills the chip (94226 x 128 x 32
//    8.1 and 7.0, 39421 x 71 x 64 7.6 and 7.5).
//  - K <= 96, walkers with one column group each: the row streams of the sets drift apart.  Behind where the last set is mostly
//    empty (115363 x 144 x 32 10.2 and 12.1, 239900 x 144 x 64 19.1 and 21.8), and for K > 32 beyond what the caches hold
//    (1000000 x 128 x 64 39.2 and 44.5, 651985 x 640 x 64 118 and 133) and with outputs that leave byte by byte (174968 x 158 x 64
//    31.5 and 36.6).
template <int NB, int KS, bool INT4, bool WIDE, bool ZW, bool STRIDED> inline bool ring_ahead(const IgemmArgs &g, int columns, int sets, int walkers, int per_walker)
{
    if (NB == 1 || (NB == 2 && KS <= 4)) return !(STRIDED && KS > 4 && per_walker == 1);
    const bool long_rows = (INT4 ? g.ldb / 2 : g.ldb) % 128 == 0;
    if (per_walker == 1 && (KS > 4 || sets * walkers <= (KS == 1 ? 400 : 300))) return long_rows || (ZW && KS == 4);
    if (STRIDED && KS > 4 && !WIDE) return long_rows; // 18819 x 640 x 240 12.6 and 14.8, 46400 x 176 x 176 11.2 and 13.2
    if (KS > 3 || WIDE) return true;
    if (sets > 1 && (int64_t)g.N * 4 < (int64_t)columns * sets * 3) return false;
    return KS == 1 || (g.N % 16 == 0 && g.M * (g.N + g.K) < 100000000);
}

// Launches one form, unless shortk.h is ahead of it (`always`: then too); whether it did.  With the add: see launch_ring_add.
template <int NB, int KS, bool INT4, int ADD, bool WIDE, bool ZW, bool STRIDED> inline bool launch_ring_form(ShortKRingArgs &a, bool always, hipStream_t s)
{
    using G = RingGeometry<NB, KS, ADD, WIDE, ZW>;
    const int steps = (int)((a.s.g.M + 32 * G::kRw - 1) / (32 * G::kRw));
    a.s.col_groups = (a.s.g.N + 32 * NB - 1) / (32 * NB);
    const int sets = (a.s.col_groups + G::kCw - 1) / G::kCw;
    const int walkers = ring_walkers(G::kResident, sets, steps), per_walker = (steps + walkers - 1) / walkers;
    const bool busy = per_walker > 1 && steps * 3ll >= 2ll * per_walker * ring_resident(G::kResident, sets);
    if (!always && !(ADD ? ADD > 1 || NB < 4 || busy : ring_ahead<NB, KS, INT4, WIDE, ZW, STRIDED>(a.s.g, 32 * NB * G::kCw, sets, walkers, per_walker))) return false;
    auto kernel = shortk_ring_kernel<NB, KS, INT4, ADD, WIDE, ZW, STRIDED>;
    static LdsOptIn opt_in; // per instantiation
    if (opt_in.ensure(reinterpret_cast<const void *>(kernel), G::kLds) != hipSuccess) return true; // the error stays pending for the caller
    a.s.walkers = walkers, a.steps = steps / walkers, a.more = steps % walkers;
    hipLaunchKernelGGL(kernel, dim3(8, (unsigned)sets, (unsigned)((walkers + 7) / 8)), dim3(G::kWaves * 64), G::kLds, s, a);
    return true;
}

// Column groups that W waves side by side leave without columns, of `total`
inline int ring_idle(int N, int columns, int W, int &total)
{
    const int groups = (N + columns - 1) / columns;
    total = (groups + W - 1) / W * W;
    return total - groups;
}

// Four waves side by side on the same rows, unless more than an eighth of them had no columns
template <int NB, int KS, bool INT4, int ADD, bool ZW, bool STRIDED> inline bool launch_ring_wide(ShortKRingArgs &a, bool always, hipStream_t s)
{
    int total;
    const int idle = ring_idle(a.s.g.N, 32 * NB, 4, total);
    if (idle * 8 <= total) return launch_ring_form<NB, KS, INT4, ADD, true, ZW, STRIDED>(a, always, s);
    return launch_ring_form<NB, KS, INT4, ADD, false, ZW, STRIDED>(a, always, s);
}

template <int KS, bool INT4, bool ZW, bool STRIDED> inline bool launch_ring_width(ShortKRingArgs &a, bool always, hipStream_t s)
{
    constexpr int NB = KS > 4 ? 2 : 4;
    const int N = a.s.g.N;
    // few columns: one wave's, no wider than they are
    if (N <= 32) return launch_ring_form<1, KS, INT4, 0, false, ZW, STRIDED>(a, always, s);
    if (NB == 4 && N <= 64) return launch_ring_form<2, KS, INT4, 0, false, ZW, STRIDED>(a, always, s);
    return launch_ring_wide<NB, KS, INT4, 0, ZW, STRIDED>(a, always, s);
}

// With the add the ring kernel has the forms that are ahead of shortk.h only (us there and here):
//  - two tables of 256 entries: up to 32 columns, or 64 with K <= 128 (22477 x 32 x 64 8.1 and 5.7 with 4-bit weights), and K <= 32 from
//    two steps on (160166 x 96 x 32 30.3 and 23.1, 16935 x 704 x 32 22.8 and 20.1) that keep two thirds of the chip busy (9046 x
//    816 x 16, 55 %, 13.5 and 19.5).  Other launches this small are set-up, and the
//    tables come on top of the weight exchange (6272 x 576 x 96 8.4 and 13.8, 2000 x 1008 x 208 6.8 and 8.5).
//  - the table of pairs, which leaves room for little besides: 96 < K <= 128 on 16 waves where less than a quarter of the columns
//    is idle (274776 x 480 x 128 82 and 69, 205520 x 1872 x 128 255 and 207; 384 columns are behind, 186836 x 384 x 128 43 and 50);
//    more than 160 with four waves side by side (50176 x 1024 x 256 53 and 43, 162833 x 1552 x 192 225 and 175), up to 192 for
//    large outputs only (25088 x 1024 x 192 25.2 and 26.0); 32 < K <= 64 with one or two full column groups and 2^25 outputs, by 1
//    to 3 % (401408 x 256 x 64 56.8 and 55.5; in the ResNet-50 stack at batch 256, 802816 x 256 x 64, 94.6 and 91.4).  Else behind:
//    400000 x 48 x 96 26 and 74, 200704 x 256 x 96 34 and 36, 300000 x 144 x 160 44 and 48.
template <int KS, bool INT4> inline bool launch_ring_add(ShortKRingArgs &a, bool always, hipStream_t s)
{
    const int N = a.s.g.N;
    [[maybe_unused]] int total;
    if (!shortk_pairs(a.s.g)) {
        if (N <= 32) return launch_ring_form<1, KS, INT4, 1, false, false, false>(a, always, s);
        if constexpr (KS <= 4)
            if (N <= 64) return launch_ring_form<2, KS, INT4, 1, false, false, false>(a, always, s);
        if constexpr (KS == 1) return launch_ring_wide<4, KS, INT4, 1, false, false>(a, always, s);
        return false;
    }
    if constexpr (KS == 4) {
        if (ring_idle(N, 64, 8, total) * 8 <= total) return launch_ring_form<2, KS, INT4, 3, true, false, false>(a, always, s);
        if (ring_idle(N, 64, 4, total) * 4 < total) return launch_ring_form<2, KS, INT4, 3, false, false, false>(a, always, s);
    }
    if constexpr (KS == 2)
        if ((N <= 128 || N == 256) && a.s.g.M * (int64_t)N >= ((int64_t)1 << 25)) return launch_ring_form<4, 2, INT4, 2, false, false, false>(a, always, s);
    if constexpr (KS > 4)
        if (ring_idle(N, 64, 4, total) * 8 <= total && (always || a.s.g.K > 192 || (a.s.g.K > 160 && a.s.g.M * (int64_t)N >= ((int64_t)1 << 26))))
            return launch_ring_form<2, KS, INT4, 2, true, false, false>(a, always, s);
    return false;
}

template <int KS, bool INT4> inline bool launch_ring_ks(ShortKRingArgs &a, bool always, hipStream_t s)
{
    if (a.s.g.R) return launch_ring_add<KS, INT4>(a, always, s);
    if (a.s.g.zw) return launch_ring_width<KS, INT4, true, false>(a, always, s);
    if (a.s.strided) return launch_ring_width<KS, INT4, false, true>(a, always, s);
    return launch_ring_width<KS, INT4, false, false>(a, always, s);
}

// the forms for ks sub-steps of 32 k (igemm_ring*.hip: 8- and 4-bit weights, up to 4 and more)
bool launch_ring_int8_low(ShortKRingArgs &a, int ks, bool always, hipStream_t s);
bool launch_ring_int8_high(ShortKRingArgs &a, int ks, bool always, hipStream_t s);
bool launch_ring_int4_low(ShortKRingArgs &a, int ks, bool always, hipStream_t s);
bool launch_ring_int4_high(ShortKRingArgs &a, int ks, bool always, hipStream_t s);

// Sub-steps beyond K cost like any other, so a form for nearly every number of them
template <bool INT4> inline bool launch_ring_low(ShortKRingArgs &a, int ks, bool always, hipStream_t s)
{
    switch (ks) {
    case 1: return launch_ring_ks<1, INT4>(a, always, s);
    case 2: return launch_ring_ks<2, INT4>(a, always, s);
    case 3: return launch_ring_ks<3, INT4>(a, always, s);
    default: return launch_ring_ks<4, INT4>(a, always, s);
    }
}
template <bool INT4> inline bool launch_ring_high(ShortKRingArgs &a, int ks, bool always, hipStream_t s)
{
    switch (ks) {
    case 5:
    case 6: return launch_ring_ks<6, INT4>(a, always, s);
    default: return launch_ring_ks<8, INT4>(a, always, s);
    }
}

} // namespace qnn
