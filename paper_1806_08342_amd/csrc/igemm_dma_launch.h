// Launch routine of the pipelined tile kernel (a template: the tile configurations are spread over several
// translation units).
#pragma once

#include "igemm_dma.h"
#include "igemm_launch.h"
#include "tuning.h"

namespace qnn {

// One rectangle of the tile grid per XCD: pick the cut (8x1, 4x2, 2x4, 1x8) with the least operand
// traffic from beyond the L2s (8/r copies of A's share + r copies of B's), among those that leave
// the XCDs within 10 % of an even load; else (xcd_rows stays 0) bands of the linear tile sequence.
inline void choose_xcd_cut(const IgemmArgs &g, int tiles_m, int tiles_n, int64_t work, int &per_xcd, int &xcd_rows)
{
    const int forced = tuning().xcd_rows;
    double best = 0.0;
    for (int r : {8, 4, 2, 1}) {
        const int c = 8 / r;
        if (forced >= 0 ? r != forced : false) continue;
        if (tiles_m < r || tiles_n < c) continue;
        const int64_t biggest = (int64_t)((tiles_m + r - 1) / r) * ((tiles_n + c - 1) / c);
        if (forced < 0 && biggest * 8 * 10 > work * 11) continue;
        const double traffic = (double)c * (double)g.M + (double)r * (double)g.N; // per unit of K
        if (xcd_rows == 0 || traffic < best) best = traffic, xcd_rows = r, per_xcd = (int)biggest;
    }
}

// second pass of split-K
inline hipError_t launch_splitk_reduce(const IgemmArgs &g, const SplitK &sk, hipStream_t s)
{
    const int64_t threads = g.M * (((int64_t)g.N + 3) / 4);
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, g, sk);
    return hipGetLastError();
}

// Whether taps outside the image may read as zero, by offsets within the images of a tile (A_CONV_ZERO, see igemm_dma.h)
inline bool zero_taps(const IgemmArgs &g, int bm)
{
    const int kh = g.K / (g.kw * g.Cin);
    return (g.z_a == 0 || (g.ph == 0 && g.pw == 0)) && g.Cin % 64 == 0 && kh * g.kw <= 32 &&
           (bm / ((int64_t)g.Ho * g.Wo) + 2) * g.H * g.W * g.Cin < (1ll << 31);
}

// `per_cu` > 0: persistent launch with that many workgroups per CU (each walks its XCD's tile
// sequence); 0: one workgroup per tile.  `prio`: issue-priority scheme of the main loop (see the kernel).
template <int BM, int BN, int WM, int WN, int A_MODE, int NSTAGE, bool SPLIT = false, bool ZW = false, bool B4 = false,
          int MINW = 1, bool KTAIL = false>
hipError_t launch_dma(const IgemmArgs &g, hipStream_t s, SplitK sk = SplitK{1, 0, nullptr}, int per_cu = 0, int prio = 0)
{
    if constexpr (A_MODE == A_CONV && !ZW && !KTAIL) // (Cin % 64 == 0: no tail)
        if (zero_taps(g, BM)) return launch_dma<BM, BN, WM, WN, A_CONV_ZERO, NSTAGE, SPLIT, ZW, B4, MINW, KTAIL>(g, s, sk, per_cu, prio);
    constexpr int kStages = NSTAGE * (BM + BN) * 64;
    constexpr int kOut = BM * (BN + 16) + 4 * WM * WN * (BN / WN / 32) * 64 + 2048 + (ZW ? 4 * BM * WN : 0); // + add tables + row sums
    constexpr int kLds = kStages > kOut ? kStages : kOut; // operand ring, reused for the output tile + column sums + add tables
    auto kernel = igemm_dma_kernel<BM, BN, WM, WN, A_MODE, NSTAGE, SPLIT, ZW, B4, MINW, KTAIL>;
    static LdsOptIn opt_in; // per instantiation
    if (hipError_t e = opt_in.ensure(reinterpret_cast<const void *>(kernel), kLds); e != hipSuccess) return e;
    const int tiles_m = (int)((g.M + BM - 1) / BM), tiles_n = (g.N + BN - 1) / BN;
    const int64_t work = (int64_t)tiles_m * tiles_n * sk.splits;
    int per_xcd = (int)((work + 7) / 8), xcd_rows = 0;
    if (!SPLIT) choose_xcd_cut(g, tiles_m, tiles_n, work, per_xcd, xcd_rows);
    const Tuning &tu = tuning();
    if (tu.persist == 0) per_cu = 0;
    else if (tu.persist > 0) per_cu = tu.persist;
    if (tu.gemm_prio >= 0) prio = tu.gemm_prio;
    int slots = per_xcd; // workgroups per XCD
    if (per_cu > 0 && slots > 32 * per_cu) slots = 32 * per_cu;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(slots * 8)), dim3(WM * WN * 64), kLds, s, g, tiles_m, tiles_n, per_xcd, xcd_rows,
                       sk, prio);
    hipError_t e = hipGetLastError();
    if (SPLIT && e == hipSuccess) {
        e = launch_splitk_reduce(g, sk, s);
    }
    return e;
}

} // namespace qnn
