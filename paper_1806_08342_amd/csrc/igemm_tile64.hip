// Launch routine of the 64x64 tiles (any K of whole chunks, weight zero-points, split-K).
#include "igemm_dma_launch.h"
#include "tile64.h"

namespace qnn {

template <int A_MODE, bool B4, bool ZW, bool SPLIT, int STAGES> static hipError_t launch_stages(const IgemmArgs &g, const SplitK &sk, hipStream_t s)
{
    using G = Tile64Geometry<B4, STAGES>;
    constexpr int kOut = 64 * (64 + 16) + 4 * 4 * 64 + 2048 + 4 * 64 * 2; // output tile, column-sum partials, add tables, row sums
    static_assert(G::kLds >= kOut, "the epilogue works in the operand ring");
    auto kernel = tile64_kernel<A_MODE, B4, ZW, SPLIT, STAGES>;
    static LdsOptIn opt_in; // per instantiation
    if (hipError_t e = opt_in.ensure(reinterpret_cast<const void *>(kernel), G::kLds); e != hipSuccess) return e;
    const int tiles_m = (int)((g.M + 63) / 64), tiles_n = (g.N + 63) / 64;
    const int64_t work = (int64_t)tiles_m * tiles_n * sk.splits;
    int per_xcd = (int)((work + 7) / 8), xcd_rows = 0;
    if (!SPLIT) choose_xcd_cut(g, tiles_m, tiles_n, work, per_xcd, xcd_rows);
    // what fits the chip in one round is not cut into rectangles of which the largest does not: 1403 x 1408 x 4096 with weight
    // zero-points (484 tiles, 66 in the largest of 8 rectangles) 26 us instead of 41
    constexpr int kRound = 32 * (STAGES == 4 ? 2 : 3); // workgroups that an XCD's CUs hold
    if (work <= 8 * kRound && per_xcd > kRound && tuning().xcd_rows < 0) xcd_rows = 0, per_xcd = (int)((work + 7) / 8);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(per_xcd * 8)), dim3(256), G::kLds, s, g, tiles_m, tiles_n, per_xcd, xcd_rows, sk);
    hipError_t e = hipGetLastError();
    if (SPLIT && e == hipSuccess) e = launch_splitk_reduce(g, sk, s);
    return e;
}

template <int A_MODE, bool B4, bool ZW, bool SPLIT> static hipError_t launch_one(const IgemmArgs &g, const SplitK &sk, hipStream_t s)
{
    // the ring as deep as the workgroups that are resident together allow: two of four stages, three of three
    const int64_t work = ((g.M + 63) / 64) * ((g.N + 63) / 64) * sk.splits;
    return work <= 512 ? launch_stages<A_MODE, B4, ZW, SPLIT, 4>(g, sk, s) : launch_stages<A_MODE, B4, ZW, SPLIT, 3>(g, sk, s);
}

template <int A_MODE> static hipError_t launch_mode(const IgemmArgs &g, bool i4, const SplitK &sk, hipStream_t s)
{
    if (sk.splits > 1) return launch_one<A_MODE, false, false, true>(g, sk, s);
    if (g.zw) return i4 ? launch_one<A_MODE, true, true, false>(g, sk, s) : launch_one<A_MODE, false, true, false>(g, sk, s);
    return i4 ? launch_one<A_MODE, true, false, false>(g, sk, s) : launch_one<A_MODE, false, false, false>(g, sk, s);
}

hipError_t launch_tile64(const IgemmArgs &g, bool mat, bool i4, const SplitK &sk, hipStream_t s)
{
    // rows of A whose offsets within 64 of them exceed 31 bits (1100 x 384 x 512 with weight zero-points, us: 5.3, rows 2^25 apart
    // 5.7; on the staged tile 6.4 and 6.5)
    if (mat && g.lda >= (1 << 25)) return i4 ? launch_one<A_FAR, true, true, false>(g, sk, s) : launch_one<A_FAR, false, true, false>(g, sk, s);
    return mat ? launch_mode<A_MATRIX>(g, i4, sk, s) : launch_mode<A_CONV>(g, i4, sk, s);
}

} // namespace qnn
