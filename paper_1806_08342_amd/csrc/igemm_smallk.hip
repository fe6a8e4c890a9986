// Launch routine of the kernel for few rows and small launches.
#include "igemm_launch.h"
#include "smallk.h"
#include "tuning.h"

namespace qnn {

// Few rows (weights streamed once), or at most 800 workgroups of 32 rows x 16 columns: about three per CU,
// beyond which the tiles' higher rate wins (784 workgroups: 3136 x 128 x 128 in 4.1 us against 6.7, 4 x 28x28x128 3x3
// in 7.4 against 10.6; 1568: 1568 x 512 x 512 in 6.8 against 6.0).  Matrices with K >= 4096 and 8-bit weights are
// left to split-K over workgroups.
bool small_shape(int64_t M, int64_t N, int64_t K, bool conv, bool int4)
{
    if (M <= 64 && !conv) return true;
    if (!tuning().small || tuning().bres == 1) return false; // tuning aids: reach the other kernels on small shapes
    if (!conv && !int4 && K >= 4096) return false;
    const int64_t wgs = ((N + 15) / 16) * ((M + 31) / 32);
    // 4-bit weights: rows of 8 bytes take a branch around every load (5.3-9.4 us against 4.2-4.9 of the short-K kernel)
    if (int4 && K < 32) return false;
    // ... and a fourth workgroup does not fit a CU, so that past 768 the last few run alone: for some K the other kernels
    // are ahead then (784 workgroups, here / there: K = 32 5.4-5.7 / 4.4-4.9, 64 6.3 / 4.8-5.3, 128 6.3 / 5.3-6.1, 192 6.3 / 4.8,
    // 288 and 384 5.6 / 5.5, 448 6.5 / 6.0; but 256 5.9 / 6.2, 264 8.1 / 7.9, 512 6.2 / 6.0, 704 6.8 / 7.0, 2048 8.7 / 12.0).  The
    // line was drawn when the short-K kernel took 5.4-6.2 at K = 64 and the 64x64 tile 5.6 and more from 448 on.
    if (int4 && wgs > 768 && (K <= 48 || (K > 256 && K <= 384 && (K % 32) == 0))) return false;
    return wgs <= 800;
}

template <int AI, bool INT4, int A_MODE, SmallExtra EXTRA> static void launch_rows(const SmallArgs &a, int waves, hipStream_t s)
{
    const dim3 grid((unsigned)((a.g.N + 15) / 16), (unsigned)((a.g.M + 8 * AI - 1) / (8 * AI)));
    // (64 rows in 16 waves do not fit the register file)
    if (waves == 4) hipLaunchKernelGGL((smallk_kernel<AI, INT4, 4, A_MODE, EXTRA>), grid, dim3(256), 0, s, a);
    else if (waves == 8 || AI == 8) hipLaunchKernelGGL((smallk_kernel<AI, INT4, 8, A_MODE, EXTRA>), grid, dim3(512), 0, s, a);
    else hipLaunchKernelGGL((smallk_kernel<AI, INT4, AI == 8 ? 8 : 16, A_MODE, EXTRA>), grid, dim3(1024), 0, s, a);
}

template <bool INT4, SmallExtra EXTRA> static void launch_small(const SmallArgs &a, bool conv, hipStream_t s)
{
    const IgemmArgs &g = a.g;
    const int64_t cols = (g.N + 15) / 16, wgs32 = cols * ((g.M + 31) / 32);
    const int steps = (g.K + (INT4 ? 255 : 127)) / (INT4 ? 256 : 128);
    // rows per workgroup: 64 where that still gives every CU a workgroup and halves the weight traffic, else 32 or fewer
    const int ai = g.M <= 8 ? 1 : (g.M <= 16 ? 2 : (g.M > 32 && g.M <= 64 && wgs32 > 256 ? 8 : 4));
    const int64_t wgs = ai == 4 ? wgs32 : cols;
    // waves: K is divided as far as one workgroup per CU goes; several workgroups per CU overlap each other instead
    // (784 workgroups on 8 x 14x14x256, 3x3: 8.9 us with 4 waves, 10.4 with 8; 64 x 8192 x 8192 28.5 against 31.7)
    const bool several = wgs > (ai == 8 ? 256 : 512) && ai >= 4;
    const int waves = several || steps <= 4 ? 4 : (ai < 8 && wgs <= 256 && steps > 8 ? 16 : 8);
    if (conv) {
        launch_rows<4, INT4, A_CONV, EXTRA>(a, waves, s);
    } else if (ai == 1) {
        launch_rows<1, INT4, A_MATRIX, EXTRA>(a, waves, s);
    } else if (ai == 2) {
        launch_rows<2, INT4, A_MATRIX, EXTRA>(a, waves, s);
    } else if (ai == 4) {
        launch_rows<4, INT4, A_MATRIX, EXTRA>(a, waves, s);
    } else {
        launch_rows<8, INT4, A_MATRIX, EXTRA>(a, waves, s);
    }
}

bool try_small(const IgemmArgs &g, int a_mode, int b_mode, hipStream_t s, qnn_status *status)
{
    const bool conv = a_mode == A_CONV;
    if (b_mode == B_INT8_ROWS || tuning().forced() || !small_shape(g.M, g.N, g.K, conv, b_mode == B_INT4)) return false;
    if (conv && (g.Cin % 16) != 0) return false;
    SmallArgs a = {};
    a.g = g;
    if (conv) {
        fast_division((uint32_t)(g.Ho * g.Wo), a.magic_hw, a.shift_hw);
        fast_division((uint32_t)g.Wo, a.magic_wo, a.shift_wo);
    }
    const bool i4 = b_mode == B_INT4;
    if (g.zw) i4 ? launch_small<true, SMALL_ZW>(a, conv, s) : launch_small<false, SMALL_ZW>(a, conv, s);
    else if (g.R) i4 ? launch_small<true, SMALL_ADD>(a, conv, s) : launch_small<false, SMALL_ADD>(a, conv, s);
    else i4 ? launch_small<true, SMALL_PLAIN>(a, conv, s) : launch_small<false, SMALL_PLAIN>(a, conv, s);
    *status = launch_status(hipGetLastError());
    return true;
}

} // namespace qnn
