// Launch routine of the weight-stationary short-K kernel; its forms for 8-bit weights.
#include "shortk_launch.h"
#include "tuning.h"

namespace qnn {

void launch_shortk_int8(const ShortKArgs &a, int ks, int64_t waves, hipStream_t s, bool v16, bool alds)
{
    if (v16) launch_shortk_ks<false, 16>(a, ks, waves, s, alds);
    else launch_shortk_ks<false, 8>(a, ks, waves, s, false);
}

bool shortk_eligible(const IgemmArgs &g, int b_mode, bool strided)
{
    if (g.K > 256 || (g.K % 8) != 0 || g.M <= 64 || g.M >= 0x7fffffe0 || b_mode == B_INT8_ROWS) return false;
    if (tuning().forced() || tuning().no_shortk) return false;
    const int64_t row_pitch = strided ? g.Cin : g.lda;
    if (!aligned_to(g.A, 8) || (row_pitch % 8) != 0) return false;
    if (!aligned_to(g.B, 4) || (g.ldb % 8) != 0) return false;
    return true;
}

qnn_status launch_shortk(IgemmArgs &g, int b_mode, bool strided, hipStream_t s)
{
    g.small_acc = 2; // K <= 256: |acc| <= 2^22
    g.c_vec16 = aligned_to(g.C, 16) && (g.ldc % 16 == 0);
    const int ks = (g.K + 31) / 32;
    const int nb = ks <= 4 ? 4 : 2;
    ShortKArgs a = {};
    a.g = g;
    a.strided = strided ? 1 : 0;
    a.stream_out = g.M * (int64_t)g.N <= ((int64_t)32 << 20); // between 26 MB (gains) and 51 MB (the next layer loses more)
    a.col_groups = (g.N + 32 * nb - 1) / (32 * nb);
    const int64_t row_blocks = (g.M + 31) / 32;
    // as many waves as stay resident together (3 per SIMD for K <= 32 without weight zero-points, else 2, on 256 CUs), spread
    // over the column groups, then trimmed so that every wave walks the same number of row blocks
    const int64_t row_pitch0 = strided ? g.Cin : g.lda;
    const bool add_fused = g.R != nullptr && aligned_to(g.A, 16) && (row_pitch0 % 16) == 0 && (g.K % 16) == 0 && g.c_vec16 &&
                           g.r_vec16 && (g.N % 16) == 0; // the variant with the add built in: 8-wave workgroups, one per CU
    const int64_t resident = 256 * 4 * ((ks <= 1 && !add_fused && !g.zw) ? 3 : 2);
    int64_t walkers = resident / a.col_groups;
    walkers = walkers < 1 ? 1 : (walkers > row_blocks ? row_blocks : walkers);
    const int64_t per_walker = (row_blocks + walkers - 1) / walkers;
    walkers = (row_blocks + per_walker - 1) / per_walker;
    a.walkers = (int)walkers;
    int64_t waves = walkers * a.col_groups;
    if (waves > 0x7fffffff) return QNN_EINVAL;
    const int64_t row_pitch = strided ? g.Cin : g.lda;
    const bool v16 = aligned_to(g.A, 16) && (row_pitch % 16) == 0 && (g.K % 16) == 0;
    // the add is built into the 16-byte variants only, for outputs and residuals made of whole aligned chunks
    const bool add_pass = g.R != nullptr && !add_fused;
    if (add_pass) a.g.R = nullptr;
    // K = 128 / 256 with enough column groups to fill a workgroup: the A rows go through LDS once per workgroup.
    // Not with the add built in: its 8-wave workgroups (one per CU, sharing the table of code pairs) lose more at
    // the barrier of every row block than the shared rows save (measured 65 against 58 us on 50176 x 1024 x 256).
    const int wg_waves = 4;
    const bool alds = tuning().shortk_alds != 0 && !strided && v16 && !a.g.R && !g.zw && (g.K == 128 || g.K == 256) && a.col_groups >= wg_waves;
    if (alds) {
        const int64_t groups = (a.col_groups + wg_waves - 1) / wg_waves;
        const int64_t resident_wgs = 256 * 2;
        int64_t wk = resident_wgs / groups;
        wk = wk < 1 ? 1 : (wk > row_blocks ? row_blocks : wk);
        const int64_t per = (row_blocks + wk - 1) / wk;
        wk = (row_blocks + per - 1) / per;
        a.walkers = (int)wk;
        waves = groups * wk; // workgroups
    }
    if (b_mode == B_INT4) launch_shortk_int4(a, ks, waves, s, v16, alds);
    else launch_shortk_int8(a, ks, waves, s, v16, alds);
    const qnn_status st = launch_status(hipGetLastError());
    if (st != QNN_OK || !add_pass) return st;
    return launch_add_inplace(g.C, g.ldc, g.R, g.ldr, g.M, g.N, g.add, s);
}

} // namespace qnn
