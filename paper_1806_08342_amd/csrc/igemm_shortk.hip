// Launch routine of the short-K kernels (shortk_ring.h and shortk.h); forms of the latter for 8-bit weights.
#include "shortk_launch.h"
#include "shortk_ring_launch.h"
#include "tuning.h"

namespace qnn {

void launch_shortk_int8(const ShortKArgs &a, int ks, bool v16, int64_t waves, hipStream_t s) { launch_shortk_ks<false>(a, ks, v16, waves, s); }

bool shortk_eligible(const IgemmArgs &g, int b_mode, bool strided)
{
    if (g.K > 256 || (g.K % 8) != 0 || g.M <= 64 || g.M >= 0x7fffffe0 || b_mode == B_INT8_ROWS) return false;
    if (tuning().forced() || tuning().no_shortk) return false;
    const int64_t row_pitch = strided ? g.Cin : g.lda;
    if (!aligned_to(g.A, 8) || (row_pitch % 8) != 0) return false;
    if (!aligned_to(g.B, 4) || (g.ldb % 8) != 0) return false;
    return true;
}

// Rows of whole, aligned 16-byte pieces, weights of any alignment, offsets within 32 rows (weights: 128) of 31 bits.  A strided
// convolution (never with weight zero-points here) has its forms without the add.
static bool ring_eligible(const IgemmArgs &g, bool strided)
{
    if (tuning().shortk_alds == 0) return false; // tuning aid: fragments from global memory
    const int64_t row_pitch = strided ? g.Cin : g.lda;
    if (!aligned_to(g.A, 16) || (row_pitch % 16) != 0 || (g.K % 16) != 0 || g.M >= (1 << 30) || g.ldb >= (1 << 23)) return false;
    if (g.N > (1 << 21)) return false; // sets of column groups: a dimension of the grid
    if (!strided) return g.lda < (1 << 26);
    return (32 / ((int64_t)g.Ho * g.Wo) + 2) * g.H * g.W * g.Cin < (1ll << 31);
}

// The ring kernel where its rows are whole 16-byte pieces and it is ahead (ring_ahead and launch_ring_add, shortk_ring_launch.h), else
// shortk.h.  us with fragments from global memory and with the ring: 802816 x 128 x 256 80 and 66, 200704 x 128 x 128 17.1 and
// 12.2, 50176 x 256 x 128 11.7 and 8.2, 50176 x 256 x 256 14.2 and 11.1, with weight zero-points on 12544 x 256 x 256 10.3 and 6.6,
// 50176 x 1024 x 256 with the add 50.3 and 42.1, stride 2 on 256 x 56 x 56 x 256 -> 512 67 and 55; 4-bit weights, 100352 x 24 x 96
// 10.6 and 6.4.
qnn_status launch_shortk(IgemmArgs &g, int b_mode, bool strided, hipStream_t s)
{
    g.small_acc = 2; // K <= 256: |acc| <= 2^22
    g.c_vec16 = aligned_to(g.C, 16) && (g.ldc % 16 == 0);
    const int ks = (g.K + 31) / 32;
    ShortKArgs a = {};
    a.g = g;
    a.strided = strided ? 1 : 0;
    a.stream_out = g.M * (int64_t)g.N <= ((int64_t)32 << 20); // between 26 MB (gains) and 51 MB (the next layer loses more)
    bool ring = ring_eligible(g, strided);
    const bool whole = g.c_vec16 && g.ldc < (1 << 26);
    const bool v16 = aligned_to(g.A, 16) && ((strided ? g.Cin : g.lda) % 16) == 0 && (g.K % 16) == 0;
    // the add is built into the forms for pieces of 16, for outputs and residuals made of whole aligned chunks (the ring kernel's: not
    // strided, pitches within its 31-bit offsets)
    const bool add_pass = g.R != nullptr && !(v16 && g.c_vec16 && g.r_vec16 && (g.N % 16) == 0);
    if (add_pass) a.g.R = nullptr;
    if (a.g.R) ring = ring && !strided && whole && g.ldr < (1 << 26);
    if (ring) {
        ShortKRingArgs r = {};
        r.s = a;
        r.whole = whole ? 1 : 0;
        if (strided) r.magic_image = magic_for((uint32_t)(g.Ho * g.Wo)), r.magic_row = magic_for((uint32_t)g.Wo);
        const bool always = tuning().shortk_alds == 2;
        if (b_mode == B_INT4) ring = ks <= 4 ? launch_ring_int4_low(r, ks, always, s) : launch_ring_int4_high(r, ks, always, s);
        else ring = ks <= 4 ? launch_ring_int8_low(r, ks, always, s) : launch_ring_int8_high(r, ks, always, s);
    }
    if (!ring) {
        const int nb = ks <= 4 ? 4 : 2;
        a.col_groups = (g.N + 32 * nb - 1) / (32 * nb);
        const int64_t row_blocks = (g.M + 31) / 32;
        // as many waves as stay resident together (3 per SIMD for K <= 32 without weight zero-points and without the add, else 2, on
        // 256 CUs), spread over the column groups, then trimmed so that every wave walks the same number of row blocks
        const int64_t resident = 256 * 4 * ((ks <= 1 && !a.g.R && !g.zw) ? 3 : 2);
        int64_t walkers = resident / a.col_groups;
        walkers = walkers < 1 ? 1 : (walkers > row_blocks ? row_blocks : walkers);
        const int64_t per_walker = (row_blocks + walkers - 1) / walkers;
        walkers = (row_blocks + per_walker - 1) / per_walker;
        a.walkers = (int)walkers;
        const int64_t waves = walkers * a.col_groups;
        if (waves > 0x7fffffff) return QNN_EINVAL;
        if (b_mode == B_INT4) launch_shortk_int4(a, ks, v16, waves, s);
        else launch_shortk_int8(a, ks, v16, waves, s);
    }
    const qnn_status st = launch_status(hipGetLastError());
    if (st != QNN_OK || !add_pass) return st;
    return launch_add_inplace(g.C, g.ldc, g.R, g.ldr, g.M, g.N, g.add, s);
}

} // namespace qnn
