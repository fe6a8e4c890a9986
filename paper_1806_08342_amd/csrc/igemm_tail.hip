// The pipelined tiles for K % 64 != 0 (whole 16-byte chunks: K % 16 == 0, 4-bit weights K % 32 == 0).
#include "igemm_dma_launch.h"

namespace qnn {

template <int A_MODE> static hipError_t launch_tail(const IgemmArgs &g, int bm, int bn, bool i4, const SplitK &sk, hipStream_t s)
{
    const SplitK one{1, 0, nullptr};
    if constexpr (A_MODE == A_CONV) // (with the tap arithmetic the 256-column tiles would spill)
        if (bn == 256) bn = 128, bm = i4 ? 128 : bm;
    if (i4) {
        if constexpr (A_MODE == A_MATRIX)
            if (bm == 256) return launch_dma<256, 256, 4, 2, A_MODE, 4, false, false, true, 1, true>(g, s);
        return launch_dma<128, 128, 2, 2, A_MODE, 4, false, false, true, 1, true>(g, s);
    }
    if (sk.splits > 1) return launch_dma<128, 128, 2, 2, A_MODE, 4, true, false, false, 1, true>(g, s, sk);
    if constexpr (A_MODE == A_MATRIX)
        if (bn == 256) {
            if (bm == 256) return launch_dma<256, 256, 4, 2, A_MODE, 4, false, false, false, 1, true>(g, s, one, 1, 1);
            return launch_dma<128, 256, 2, 2, A_MODE, 3, false, false, false, 2, true>(g, s, one, 2, 2);
        }
    if (bm == 256 && bn == 128) return launch_dma<256, 128, 4, 2, A_MODE, 4, false, false, false, 1, true>(g, s, one, 1, 0);
    if (bm == 256) return launch_dma<256, 64, 4, 1, A_MODE, 4, false, false, false, 1, true>(g, s);
    return launch_dma<128, 128, 2, 2, A_MODE, 4, false, false, false, 1, true>(g, s);
}

hipError_t launch_tail_tile(const IgemmArgs &g, int bm, int bn, bool mat, bool i4, const SplitK &sk, hipStream_t s)
{
    return mat ? launch_tail<A_MATRIX>(g, bm, bn, i4, sk, s) : launch_tail<A_CONV>(g, bm, bn, i4, sk, s);
}

} // namespace qnn
