// 64x64 tiles of the implicit GEMM for products with few output tiles: at most a few workgroups per CU.
//
// Four waves of 32x32 outputs; operands by buffer loads (a convolution's activations: global_load_lds) into a ring of STAGES stages of 128 k, one barrier per stage, all
// fragments of a stage (4 + 4 reads) requested before its first matrix instruction.  A lone tile is bound by this chain
// (barrier, LDS round trip, four matrix instructions, the next requests), about 0.45 us per 128 k however deep the ring is.
// Against the same tile on igemm_dma.h (stages of 64 k): 3136 x 512 x 512 6.7 -> 6.2 us, 784 x 1024 x 512 5.8 -> 5.3,
// 6272 x 64 x 384 with 4-bit weights 5.6 -> 5.0.  (The waves dividing K instead of the tile, each on a ring of its own, and
// exchanging quadrants at the end: 784 x 1024 x 1024 7.6 -> 7.1, but 3136 x 512 x 512 6.6 and the 4-bit layer 5.6.)
//
// Any K that is whole chunks (K % 16 == 0, 4-bit weights K % 32 == 0): what lies beyond K reads as zero, outside the bounds
// of a buffer; the row sums of weight zero-points are corrected for the codes 0 there.  (A convolution's activations, by
// global_load_lds, come from a chunk of the code 128 there, which adds nothing to the row sums.  Its 4-bit
// weights with zero-points are copied by global_load_lds too, see PLAIN in igemm_dma.h: 4312 x 192 x 5760 35.6 us, like this 34.4.)
// The copies are buffer loads with 32-bit lane offsets (the dispatcher guarantees pitches below 2^25): see igemm_dma.h.  A_FAR: rows
// of a matrix further apart, by global_load_lds (with weight zero-points; other products of such rows never come here).
#pragma once

#include "igemm_dma.h"

namespace qnn {

template <bool B4, int STAGES> struct Tile64Geometry {
    static constexpr int kBk = 128;
    static constexpr int kBRow = B4 ? 64 : 128; // bytes of a weight row per stage
    static constexpr int kStageBytes = 64 * kBk + 64 * kBRow;
    static constexpr int kLds = STAGES * kStageBytes; // the output tile takes the ring's place
};

template <int A_MODE, bool B4, bool ZW, bool SPLIT, int STAGES>
__global__ void __launch_bounds__(256, 2) tile64_kernel(const IgemmArgs g, const int tiles_m, const int tiles_n, const int per_xcd, const int xcd_rows,
                                                        const SplitK sk)
{
    using G = Tile64Geometry<B4, STAGES>;
    constexpr int BK = G::kBk, A_LOADS = 2, B_LOADS = B4 ? 1 : 2, LOADS = A_LOADS + B_LOADS;
    constexpr int BCPR = G::kBRow / 16; // 16-byte chunks of a weight row per stage
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    int tile_row, tile_col, split;
    if (!assign_tile<SPLIT>(blockIdx.x >> 3, tiles_m, tiles_n, per_xcd, xcd_rows, sk.splits, tile_row, tile_col, split)) return;
    const int64_t m0 = (int64_t)tile_row * 64;
    const int n0 = tile_col * 64;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave_m = wave >> 1, wave_n = wave & 1, frow = lane & 31, fhalf = lane >> 5;

    // k range of this workgroup, in stages of 128
    const int k_begin = SPLIT ? split * sk.ksteps * 64 : 0;
    const int k_end = SPLIT ? (k_begin + sk.ksteps * 64 < g.K ? k_begin + sk.ksteps * 64 : g.K) : g.K;
    const int steps = (k_end - k_begin + BK - 1) / BK;

    // ---- chunks this lane copies: LDS chunk q = (row, position) holds chunk position ^ swizzle(row) of the row, so that
    // the fragment reads of 32 rows are free of bank conflicts
    auto swz_a = [](int row) { return (row >> 1) & 7; };
    auto swz_b = [](int row) { return B4 ? (row >> 2) & 3 : (row >> 1) & 7; };
    const uint8_t *a_src[A_LOADS];
    const uint8_t *const a_tile = g.A + m0 * g.lda, *const b_tile = g.B + ((int64_t)n0 * g.ldb >> (B4 ? 1 : 0));
    uint32_t a_off[A_LOADS], b_off[B_LOADS];
    int a_k[A_LOADS], b_k[B_LOADS], a_hi0[A_LOADS], a_wi0[A_LOADS];
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) {
        const int q = (wave * A_LOADS + i) * 64 + lane, row = q >> 3;
        a_k[i] = ((q & 7) ^ swz_a(row)) * 16;
        int64_t m = m0 + row;
        m = m < g.M ? m : g.M - 1;
        a_hi0[i] = a_wi0[i] = 0;
        a_off[i] = 0;
        if constexpr (A_MODE == A_FAR) {
            a_src[i] = g.A + m * g.lda + a_k[i] + k_begin;
        } else if constexpr (A_MODE == A_MATRIX) {
            a_off[i] = (uint32_t)((int)(m - m0) * (int)g.lda + a_k[i] + k_begin);
        } else {
            const int64_t img = m / ((int64_t)g.Ho * g.Wo);
            const int rem = (int)(m - img * ((int64_t)g.Ho * g.Wo));
            const int ho = rem / g.Wo, wo = rem - ho * g.Wo;
            a_hi0[i] = ho * g.sh - g.ph;
            a_wi0[i] = wo * g.sw - g.pw;
            // tap (0, 0) of this pixel (may lie outside the image: only dereferenced after the bounds check)
            a_src[i] = g.A + ((img * g.H + a_hi0[i]) * g.W + a_wi0[i]) * g.Cin;
        }
    }
#pragma unroll
    for (int i = 0; i < B_LOADS; ++i) {
        const int q = (wave * B_LOADS + i) * 64 + lane, row = q / BCPR;
        b_k[i] = ((q % BCPR) ^ swz_b(row)) * (B4 ? 32 : 16);
        int n = n0 + row;
        n = n < g.N ? n : g.N - 1;
        b_off[i] = (uint32_t)(((n - n0) * (int)g.ldb + b_k[i] + k_begin) >> (B4 ? 1 : 0));
    }
    const uint8_t *const zero_xs = &g_fill_table.v[128][0], *const outside = &g_fill_table.v[g.z_a][0];
    constexpr uint32_t NOWHERE = 0x80000000u;
    auto request = [&](int st) __attribute__((always_inline)) {
        uint8_t *const stage = smem + (st % STAGES) * G::kStageBytes;
        const int k0 = st * BK;
#pragma unroll
        for (int i = 0; i < A_LOADS; ++i) {
            const int k = k_begin + k0 + a_k[i];
            if constexpr (A_MODE == A_MATRIX) {
                buffer_to_lds16(a_tile + k0, 0x7fffffff, k < k_end ? a_off[i] : NOWHERE, stage + (wave * A_LOADS + i) * 1024);
                continue;
            }
            const uint8_t *src = zero_xs;
            if constexpr (A_MODE == A_FAR) {
                if (k < k_end) src = a_src[i] + k0;
            } else if (k < k_end) {
                const uint32_t tap = fast_div((uint32_t)k, (uint32_t)g.Cin, g.magic_cin);
                const uint32_t ta = fast_div(tap, (uint32_t)g.kw, g.magic_kw);
                const int a = (int)ta, b = (int)(tap - ta * (uint32_t)g.kw);
                const bool inside = (unsigned)(a_hi0[i] + a) < (unsigned)g.H && (unsigned)(a_wi0[i] + b) < (unsigned)g.W;
                src = inside ? a_src[i] + ((int64_t)a * g.W + b) * g.Cin + (k - (int)tap * g.Cin) : outside;
            }
            dma16(src, stage + (wave * A_LOADS + i) * 1024);
        }
#pragma unroll
        for (int i = 0; i < B_LOADS; ++i) {
            const uint8_t *const b_step = b_tile + (B4 ? k0 >> 1 : k0);
            uint8_t *const dst = stage + 64 * BK + (wave * B_LOADS + i) * 1024;
            const bool in = k_begin + k0 + b_k[i] < k_end;
            if constexpr (A_MODE == A_CONV && B4 && ZW) dma16(in ? b_step + b_off[i] : &g_fill_table.v[0][0], dst);
            else buffer_to_lds16(b_step, 0x7fffffff, in ? b_off[i] : NOWHERE, dst);
        }
    };
#pragma unroll
    for (int st = 0; st < STAGES - 1; ++st)
        if (st < steps) request(st);
    ChannelParams<1> cparams = {};
    if constexpr (!SPLIT) cparams = load_channel_params<64, 2, 1>(g, n0);

    int a_at[4], b_at[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const int ra = wave_m * 32 + frow, rb = wave_n * 32 + frow;
        a_at[ks] = ra * BK + (((2 * ks + fhalf) ^ swz_a(ra)) & 7) * 16;
        b_at[ks] = 64 * BK + rb * G::kBRow + (B4 ? ((ks ^ swz_b(rb)) & 3) * 16 + fhalf * 8 : (((2 * ks + fhalf) ^ swz_b(rb)) & 7) * 16);
    }
    i32x16 acc0, acc1; // two chains
#pragma unroll
    for (int r = 0; r < 16; ++r) acc0[r] = acc1[r] = 0;
    int32_t colsum[1] = {0}, rowsum[1] = {0};
    const bool need_colsum = g.z_a != 128;
    for (int st = 0; st < steps; ++st) {
        // this stage has landed when only those requested after it are left
        const int younger = steps - 1 - st < STAGES - 2 ? steps - 1 - st : STAGES - 2;
        static_assert(STAGES == 3 || STAGES == 4, "the cases below");
        if (STAGES == 4 && younger == 2) wait_vmcnt<2 * LOADS>();
        else if (younger == 1) wait_vmcnt<LOADS>();
        else wait_vmcnt<0>();
        lds_barrier(); // ... in all waves, and every wave has read the stage that the next request overwrites
        if (st + STAGES - 1 < steps) request(st + STAGES - 1);
        const uint8_t *const stage = smem + (st % STAGES) * G::kStageBytes;
        i32x4 fa[4], fb[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            fa[ks] = *reinterpret_cast<const i32x4 *>(stage + a_at[ks]);
            if constexpr (B4) fb[ks] = expand_int4(*reinterpret_cast<const u32x2 *>(stage + b_at[ks]));
            else fb[ks] = *reinterpret_cast<const i32x4 *>(stage + b_at[ks]);
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const i32x4 xs = fa[ks] ^ (int32_t)0x80808080; // uint8 code -> signed (code - 128)
            if (ks & 1) acc1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(xs, fb[ks], acc1, 0, 0, 0);
            else acc0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(xs, fb[ks], acc0, 0, 0, 0);
            if constexpr (ZW)
                if ((ks & 1) == wave_n) add_rowsum(rowsum[0], xs); // the two wave columns share the sub-steps
        }
        if (need_colsum) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int d = 0; d < 4; ++d) colsum[0] = __builtin_amdgcn_sdot4(fb[ks][d], 0x01010101, colsum[0], false);
        }
    }
    if constexpr (ZW && A_MODE == A_MATRIX) { // the codes 0 beyond K counted as -128
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            if ((ks & 1) == wave_n && k_begin + (steps - 1) * BK + (2 * ks + fhalf) * 16 >= k_end) rowsum[0] += 16 * 128;
    }
    i32x16 acc[1][1];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][0][r] = acc0[r] + acc1[r];
    if constexpr (SPLIT) { // partial sums, see igemm_dma.h
        int32_t *const plane = sk.partial + (int64_t)split * g.M * g.N;
        const int32_t corr = (128 - g.z_a) * (colsum[0] + __shfl_xor(colsum[0], 32));
        const int col = n0 + wave_n * 32 + frow;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t row = m0 + wave_m * 32 + 8 * (r >> 2) + 4 * fhalf + (r & 3);
            if (row < g.M && col < g.N) plane[row * g.N + col] = acc[0][0][r] + corr;
        }
    } else {
        lds_barrier(); // every wave has read its last fragments: the ring's memory is reused for the output
        igemm_epilogue_impl<64, 64, 2, 2, B4, ZW>(g, acc, colsum, cparams, smem, m0, n0, rowsum, g.K);
    }
}

} // namespace qnn
