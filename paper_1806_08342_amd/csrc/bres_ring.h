// Weight-resident kernel of bres.h (256 < K, few output channels) for matrices, with the rows through an LDS ring.
//
// What bound it: the matrix-instruction fragments of the rows, fetched straight from global memory, put every lane on a row of
// its own, 15 bytes per cycle and CU.  Here a wave copies 64 k of its 32 rows (whole 64-byte pieces) by buffer loads into a ring
// of RING slots of its own, without a barrier; rows beyond M are outside the bounds of the buffer.  Fragments of the next
// slot, of rows and of weights, are read under the matrix instructions of this one.
// Requires K % 64 == 0 and 32 rows within 31 bits.  us before and now: 200704 x 128 x 512 41 and 38, 200704 x 256 x 512 57
// and 55.  (Convolutions stay with bres.h: 256 x 56 x 56 x 64, 3x3, took 77 us instead of 67 like this, with a test of the tap
// per request and the division of the rows once in nine.)
#pragma once

#include <type_traits>

#include "bres.h"
#include "buffer_ops.h"
#include "lds_ring.h"

namespace qnn {

template <int NB, int RING, bool INT4>
__global__ void __launch_bounds__(512, 2) bres_ring_kernel(const BResArgs s)
{
    constexpr int NW = 8;                     // waves per workgroup
    constexpr int PITCH = 32 * NB + 32;       // staged output row (see shortk.h)
    constexpr int SLOT = 2048;                // 32 rows x 64 k
    constexpr uint32_t NOWHERE = 0x80000000u; // beyond the bounds of every buffer
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const IgemmArgs &g = s.g;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int frow = lane & 31, fhalf = lane >> 5;
    const int KS = g.K / 32, pairs = KS / 2;
    uint8_t *const bfrag = smem;                                   // KS * NB fragments of 1 KB
    uint8_t *const stage = smem + KS * NB * 1024 + wave * 32 * PITCH;
    uint8_t *const ring = smem + KS * NB * 1024 + NW * 32 * PITCH + wave * (RING * SLOT);

    const int cg = blockIdx.x % s.col_groups, wg_walker = blockIdx.x / s.col_groups;
    const int n0 = cg * 32 * NB;
    const int blocks_here = (g.N - n0 + 31) / 32 < NB ? (g.N - n0 + 31) / 32 : NB;
    const int M = (int)g.M; // (the dispatcher guarantees M < 2^30)
    const int row_blocks = (M + 31) / 32;
    const int walkers = s.groups_walkers * NW;
    const int walker = wg_walker * NW + wave;

    // ---- the stream of requests: 64 k of a block of rows after the other, RING of them ahead.  A lane copies chunk
    // (lane & 3) ^ swizzle of rows lane / 4 and 16 + lane / 4.
    const uint8_t *r_base = g.A;
    int r_bytes = 0, r_block = walker, r_pair = 0;
    uint32_t r_off[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = i * 16 + (lane >> 2);
        r_off[i] = (uint32_t)(row * (int)g.lda + ((lane & 3) ^ lds_swizzle(row)) * 16);
    }
    auto start_block = [&] { // the rows of block r_block
        const int first = r_block * 32, rows = M - first < 32 ? M - first : 32;
        r_base = g.A + (int64_t)first * g.lda;
        r_bytes = rows > 0 ? (rows - 1) * (int)g.lda + g.K : 0;
    };
    auto request = [&](int slot) __attribute__((always_inline)) { // the next 64 k into a slot of the ring
        uint8_t *const dst = ring + slot * SLOT;
#pragma unroll
        for (int i = 0; i < 2; ++i) buffer_to_lds16(r_base, r_bytes, r_off[i] + (uint32_t)(r_pair * 64), dst + i * 1024);
        if (++r_pair == pairs) {
            r_pair = 0, r_block += walkers;
            start_block();
        }
    };
    start_block();
#pragma unroll
    for (int t = 0; t < RING; ++t) request(t);

    // ---- weights -> LDS, in fragment order (bres.h)
    bres_weights_to_lds<NB, INT4, NW>(g, n0, KS, wave, lane, bfrag);
    lds_barrier(); // the only workgroup barrier
    if (walker >= row_blocks) {
        wait_vmcnt<0>();
        return;
    }

    // ---- per-column epilogue constants
    BResColumns<NB> c;
    bres_columns<NB>(g, n0, KS, lane, bfrag, c);

    // ---- output tile: lane-invariant addresses; whole 16-byte chunks leave by buffer stores
    int st_lds[NB];
    uint32_t st_off[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int idx = i * 64 + lane, row = idx / (2 * NB), col0 = n0 + idx % (2 * NB) * 16;
        st_lds[i] = row * PITCH + idx % (2 * NB) * 16;
        st_off[i] = col0 < g.N ? (uint32_t)row * (uint32_t)g.ldc + (uint32_t)col0 : NOWHERE;
    }
    const int put_base = (4 * fhalf + (lane & 3)) * PITCH + (frow & ~3);
    const bool chunks_whole = g.c_vec16 && g.ldc < (1 << 26) && ((g.N & 15) == 0 || n0 + 32 * NB <= g.N);
    const int quad_lane = lane & 3;
    const uint32_t sel1 = (quad_lane & 1) ? 0x03070105u : 0x06020400u;
    const uint32_t sel2 = (quad_lane & 2) ? 0x03020706u : 0x05040100u;
    auto wave_sync = [] { // orders the wave's own LDS traffic for the compiler; the hardware keeps it in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto store_block = [&](int rbx) {
        wave_sync();
        uint8_t *const c_block = g.C + (int64_t)rbx * 32 * g.ldc;
        if (chunks_whole) {
            const int left = M - rbx * 32 < 32 ? M - rbx * 32 : 32;
#pragma unroll
            for (int i = 0; i < NB; ++i) buffer_store16<false>(c_block, left * (int)g.ldc, st_off[i], *reinterpret_cast<const u32x4 *>(stage + st_lds[i]));
        } else {
#pragma nounroll
            for (int i = 0; i < NB; ++i) {
                const int idx = i * 64 + lane;
                const int row = idx / (2 * NB), ch = idx % (2 * NB);
                const int n = n0 + ch * 16;
                if (rbx * 32 + row >= M || n >= g.N) continue;
                uint8_t *dst = c_block + (int64_t)row * g.ldc + n;
                const uint8_t *src = stage + row * PITCH + ch * 16;
#pragma nounroll
                for (int e = 0; e < 16 && n + e < g.N; ++e) dst[e] = src[e];
            }
        }
        wave_sync();
    };

    const int a_at[2] = {lds_chunk_offset(frow, fhalf), lds_chunk_offset(frow, 2 + fhalf)};
    auto walk = [&](auto mode_tag) {
        using Mode = RescaleModeTraits<decltype(mode_tag)::value>;
        i32x4 a0[2], a1[2], b0[2][NB], b1[2][NB]; // fragments of the slot at the matrix instructions and of the next one
        i32x16 acc[NB];
        auto read_rows = [&](int slot, i32x4 (&fa)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 2; ++u) fa[u] = *reinterpret_cast<const i32x4 *>(ring + slot * SLOT + a_at[u]);
        };
        auto read_weights = [&](int pair, i32x4 (&fb)[2][NB]) __attribute__((always_inline)) {
            const uint8_t *const p = bfrag + pair * (2 * NB * 1024) + lane * 16;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int j = 0; j < NB; ++j) fb[u][j] = *reinterpret_cast<const i32x4 *>(p + (u * NB + j) * 1024);
        };
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][r] = 0;
        int rb = walker, pair = 0, slot = 0, rb_stored = -1;
        wait_vmcnt<(RING - 1) * 2>(); // slot 0: RING - 1 requests of two copies behind it
        asm volatile("" ::: "memory");
        read_rows(0, a0);
        read_weights(0, b0);
        auto step = [&](i32x4 (&fa)[2], i32x4 (&fb)[2][NB], i32x4 (&na)[2], i32x4 (&nb)[2][NB]) __attribute__((always_inline)) {
            const int next_slot = slot + 1 < RING ? slot + 1 : 0, next_pair = pair + 1 < pairs ? pair + 1 : 0;
            i32x4 xs[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) xs[u] = fa[u] ^ (int32_t)0x80808080; // uint8 code -> signed (code - 128)
            // the next slot has landed when only the RING - 2 behind it are outstanding (a block's stores, if younger, make the wait
            // longer); this one's fragments are in registers (used above): it is refilled
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((RING - 2) * 2), "v"(xs[0]), "v"(xs[1]) : "memory");
            read_rows(next_slot, na);
            read_weights(next_pair, nb);
            asm volatile("" ::: "memory");
            request(slot);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xs[u], fb[u][j], acc[j], 0, 0, 0);
            if (pair == 0 && rb_stored >= 0) { // the block before this one
                store_block(rb_stored);
                rb_stored = -1;
            }
            if (pair == pairs - 1) { // the block is complete: epilogue into the wave's LDS tile
                auto put = [&](int j, int q, uint32_t x) {
                    uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true);
                    x = __builtin_amdgcn_perm(o, x, sel1);
                    o = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, true);
                    x = __builtin_amdgcn_perm(o, x, sel2);
                    *reinterpret_cast<uint32_t *>(stage + put_base + q * 8 * PITCH + j * 32) = x;
                };
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    if (j >= blocks_here) break;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int32_t a[4] = {acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
                        if constexpr (Mode::kFused) put(j, q, channel_codes4<Mode::kTies, Mode::kFull>(a, c.r[j]));
                        else put(j, q, other_codes4(a, c.mult[j], c.shift[j], c.corr[j], c.in_range, g.z_out, g.lo_rel, g.hi_rel));
                    }
                }
                wave_sync();
                rb_stored = rb;
                rb += walkers;
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[j][r] = 0;
            }
            pair = next_pair, slot = next_slot;
        };
        for (;;) {
            step(a0, b0, a1, b1);
            if (rb >= row_blocks) break;
            step(a1, b1, a0, b0);
            if (rb >= row_blocks) break;
        }
        store_block(rb_stored);
    };
    with_rescale_mode(c.fused, g.z_out, g.lo_rel, g.hi_rel, walk);
    wait_vmcnt<0>(); // no copy into this workgroup's LDS may outlive it
}

} // namespace qnn
