// Quantized GEMM with very few rows (M <= 64: a fully connected layer at small batch).
//
// The product is bound by streaming the weights once (K*N bytes, half of that for 4-bit weights), so the
// kernel is organised around memory-level parallelism, not MFMA rate: one workgroup owns 16 output
// columns, its 8 or 16 waves split K between them, and every lane fetches its own MFMA fragments
// straight from global memory with 16-byte loads, a whole batch of K-steps in flight, no LDS staging.
// The roles of the operands are swapped with respect to the big kernel: the weights are the A operand of
// v_mfma_i32_16x16x64_i8 (16 columns n x 64 k) and the activations the B operand (16 rows m), so a lane
// ends up with 4 consecutive output columns of one row m: one dword store, no transposition.
//
// A K-step is 128 deep, two matrix instructions.  8-bit weights: instruction h takes k = 64 h + 16 q +
// (0..15) in quarter q of the lanes, so that a wave reads the two halves of every 128-byte line back to
// back.  4-bit weights: one 16-byte load holds 32 consecutive weights, instruction h takes k = 32 q +
// 16 h + (0..15) -- on both operands alike; a sum does not care about the order of its terms -- so that
// as many weight bytes are in flight as with 8-bit weights; they are unpacked in registers (kept times
// 16 in int8, accumulators shifted back exactly).
//
// Any K, any pitch, any alignment: gfx950 loads 16 bytes from any byte address, and the piece that
// sticks out of a row's end is read from K - 16 instead and shifted (load_tail16).  Only the last,
// partial K-step pays for that.  The per-column parameters are requested before the main loop: behind
// the reduction their latency was a fifth of the kernel (M = 1, 4096 x 4096).
#pragma once

#include "igemm.h"

namespace qnn {

// 16 bytes from any byte address
__device__ __forceinline__ u32x4 load16_any(const uint8_t *p)
{
    u32x4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

// bytes k .. k + 15 of a row of `len` bytes, zero from `len` on; reads inside the row only
__device__ __forceinline__ u32x4 load_tail16(const uint8_t *row, int k, int len)
{
    if (k + 16 <= len) return load16_any(row + k);
    if (k >= len) return u32x4{0, 0, 0, 0};
    if (len < 16) { // k == 0: the row is shorter than one load
        u32x4 v = {0, 0, 0, 0};
        for (int i = 0; i < len; ++i) v[i >> 2] |= (uint32_t)row[i] << (8 * (i & 3));
        return v;
    }
    const u32x4 v = load16_any(row + len - 16);
    const uint32_t s = (uint32_t)(k - (len - 16)); // 1 .. 15 bytes to drop
    uint64_t lo = (uint64_t)v.x | ((uint64_t)v.y << 32), hi = (uint64_t)v.z | ((uint64_t)v.w << 32);
    if (s >= 8) {
        lo = hi >> (8 * (s - 8));
        hi = 0;
    } else {
        lo = (lo >> (8 * s)) | (hi << (64 - 8 * s));
        hi >>= 8 * s;
    }
    return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

// 16 weights from 8 packed bytes (element 2j in the low nibble of byte j), each times 16
__device__ __forceinline__ i32x4 widen_int4(uint32_t r0, uint32_t r1)
{
    const uint32_t r[2] = {r0, r1};
    i32x4 w;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const uint32_t even = (r[d] << 4) & 0xF0F0F0F0u, odd = r[d] & 0xF0F0F0F0u;
        w[2 * d] = (int32_t)__builtin_amdgcn_perm(odd, even, 0x05010400u);
        w[2 * d + 1] = (int32_t)__builtin_amdgcn_perm(odd, even, 0x07030602u);
    }
    return w;
}

template <int MT, bool INT4, int NW>
__global__ void __launch_bounds__(NW * 64) skinny_gemm_kernel(const IgemmArgs g)
{
    constexpr int BN = 16, STEP = 128, NB = INT4 ? 1 : 2; // weight loads per step and lane
    constexpr int UNROLL = MT == 1 ? 4 : 2;               // steps in flight per wave
    constexpr int PW = NW < 8 ? NW : 8;                   // waves whose partial sums fit LDS at a time
    __shared__ i32x4 part[PW][MT][64];
    __shared__ int32_t csum[NW][BN];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6); // wave-uniform
    const int n0 = blockIdx.x * BN;
    const int frow = lane & 15, quarter = lane >> 4;

    // weight row (output column) and activation rows of this lane's fragments, clamped
    int nw = n0 + frow;
    nw = nw < g.N ? nw : g.N - 1;
    const uint8_t *const brow = INT4 ? g.B + (((int64_t)nw * g.ldb) >> 1) : g.B + (int64_t)nw * g.ldb;
    const uint8_t *arow[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        int64_t m = t * 16 + frow;
        m = m < g.M ? m : g.M - 1;
        arow[t] = g.A + m * g.lda;
    }
    // byte offsets inside a step: weights, and the activations of the two matrix instructions
    const int boff = 16 * quarter;
    const int aoff[2] = {INT4 ? 32 * quarter : 16 * quarter, INT4 ? 32 * quarter + 16 : 64 + 16 * quarter};

    // per-column parameters of the output this thread writes: row m = 16 t + (lane & 15), 4 columns from nb
    const int nb = n0 + 4 * quarter;
    int32_t p_bias[4], p_mult[4], p_shift[4];
    const int32_t *const bias_or_any = g.bias ? g.bias : g.mult; // no branch around the load; the value is dropped below
    if (wave < MT && (g.N & 3) == 0) { // whole groups of four: one load each
        const int n = nb < g.N ? nb : g.N - 4;
        __builtin_memcpy(p_bias, bias_or_any + n, 16);
        __builtin_memcpy(p_mult, g.mult + n, 16);
        __builtin_memcpy(p_shift, g.shift + n, 16);
    } else if (wave < MT) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int n = nb + e < g.N ? nb + e : g.N - 1;
            p_bias[e] = bias_or_any[n];
            p_mult[e] = g.mult[n];
            p_shift[e] = g.shift[n];
        }
    }

    i32x4 acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = i32x4{0, 0, 0, 0};
    int32_t colsum = 0;
    const bool need_colsum = g.z_a != 128;
    // one step: wv the weight loads, av the activation loads of both matrix instructions
    auto multiply = [&](const u32x4 (&wv)[NB], const u32x4 (&av)[2][MT]) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            i32x4 fb;
            if constexpr (INT4) fb = widen_int4(wv[0][2 * h], wv[0][2 * h + 1]);
            else fb = i32x4{(int32_t)wv[h].x, (int32_t)wv[h].y, (int32_t)wv[h].z, (int32_t)wv[h].w};
            if (need_colsum) {
#pragma unroll
                for (int d = 0; d < 4; ++d) colsum = __builtin_amdgcn_sdot4(fb[d], 0x01010101, colsum, false);
            }
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const u32x4 x = av[h][t] ^ 0x80808080u; // uint8 code -> signed (code - 128)
                const i32x4 xs = {(int32_t)x.x, (int32_t)x.y, (int32_t)x.z, (int32_t)x.w};
                acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb, xs, acc[t], 0, 0, 0);
            }
        }
    };

    const int steps = g.K / STEP;
    // `count` steps of this wave, all their loads ahead of the first wait
    auto batch = [&](int s0, auto count) __attribute__((always_inline)) {
        constexpr int U = decltype(count)::value;
        u32x4 wv[U][NB], av[U][2][MT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (s0 + u * NW) * STEP;
#pragma unroll
            for (int i = 0; i < NB; ++i) wv[u][i] = load16_any(brow + (INT4 ? k >> 1 : k) + boff + 64 * i);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int t = 0; t < MT; ++t) av[u][h][t] = load16_any(arow[t] + k + aoff[h]);
        }
        asm volatile("" ::: "memory"); // the loads stay where they are
#pragma unroll
        for (int u = 0; u < U; ++u) multiply(wv[u], av[u]);
    };
    int s0 = wave;
    for (; s0 + (UNROLL - 1) * NW < steps; s0 += UNROLL * NW) batch(s0, std::integral_constant<int, UNROLL>{});
    if (UNROLL > 3 && s0 + 2 * NW < steps) batch(s0, std::integral_constant<int, 3>{});
    else if (UNROLL > 2 && s0 + NW < steps) batch(s0, std::integral_constant<int, 2>{});
    else if (s0 < steps) batch(s0, std::integral_constant<int, 1>{});
    if (steps * STEP < g.K && wave == steps % NW) { // the partial step: weights beyond K read as zero
        const int k = steps * STEP;
        u32x4 wv[NB], av[2][MT];
#pragma unroll
        for (int i = 0; i < NB; ++i) wv[i] = INT4 ? load_tail16(brow, (k >> 1) + boff, g.K >> 1) : load_tail16(brow, k + boff + 64 * i, g.K);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < MT; ++t) av[h][t] = load_tail16(arow[t], k + aoff[h], g.K);
        multiply(wv, av);
    }

    // ---- combine the waves (16 waves: the second half hands its sums to the first one)
    colsum += __shfl_xor(colsum, 16);
    colsum += __shfl_xor(colsum, 32);
    if (lane < BN) csum[wave][lane] = colsum;
    if constexpr (NW > PW) {
        if (wave >= PW) {
#pragma unroll
            for (int t = 0; t < MT; ++t) part[wave - PW][t][lane] = acc[t];
        }
        __syncthreads();
        if (wave < PW) {
#pragma unroll
            for (int t = 0; t < MT; ++t) acc[t] += part[wave][t][lane];
        }
    }
    if (wave < PW) { // every wave overwrites only what it has read itself
#pragma unroll
        for (int t = 0; t < MT; ++t) part[wave][t][lane] = acc[t];
    }
    __syncthreads();

    // ---- epilogue: wave t finishes m tile t
    if (wave >= MT) return;
    const int64_t m = wave * 16 + frow;
    if (m >= g.M || nb >= g.N) return;
    i32x4 sum = {0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < PW; ++w) sum += part[w][wave][lane];
    uint32_t packed = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        int32_t a = sum[e], cs = 0;
        if (need_colsum) {
#pragma unroll
            for (int w = 0; w < NW; ++w) cs += csum[w][4 * quarter + e];
        }
        if (INT4) {
            a >>= 4; // weights were kept times 16; exact
            cs >>= 4;
        }
        a += (g.bias ? p_bias[e] : 0) + (128 - g.z_a) * cs;
        const int32_t y = clamp_i32(g.lo_rel, g.hi_rel, rescale_general(a, make_rescale(p_mult[e], p_shift[e]))) + g.z_out;
        packed |= (uint32_t)y << (8 * e);
    }
    uint8_t *dst = g.C + m * g.ldc + nb;
    if (nb + 4 <= g.N) {
        __builtin_memcpy(dst, &packed, 4);
    } else {
        for (int e = 0; nb + e < g.N; ++e) dst[e] = (uint8_t)(packed >> (8 * e));
    }
}

} // namespace qnn
