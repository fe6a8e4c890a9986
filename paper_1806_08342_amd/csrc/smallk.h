// Quantized product for launches that are small altogether: few rows (M <= 64, a fully connected layer at
// small batch), or any matrix / convolution whose work does not fill the chip (networks at batch 1).
//
// Such a launch is bound by latencies and, with few rows, by streaming the weights once, so the kernel is
// organised around memory-level parallelism, not MFMA rate: one workgroup owns 16 output columns of up to
// 64 rows, its 4, 8 or 16 waves split K between them, and every wave keeps a whole batch of K-steps in flight.
// On 64x64 tiles the same K loop is a serial chain of barriers, 0.2 us per 64 k behind 4 us of set-up (7x7x512
// -> 512, 3x3: 31 us; 196 x 512 x 512: 5.8 us; here 6.0 and 3.0).
// The roles of the operands are swapped with respect to the big kernel: the weights are the A operand of
// v_mfma_i32_16x16x64_i8 (16 columns n x 64 k) and the activations the B operand (16 rows m), so a lane
// ends up with 4 consecutive output columns of one row m: one dword store, no transposition.
//
// A fragment has its 16 rows in 16 consecutive lanes.  Loaded like that, every lane sits on a cache line
// of its own and the vector cache delivers 15 bytes per clock and CU whatever the hit rate (measured
// 9.3 TB/s over the chip from L2, against 31 TB/s when 8 consecutive lanes read one 128-byte line).  So a
// load takes 8 rows x 128 bytes, and the rows change places in 4 KB of LDS that belong to the wave alone
// (no barrier; chunk c of row r sits at c ^ (r / 2), conflict-free for the 8-bit fragment reads).
//
// A K-step is 128 bytes of every weight row: 128 weights, or 256 packed 4-bit weights, which are widened in
// registers (kept times 16 in int8, accumulators shifted back exactly).
//
// Any K, any pitch, any alignment: gfx950 loads 16 bytes from any byte address, and the piece that
// sticks out of a row's end is read from K - 16 instead and shifted (load_tail16).  Only the last,
// partial K-step pays for that.  The per-column parameters are requested before the main loop: behind
// the reduction their latency was a fifth of the kernel (M = 1, 4096 x 4096).
#pragma once

#include "fill_table.h"
#include "igemm.h"

namespace qnn {

struct SmallArgs {
    IgemmArgs g;
    // convolutions: pixel m -> (image, ho, wo) by multiply-high: m / (Ho * Wo) and rest / Wo, m < 2^31
    uint32_t magic_hw, shift_hw, magic_wo, shift_wo;
};

__device__ __forceinline__ uint32_t div_magic(uint32_t x, uint32_t d, uint32_t magic, uint32_t shift)
{
    return d == 1 ? x : __umulhi(x, magic) >> shift;
}

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

// AI: load instructions per 128 bytes of the activation rows, 8 rows each (a workgroup owns 8 * AI rows).
// A_CONV: the 16-byte chunks of a row are gathered from the image; Cin % 16 == 0, so a chunk lies inside one tap.
// SMALL_ZW: per-column weight zero-points (see igemm_epilogue_impl).
// SMALL_ADD: the rescaling add with g.R.  A lane ends up with 4 codes of one row, so it needs one dword of the residual,
// requested with the per-column parameters; the tables of the add are filled while these are on their way.
enum SmallExtra { SMALL_PLAIN, SMALL_ZW, SMALL_ADD };

template <int AI, bool INT4, int NW, int A_MODE, SmallExtra EXTRA>
__global__ void __launch_bounds__(NW * 64) smallk_kernel(const SmallArgs args)
{
    const IgemmArgs &g = args.g;
    constexpr bool ZW = EXTRA == SMALL_ZW, ADD = EXTRA == SMALL_ADD;
    constexpr int MT = (AI + 1) / 2, BN = 16, STEP = INT4 ? 256 : 128, HALVES = STEP / 128;
    constexpr int STEP_REGS = 4 * (2 + AI * HALVES);
    constexpr int UNROLL = STEP_REGS <= 16 ? 4 : (STEP_REGS <= (NW > 8 ? 24 : 40) ? 2 : 1); // steps in flight per wave (what the registers hold)
    constexpr int PW = NW < 8 ? NW : 8; // waves whose partial sums fit LDS at a time
    static_assert(NW * 4096 >= PW * MT * 1024, "the partial sums take the place of the row exchange");
    __shared__ __attribute__((aligned(16))) uint8_t smem[NW * 4096];
    __shared__ int32_t csum[NW][BN];
    __shared__ int32_t rsum[ZW ? NW : 1][MT][16];
    __shared__ int32_t add_tab[ADD ? 512 : 1];
    i32x4(*const part)[MT][64] = reinterpret_cast<i32x4(*)[MT][64]>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6); // wave-uniform
    const int n0 = blockIdx.x * BN;
    const int64_t m0 = (int64_t)blockIdx.y * (8 * AI);
    const int frow = lane & 15, quarter = lane >> 4; // fragment layout
    const int lrow = lane >> 3, lchunk = lane & 7;   // load layout

    // weight and activation rows this lane loads from, clamped
    const uint8_t *brow[2], *arow[AI];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int n = n0 + 8 * i + lrow;
        n = n < g.N ? n : g.N - 1;
        brow[i] = INT4 ? g.B + (((int64_t)n * g.ldb) >> 1) : g.B + (int64_t)n * g.ldb;
    }
    int hi0[AI], wi0[AI]; // A_CONV: window origin; arow then points at its (possibly outside) pixel
#pragma unroll
    for (int i = 0; i < AI; ++i) {
        int64_t m = m0 + 8 * i + lrow;
        m = m < g.M ? m : g.M - 1;
        if constexpr (A_MODE == A_MATRIX) {
            arow[i] = g.A + m * g.lda;
        } else {
            const uint32_t img = div_magic((uint32_t)m, (uint32_t)(g.Ho * g.Wo), args.magic_hw, args.shift_hw);
            const uint32_t rest = (uint32_t)m - img * (uint32_t)(g.Ho * g.Wo);
            const uint32_t ho = div_magic(rest, (uint32_t)g.Wo, args.magic_wo, args.shift_wo), wo = rest - ho * (uint32_t)g.Wo;
            hi0[i] = (int)ho * g.sh - g.ph;
            wi0[i] = (int)wo * g.sw - g.pw;
            arow[i] = g.A + (((int64_t)img * g.H + hi0[i]) * g.W + wi0[i]) * g.Cin;
        }
    }
    // chunk of 16 activations at k (the lane's) of every row; TAIL: k may reach beyond K
    auto load_a = [&](int k, auto tail, u32x4 (&v)[AI]) __attribute__((always_inline)) {
        if constexpr (A_MODE == A_MATRIX) {
#pragma unroll
            for (int i = 0; i < AI; ++i) v[i] = decltype(tail)::value ? load_tail16(arow[i], k, g.K) : load16_any(arow[i] + k);
        } else { // taps outside the image, and taps beyond the kernel that fall outside, read as the code z_a
            const uint32_t tap = fast_div((uint32_t)k, (uint32_t)g.Cin, g.magic_cin);
            const uint32_t ta = fast_div(tap, (uint32_t)g.kw, g.magic_kw);
            const int a = (int)ta, b = (int)(tap - ta * (uint32_t)g.kw);
            const int64_t delta = ((int64_t)a * g.W + b) * g.Cin + (k - (int)tap * g.Cin);
            const uint8_t *const fill = &g_fill_table.v[g.z_a][0];
#pragma unroll
            for (int i = 0; i < AI; ++i) {
                const bool inside = (unsigned)(hi0[i] + a) < (unsigned)g.H && (unsigned)(wi0[i] + b) < (unsigned)g.W;
                v[i] = load16_any(inside ? arow[i] + delta : fill);
                if constexpr (ZW && decltype(tail)::value) // beyond K: zero like a matrix row's tail (the row sum is corrected for it)
                    if (k >= g.K) v[i] = u32x4{0, 0, 0, 0};
            }
        }
    };
    // The partial step of rows that are whole 16-byte pieces.  With a branch around every load, as other rows need it, it is
    // a chain of waits: 64 columns of K = 64 over 3197 rows in 5.1 us (3.7 warm), 3.8 (3.4) like this, 4.1 on the short-K kernel.
    auto load_tail_whole = [&](int kb, int wlen, u32x4 (&wv)[2], u32x4 (&av)[HALVES][AI]) __attribute__((always_inline)) {
        const bool beyond = kb >= wlen;
#pragma unroll
        for (int i = 0; i < 2; ++i) wv[i] = load16_any(brow[i] + (beyond ? wlen - 16 : kb));
#pragma unroll
        for (int p = 0; p < HALVES; ++p) {
            const int k = g.K / STEP * STEP + p * 128 + 16 * lchunk;
            if constexpr (A_MODE == A_MATRIX) {
#pragma unroll
                for (int i = 0; i < AI; ++i) av[p][i] = load16_any(arow[i] + (k < g.K ? k : g.K - 16));
            } else {
                load_a(k, std::true_type{}, av[p]);
            }
        }
        if (beyond) wv[0] = wv[1] = u32x4{0, 0, 0, 0}; // and the activations meet zero weights
        if constexpr (ZW && A_MODE == A_MATRIX) { // ... but count in the row sum
#pragma unroll
            for (int p = 0; p < HALVES; ++p)
#pragma unroll
                for (int i = 0; i < AI; ++i)
                    if (g.K / STEP * STEP + p * 128 + 16 * lchunk >= g.K) av[p][i] = u32x4{0, 0, 0, 0};
        }
    };
    // row exchange: 16 weight rows, behind them 16 activation rows, of 128 bytes each
    uint8_t *const xb = smem + wave * 4096, *const xa = xb + 2048;
    auto slot = [](int row, int chunk) { return row * 128 + ((chunk ^ (row >> 1)) & 7) * 16; };
    const int put[2] = {slot(lrow, lchunk), slot(8 + lrow, lchunk)};
    int get_b[2], get_a[2]; // chunk read for matrix instruction h (4-bit weights: for pair h of instructions, see multiply)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        get_b[h] = slot(frow, 4 * h + quarter);
        get_a[h] = slot(frow, INT4 ? 2 * quarter + h : 4 * h + quarter);
    }

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
    uint32_t residual = 0;
    if constexpr (ADD) {
        if (wave < MT) {
            const int64_t m = m0 + wave * 16 + frow;
            const uint8_t *const r = g.R + (m < g.M ? m : g.M - 1) * g.ldr;
            if (nb + 4 <= g.N) {
                __builtin_memcpy(&residual, r + nb, 4);
            } else {
                for (int e = 0; nb + e < g.N; ++e) residual |= (uint32_t)r[nb + e] << (8 * e);
            }
        }
        add_fill_tables(add_tab, g.add, tid, NW * 64);
    }

    i32x4 acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = i32x4{0, 0, 0, 0};
    int32_t colsum = 0, rowsum[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) rowsum[t] = 0;
    const bool need_colsum = g.z_a != 128;
    // orders the wave's own row exchange for the compiler (other lanes read what a lane stores); the hardware keeps LDS
    // accesses of a wave in order, so it costs no wait
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    };
    // one step: wv the weight rows, av the activation rows, by halves of 128 bytes
    auto multiply = [&](const u32x4 (&wv)[2], const u32x4 (&av)[HALVES][AI]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) *reinterpret_cast<u32x4 *>(xb + put[i]) = wv[i];
        wave_sync();
        u32x4 w[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) w[h] = *reinterpret_cast<const u32x4 *>(xb + get_b[h]);
#pragma unroll
        for (int p = 0; p < HALVES; ++p) {
            // the weights of the two matrix instructions on activation half p.  8-bit: chunk 4 h + q, k = 64 h + 16 q + (0..15).
            // 4-bit: chunk 4 p + q holds k = 128 p + 32 q + (0..31), instruction h takes 16 h + (0..15) of them, on both
            // operands alike -- a sum does not care about the order of its terms.
            i32x4 fb[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if constexpr (INT4) fb[h] = expand_int4(u32x2{w[p][2 * h], w[p][2 * h + 1]});
                else fb[h] = i32x4{(int32_t)w[h].x, (int32_t)w[h].y, (int32_t)w[h].z, (int32_t)w[h].w};
            }
            if (need_colsum) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int d = 0; d < 4; ++d) colsum = __builtin_amdgcn_sdot4(fb[h][d], 0x01010101, colsum, false);
            }
#pragma unroll
            for (int t = 0; t < MT; ++t) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (2 * t + i < AI) *reinterpret_cast<u32x4 *>(xa + put[i]) = av[p][2 * t + i] ^ 0x80808080u; // code -> signed (code - 128)
                wave_sync();
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const i32x4 xs = *reinterpret_cast<const i32x4 *>(xa + get_a[h]); // (AI odd: rows 8..15 of the tile are nobody's)
                    acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[h], xs, acc[t], 0, 0, 0);
                    if constexpr (ZW) add_rowsum(rowsum[t], xs);
                }
                wave_sync(); // before the next rows take the place of these
            }
        }
    };

    const int steps = g.K / STEP;
    // `count` steps of this wave, all their loads ahead of the first wait
    auto batch = [&](int s0, auto count) __attribute__((always_inline)) {
        constexpr int U = decltype(count)::value;
        u32x4 wv[U][2], av[U][HALVES][AI];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int st = s0 + u * NW;
#pragma unroll
            for (int i = 0; i < 2; ++i) wv[u][i] = load16_any(brow[i] + st * 128 + 16 * lchunk);
#pragma unroll
            for (int p = 0; p < HALVES; ++p) load_a(st * STEP + p * 128 + 16 * lchunk, std::false_type{}, av[u][p]);
        }
        asm volatile("" ::: "memory"); // the loads stay where they are
#pragma unroll
        for (int u = 0; u < U; ++u) multiply(wv[u], av[u]);
    };
    int s0 = wave;
    for (; s0 + (UNROLL - 1) * NW < steps; s0 += UNROLL * NW) batch(s0, std::integral_constant<int, UNROLL>{});
    if (UNROLL > 3 && s0 + 2 * NW < steps) batch(s0, std::integral_constant<int, UNROLL < 3 ? UNROLL : 3>{});
    else if (UNROLL > 2 && s0 + NW < steps) batch(s0, std::integral_constant<int, UNROLL < 2 ? UNROLL : 2>{});
    else if (s0 < steps) batch(s0, std::integral_constant<int, 1>{});
    if (steps * STEP < g.K && wave == steps % NW) { // the partial step: weights beyond K read as zero
        u32x4 wv[2], av[HALVES][AI];
        const int kb = steps * 128 + 16 * lchunk, wlen = INT4 ? g.K >> 1 : g.K; // bytes of a weight row
        if ((wlen & 15) == 0) { // pieces lie inside the row or outside: all loads at once, from clamped addresses
            load_tail_whole(kb, wlen, wv, av);
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) wv[i] = load_tail16(brow[i], kb, wlen);
#pragma unroll
            for (int p = 0; p < HALVES; ++p) load_a(steps * STEP + p * 128 + 16 * lchunk, std::true_type{}, av[p]);
        }
        multiply(wv, av);
    }

    // ---- combine the waves (16 waves: the second half hands its sums to the first one)
    colsum += __shfl_xor(colsum, 16);
    colsum += __shfl_xor(colsum, 32);
    if (lane < BN) csum[wave][lane] = colsum;
    if constexpr (ZW) {
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            int32_t r = rowsum[t];
            r += __shfl_xor(r, 16);
            r += __shfl_xor(r, 32);
            if (lane < 16) rsum[wave][t][lane] = r;
        }
    }
    __syncthreads(); // every wave is done with its row exchange
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
    const int64_t m = m0 + wave * 16 + frow;
    if (m >= g.M || nb >= g.N) return;
    i32x4 sum = {0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < PW; ++w) sum += part[w][wave][lane];
    int32_t rs = 0; // sum_k (code - z_a) of this row: the parts count code - 128, and -128 for every k of the last step beyond K
    if constexpr (ZW) {
#pragma unroll
        for (int w = 0; w < NW; ++w) rs += rsum[w][wave][frow];
        rs += 128 * ((g.K + STEP - 1) / STEP * STEP - g.K) + g.K * (128 - g.z_a);
    }
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
        if constexpr (ZW) a = (int32_t)((uint32_t)a - (uint32_t)g.zw[nb + e < g.N ? nb + e : g.N - 1] * (uint32_t)rs);
        const int32_t y = clamp_i32(g.lo_rel, g.hi_rel, rescale_general(a, make_rescale(p_mult[e], p_shift[e]))) + g.z_out;
        packed |= (uint32_t)y << (8 * e);
    }
    if constexpr (ADD) {
        const AddOut ao = make_add_out(g.add);
        packed = ao.fused ? add_codes4<true>(packed, residual, add_tab, ao) : add_codes4<false>(packed, residual, add_tab, ao);
    }
    uint8_t *dst = g.C + m * g.ldc + nb;
    if (nb + 4 <= g.N) {
        __builtin_memcpy(dst, &packed, 4);
    } else {
        for (int e = 0; nb + e < g.N; ++e) dst[e] = (uint8_t)(packed >> (8 * e));
    }
}

} // namespace qnn
