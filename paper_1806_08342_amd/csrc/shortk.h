// Dense quantized layer with a short reduction (K <= 256, K % 8 == 0) where shortk_ring.h is not ahead (small launches, mostly: see
// ring_ahead) or does not apply: rows that are whole 8-byte pieces only, or pitches beyond its 32-bit offsets.  Here also: what the
// two kernels share, the epilogue constants of a column and the add of two codes by table.
//
// Weight-stationary and barrier-free: a wave owns up to 32*NB output columns, loads their weights
// ONCE into registers as MFMA B fragments (4-bit weights are unpacked there, kept times 16),
// derives the per-column epilogue constants once (column sums for the zero-point correction,
// bias, fixed-point multiplier and shift), and then walks over blocks of 32 rows: the A fragments
// of a block come straight from global memory (each lane fetches the 16 bytes its MFMA operand
// needs; the next block's are requested as soon as the current block's MFMAs are issued), NB*KS MFMAs,
// epilogue, and the 32 x 32*NB byte tile goes through a wave-private LDS area to become 16-byte
// row stores.  Waves never synchronise with each other; a workgroup is just four such waves on
// neighbouring column groups of the same rows (they share the A rows through the vector cache).
// Arithmetic as in igemm.h (eq. 4-6 with z_w = 0, bias, RESCALE, clamp).
#pragma once

#include <type_traits>

#include "arguments.h"
#include "igemm.h"

namespace qnn {

struct ShortKArgs {
    IgemmArgs g;       // A_MATRIX fields, or the geometry of a strided 1x1 convolution
    int col_groups;    // ceil(N / (32 * NB))
    int walkers;       // waves that share one column group (they interleave over the row blocks)
    int strided;       // rows of A are pixels (n, ho*sh, wo*sw) of an NHWC image (1x1 convolution, stride > 1)
    int stream_out;    // non-temporal output stores
};

// Whether the add of a launch goes through the 65536-entry table of code pairs: from 2^24 outputs on it pays for itself; below,
// two 256-entry tables.
inline bool shortk_pairs(const IgemmArgs &g) { return g.M * (int64_t)g.N >= ((int64_t)1 << 24); }

// 16 consecutive k of one row / column as 4 dwords, zero beyond K (K % 8 == 0).  VEC = bytes per load; 16 (K % 16 == 0, any
// address): without a branch, from a clamped address, and beyond K any bytes (the other operand is zero there).
template <int VEC> __device__ __forceinline__ i32x4 shortk_load16(const uint8_t *p, int k, int K)
{
    i32x4 v = {0, 0, 0, 0};
    if constexpr (VEC == 16) {
        __builtin_memcpy(&v, p + (k + 16 <= K ? k : K - 16), 16);
    } else if constexpr (VEC == 8) {
        if (k + 8 <= K) {
            const u32x2 a = *reinterpret_cast<const u32x2 *>(p + k);
            v[0] = (int32_t)a.x, v[1] = (int32_t)a.y;
        }
        if (k + 16 <= K) {
            const u32x2 b = *reinterpret_cast<const u32x2 *>(p + k + 8);
            v[2] = (int32_t)b.x, v[3] = (int32_t)b.y;
        }
    } else {
#pragma unroll
        for (int d = 0; d < 4; ++d)
            if (k + 4 * d + 4 <= K) v[d] = *reinterpret_cast<const int32_t *>(p + k + 4 * d);
    }
    return v;
}

// Epilogue constants of one column (ChannelRescale: fused forms; the rest: general form and weight zero-points)
struct ShortKColumn {
    ChannelRescale r;
    int32_t mult, shift, zw;
};

// Constants of a column from the sum of its weights and its parameters; k_loaded: the k that a weight zero-point's
// activation sums run over (those from K on read as the code 0).
__device__ __forceinline__ void shortk_column(ShortKColumn &c, const IgemmArgs &g, int32_t colsum, int32_t bias, int32_t mult, int32_t shift,
                                              int32_t zw, int k_loaded)
{
    const int32_t corr = bias + (128 - g.z_a) * colsum - zw * (g.K * (128 - g.z_a) + 128 * (k_loaded - g.K));
    c.mult = mult, c.shift = shift, c.zw = zw;
    c.r = make_channel_rescale(mult, shift, corr, g.z_out, g.lo_rel + g.z_out, g.hi_rel + g.z_out, rescale_ties(g.lo_rel));
}

// All 65536 results of an add from its tables of rescaled codes (add_fill_tables).  Entry [m][r] = code of the sum, at
// byte 256 m + (r ^ 4 (m % 64)): the bank of a gather then depends on both codes.  (With r alone choosing the bank, the
// lanes whose residual is the code of zero, half of them behind a ReLU, met in one bank.)  A lane fills the same 4
// consecutive r for every m of its wave, so that the value of m is one broadcast read and those of r stay in registers.
template <int WAVES> __device__ __forceinline__ void fill_pair_table(uint8_t *pair_tab, const int32_t *tab, const AddParams &add)
{
    const int r0 = (int)(threadIdx.x & 63u) * 4;
    int32_t tr[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) tr[e] = tab[256 + r0 + e];
    uint32_t *const out = reinterpret_cast<uint32_t *>(pair_tab);
    const AddParams &p = add;
    const bool ties = rescale_ties(p.act_min - p.z_out);
    const ChannelRescale r = make_channel_rescale(p.mult_o, p.shift_o, 0, p.z_out, p.act_min, p.act_max, ties);
    const AddOut ao = make_add_out(p);
    with_rescale_mode(ao.fused && channel_rescale_ok(p.mult_o, p.shift_o, ties), p.z_out, p.act_min - p.z_out, p.act_max - p.z_out, [&](auto mode_tag) {
        using Mode = RescaleModeTraits<decltype(mode_tag)::value>;
#pragma unroll 4
        for (int i = 0; i < 256 / WAVES; ++i) {
            const int m = i * WAVES + (int)(threadIdx.x >> 6);
            const int32_t tm = tab[m];
            uint32_t x = 0;
            if constexpr (Mode::kFused) {
                const int32_t sum[4] = {tm + tr[0], tm + tr[1], tm + tr[2], tm + tr[3]};
                x = channel_codes4<Mode::kTies, Mode::kFull>(sum, r);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) x |= (ao.fused ? add_value1<true>(tm, tr[e], ao) : add_value1<false>(tm, tr[e], ao)) << (8 * e);
            }
            out[m * 64 + ((threadIdx.x ^ (uint32_t)m) & 63u)] = x;
        }
    });
}

// 4 codes of the layer (v) and of the residual (r): the byte pairs are interleaved into 16-bit indices of the table, one
// byte gather each
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void pairs_lookup(const uint8_t *pair_tab, uint32_t v, uint32_t r, u16x2 (&t)[2])
{
    const uint32_t rs = r ^ ((v << 2) & 0xfcfcfcfcu); // the table's order
    const uint32_t i01 = __builtin_amdgcn_perm(v, rs, 0x05010400u), i23 = __builtin_amdgcn_perm(v, rs, 0x07030602u);
    t[0] = u16x2{pair_tab[i01 & 0xffffu], pair_tab[i23 & 0xffffu]};
    t[1] = u16x2{pair_tab[i01 >> 16], pair_tab[i23 >> 16]};
}
__device__ __forceinline__ uint32_t pairs_combine(const u16x2 (&t)[2])
{
    return __builtin_bit_cast(uint32_t, t[0]) | (__builtin_bit_cast(uint32_t, t[1]) << 8);
}

// 16 codes of the layer and of the residual -> 16 output codes.  All 16 gathers are on their way before the first is combined.
__device__ __forceinline__ u32x4 add_pairs16(const uint8_t *pair_tab, u32x4 v, u32x4 r)
{
    u16x2 t[4][2];
#pragma unroll
    for (int d = 0; d < 4; ++d) pairs_lookup(pair_tab, v[d], r[d], t[d]);
    __builtin_amdgcn_sched_barrier(0);
    u32x4 y;
#pragma unroll
    for (int d = 0; d < 4; ++d) y[d] = pairs_combine(t[d]);
    return y;
}

// The same with the tables of an ADD form: 1 two 256-entry tables of rescaled codes, else the table of all pairs
template <int ADD> __device__ __forceinline__ u32x4 add_chunk(u32x4 v, u32x4 r, const uint8_t *pair_tab, const int32_t *tab, const AddOut &ao)
{
    u32x4 y;
    if constexpr (ADD >= 2) {
        y = add_pairs16(pair_tab, v, r);
    } else if (ao.fused) {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            y[d] = add_codes4<true>(v[d], r[d], tab, ao);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma nounroll
        for (int d = 0; d < 4; ++d) y[d] = add_codes4<false>(v[d], r[d], tab, ao);
    }
    return y;
}

// ZW: per-column weight zero-points (see igemm_epilogue_impl): the activation sum of a row is one more accumulator,
// fed by one matrix instruction per K sub-step whose B fragment is all ones, which leaves the sums in the registers
// and lanes where the rescale of the same rows needs them.
// VEC: bytes per load of the rows, 16 or 8.
// ADD (VEC 16): the rescaling add with a residual tensor (g.R), as in shortk_ring.h: 1 through two 256-entry tables, 2 through the
// table of all pairs, which eight waves share.
template <int NB, int KS, bool INT4, int VEC, int ADD = 0, bool ZW = false>
__global__ void __launch_bounds__(ADD == 2 ? 512 : 256, ADD == 2 ? 1 : (KS <= 1 && !ZW ? 3 : 2)) shortk_kernel(const ShortKArgs s)
{
    // (4-bit weights without the add: 6272 x 576 x 96 5.30 and 5.11 us, strided 16 x 56 x 56 x 96 -> 192 5.65 and 5.20; with 8-bit
    // weights matrices lose 1 to 2 %, with the add 0.5 %)
    if constexpr (INT4 && !ADD) fetch_arguments<sizeof(ShortKArgs)>();
    constexpr int PITCH = 32 * NB + 32; // bytes per staged output row: the 8 rows a store instruction touches fall in distinct banks
    constexpr int WAVES = ADD == 2 ? 8 : 4;
    __shared__ __attribute__((aligned(16))) uint8_t stage_static[ADD ? 16 : WAVES * 32 * PITCH];
    extern __shared__ __attribute__((aligned(16))) uint8_t shortk_lds[]; // ADD: tables, then the output tiles of the waves
    constexpr int TABLES = ADD == 2 ? 65536 : 2048;
    uint8_t *const stage_all = ADD ? shortk_lds + TABLES : stage_static;
    const IgemmArgs &g = s.g;
    int32_t *const tab = reinterpret_cast<int32_t *>(ADD == 2 ? stage_all : shortk_lds);
    if constexpr (ADD) { // the only workgroup barriers, before any wave may leave
        add_fill_tables(tab, g.add, threadIdx.x, WAVES * 64);
        __syncthreads();
        if constexpr (ADD == 2) {
            fill_pair_table<WAVES>(shortk_lds, tab, g.add);
            __syncthreads();
        }
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); // wave-uniform: row-block arithmetic stays scalar
    uint8_t *stage = stage_all + wave * (32 * PITCH);
    const int frow = lane & 31, fhalf = lane >> 5;

    // wave -> (column group, walker): neighbouring waves take neighbouring column groups of the same rows
    const int64_t gw = (int64_t)blockIdx.x * WAVES + wave;
    const int cg = (int)(gw % s.col_groups), walker = (int)(gw / s.col_groups);
    if (walker >= s.walkers) return; // no barriers below: a wave may leave alone
    const int n0 = cg * 32 * NB;
    const int blocks_here = (g.N - n0 + 31) / 32 < NB ? (g.N - n0 + 31) / 32 : NB; // column blocks that exist

    // ---- weights: B fragments of all K sub-steps, for good.  The parameters of the columns, all weights and the rows of the
    // first block are requested before any of them is waited for.
    i32x4 fb[KS][NB];
    u32x2 packed[INT4 ? KS : 1][INT4 ? NB : 1];
    ShortKColumn col[NB];
    int32_t p_bias[NB], p_mult[NB], p_shift[NB], p_zw[NB];
    const int32_t *const bias_or_any = g.bias ? g.bias : g.mult; // no branch around the load; the value is dropped below
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        int n = n0 + j * 32 + frow;
        n = n < g.N ? n : g.N - 1;
        p_bias[j] = bias_or_any[n], p_mult[j] = g.mult[n], p_shift[j] = g.shift[n];
        p_zw[j] = ZW ? g.zw[n] : 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int k = ks * 32 + fhalf * 16;
            if constexpr (INT4) {
                const uint8_t *p = g.B + (((int64_t)n * g.ldb) >> 1);
                if constexpr (VEC == 16) {
                    __builtin_memcpy(&packed[ks][j], p + ((k + 16 <= g.K ? k : g.K - 16) >> 1), 8);
                    continue;
                }
                packed[ks][j] = u32x2{0u, 0u};
                if (k + 16 <= g.K) __builtin_memcpy(&packed[ks][j], p + (k >> 1), 8);
                else if (k + 8 <= g.K) packed[ks][j][0] = *reinterpret_cast<const uint32_t *>(p + (k >> 1));
            } else {
                fb[ks][j] = shortk_load16<VEC == 16 ? 16 : 4>(g.B + (int64_t)n * g.ldb, k, g.K);
            }
        }
    }
    const int M = (int)g.M; // (the dispatcher guarantees M < 2^31)
    const int row_blocks = (M + 31) / 32;
    // ---- rows
    auto load_rows = [&](int rb, i32x4 (&fa)[KS]) __attribute__((always_inline)) {
        const uint8_t *p;
        int m = rb * 32 + frow;
        m = m < M ? m : M - 1;
        if (s.strided) {
            const uint32_t per_image = (uint32_t)g.Ho * (uint32_t)g.Wo;
            const uint32_t img = (uint32_t)m / per_image, rem = (uint32_t)m - img * per_image;
            const uint32_t ho = rem / (uint32_t)g.Wo, wo = rem - ho * (uint32_t)g.Wo;
            p = g.A + (((int64_t)img * g.H + ho * g.sh) * g.W + wo * g.sw) * g.Cin + fhalf * 16;
        } else {
            p = g.A + (int64_t)m * g.lda + fhalf * 16;
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) fa[ks] = shortk_load16<VEC>(p, ks * 32, g.K - fhalf * 16);
    };
    // (Not where these rows and the weights as loaded do not fit the registers together: the forms for K <= 128 with the add
    // spilled 12 to 52 bytes, 20000 x 144 x 112 11.5 us, not 11.0.)
    constexpr bool FIRST_AHEAD = VEC == 8 || (!ZW && !(ADD && KS == 4));
    i32x4 first[KS];
    if constexpr (FIRST_AHEAD) load_rows(walker < row_blocks ? walker : row_blocks - 1, first);

    bool range_ok = g.small_acc >= 2, fused_ok = true;
    const bool ties = rescale_ties(g.lo_rel);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        int32_t colsum = 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (INT4) fb[ks][j] = expand_int4(packed[ks][j]);
            if (VEC == 16 && ks * 32 + fhalf * 16 + 16 > g.K) fb[ks][j] = i32x4{0, 0, 0, 0};
#pragma unroll
            for (int d = 0; d < 4; ++d) colsum = __builtin_amdgcn_sdot4(fb[ks][j][d], 0x01010101, colsum, false);
        }
        colsum += __shfl_xor(colsum, 32);
        if (INT4) colsum >>= 4; // weights are kept times 16; exact
        // (the sums of ZW count code - 128; where pieces of 8 are loaded, also -128 for every k from K to KS * 32, read as zeros)
        const int32_t b = g.bias ? p_bias[j] : 0;
        shortk_column(col[j], g, colsum, b, p_mult[j], p_shift[j], p_zw[j], VEC == 16 ? g.K : KS * 32);
        range_ok = range_ok && rescale_in_range(p_shift[j]) && b > -(1 << 27) && b < (1 << 27);
        fused_ok = fused_ok && range_ok && channel_rescale_ok(p_mult[j], p_shift[j], ties);
    }
    const bool fused = __all(fused_ok), in_range = __all(range_ok), k_tail = VEC == 16 && g.K != KS * 32;
    const i32x4 ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};

    // lane-invariant parts of the LDS and global addresses of the output tile
    int st_lds[NB], st_row[NB];
    bool st_col_ok[NB];
    int64_t st_off[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int idx = i * 64 + lane;
        st_row[i] = idx / (2 * NB);
        const int col0 = n0 + (idx % (2 * NB)) * 16;
        st_col_ok[i] = col0 < g.N;
        st_lds[i] = st_row[i] * PITCH + (idx % (2 * NB)) * 16;
        st_off[i] = (int64_t)st_row[i] * g.ldc + col0;
    }
    const int put_base = (4 * fhalf + (lane & 3)) * PITCH + (frow & ~3);
    // whole 16-byte chunks only, all aligned: one store per lane and chunk, no tail handling
    const bool chunks_whole = g.c_vec16 && ((g.N & 15) == 0 || n0 + 32 * NB <= g.N);

    const int quad_lane = lane & 3;
    const uint32_t sel1 = (quad_lane & 1) ? 0x03070105u : 0x06020400u;
    const uint32_t sel2 = (quad_lane & 2) ? 0x03020706u : 0x05040100u;
    const int32_t lo_rel = g.lo_rel, hi_rel = g.hi_rel, z_out = g.z_out;

    // residual chunks of a row block (ADD), requested one round ahead: same lanes and addresses as the stores of that block
    int64_t st_roff[NB];
    u32x4 rres[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        st_roff[i] = (int64_t)st_row[i] * g.ldr + (n0 + (i * 64 + lane) % (2 * NB) * 16);
        rres[i] = u32x4{0u, 0u, 0u, 0u};
    }
    auto load_res = [&](int rbx) __attribute__((always_inline)) {
        const uint8_t *const r_block = g.R + (int64_t)rbx * 32 * g.ldr; // wave-uniform
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if (st_col_ok[i] && rbx * 32 + st_row[i] < M) rres[i] = *reinterpret_cast<const u32x4 *>(r_block + st_roff[i]);
    };
    const AddOut ao = make_add_out(g.add);

    // (Non-temporal stores, s.stream_out: 4-9 % on 6-26 MB outputs -- what is left in the L2s is written back when the
    // kernel ends.  Larger outputs and the add built in are faster with plain ones: ResNet-50 at batch 256, 103 MB,
    // K = 256: 84 us and 93 with non-temporal ones, 70 and 76; 51 MB, K = 256: 57 and 54, but the 3x3 layer that reads
    // them then takes 67 instead of 64.)
    // the output tile of row block rbx, from the wave's LDS area to global memory.  Called one
    // round late, right after the next block's MFMAs and the loads of the block after it are issued.
    auto store_block = [&](int rbx) __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        uint8_t *const c_block = g.C + (int64_t)rbx * 32 * g.ldc; // wave-uniform
        if constexpr (ADD) { // the launcher uses ADD only when every output chunk is a whole, aligned 16-byte chunk
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if (st_col_ok[i] && rbx * 32 + st_row[i] < M)
                    *reinterpret_cast<u32x4 *>(c_block + st_off[i]) = add_chunk<ADD>(*reinterpret_cast<const u32x4 *>(stage + st_lds[i]), rres[i], shortk_lds, tab, ao);
                __builtin_amdgcn_sched_barrier(0); // one chunk at a time: the table reads of all chunks at once would spill
            }
        } else if (chunks_whole && rbx * 32 + 32 <= M && s.stream_out) { // the common case: only the lane-invariant column test
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (st_col_ok[i])
                    __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(stage + st_lds[i]), reinterpret_cast<u32x4 *>(c_block + st_off[i]));
        } else if (chunks_whole && rbx * 32 + 32 <= M) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (st_col_ok[i])
                    *reinterpret_cast<u32x4 *>(c_block + st_off[i]) = *reinterpret_cast<const u32x4 *>(stage + st_lds[i]);
        } else if (chunks_whole) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (st_col_ok[i] && rbx * 32 + st_row[i] < M)
                    *reinterpret_cast<u32x4 *>(c_block + st_off[i]) = *reinterpret_cast<const u32x4 *>(stage + st_lds[i]);
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
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    // the row loop exists twice (fast and general epilogue) and the choice is made once, outside:
    // inside the loop the compiler would evaluate both forms for every output and select
    auto walk = [&](auto mode_tag) {
    using Mode = RescaleModeTraits<decltype(mode_tag)::value>;
    i32x4 fa[KS];
    int rb = walker, rb_stored = -1;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fa[ks] = first[ks];
    if constexpr (!FIRST_AHEAD) load_rows(rb < row_blocks ? rb : row_blocks - 1, fa);
    for (; rb < row_blocks; rb += s.walkers) {
        i32x16 acc[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][r] = 0;
        i32x16 sums = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}; // ZW: sum_k (code - 128) of the rows
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            i32x4 xs = fa[ks] ^ (int32_t)0x80808080; // uint8 code -> signed (code - 128)
            if constexpr (ZW) {
                if (k_tail && ks * 32 + fhalf * 16 >= g.K) xs = i32x4{0, 0, 0, 0}; // counts in the sum
                sums = __builtin_amdgcn_mfma_i32_32x32x32_i8(xs, ones, sums, 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < NB; ++j)
                acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xs, fb[ks][j], acc[j], 0, 0, 0); // columns past N: clamped loads, never stored
        }
        // The fragments are consumed: the next block's are requested into the same registers now, ahead of the stores, so that
        // the wait for them is no wait for these (requests retire in order).
        if (rb + s.walkers < row_blocks) load_rows(rb + s.walkers, fa);
        if (rb_stored >= 0) store_block(rb_stored);
        if constexpr (ADD) load_res(rb); // used one round from now, when this block is stored

        // ---- epilogue into the wave's LDS tile: after the 4x4 byte transposition inside each
        // quad of lanes a lane holds 4 consecutive columns of one row
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
                int32_t a[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    a[e] = acc[j][4 * q + e];
                    if (INT4) a[e] >>= 4;
                    if constexpr (ZW) a[e] -= __mul24(col[j].zw, sums[4 * q + e]);
                }
                if constexpr (Mode::kFused) put(j, q, channel_codes4<Mode::kTies, Mode::kFull>(a, col[j].r));
                else put(j, q, other_codes4(a, col[j].mult, col[j].shift, -col[j].r.ncorr, in_range, z_out, lo_rel, hi_rel));
            }
        }
        // the tile is private to the wave and LDS operations of one wave complete in order:
        // no barrier, only the data dependence through memory
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        rb_stored = rb; // its stores are issued in the next round, after that round's MFMAs
    }
    if (rb_stored >= 0) store_block(rb_stored);
    };
    with_rescale_mode(fused, z_out, lo_rel, hi_rel, walk);
}

} // namespace qnn
