// Dense quantized layer with a short reduction (K <= 256) whose rows are whole 16-byte pieces: 1x1 convolutions of any
// stride and GEMMs, bound by their memory streams, then by their epilogue.
//
// Weight-stationary, as shortk.h: a wave owns up to 32*NB output columns and keeps their B fragments and epilogue constants
// in registers.  What differs is how the operands get there.  A matrix-instruction fragment fetched straight from global
// memory puts every lane on a row of its own, and the texture path then takes 69 cycles per 1 KB: 15 bytes per cycle and CU
// (8 TB/s of the whole chip, once per column group), where copies into LDS run at 95 with 8 lanes per 128-byte line and 128
// with contiguous rows.  So
//  - the rows travel by buffer_load_dwordx4 ... lds into a ring of blocks.  WIDE: four waves of a workgroup own neighbouring
//    column groups of the same 32 rows and share them, one barrier per step; else a wave has rows of its own and no barrier.
//    The fragments of the next step are read back under the epilogue of this one, and all blocks of the ring but the one
//    in use are on their way, so that the wait for a step's rows is no wait for the stores of the last;
//  - the weights are loaded as whole rows too and exchanged through LDS (64 KB of them as fragments took 4 us of a launch).
// us before (fragments from global memory) and now: see launch_shortk.
#pragma once

#include "arguments.h"
#include "buffer_ops.h"
#include "lds_ring.h"
#include "shortk.h"

namespace qnn {

struct ShortKRingArgs {
    ShortKArgs s;                     // walkers: workgroups that share a set of column groups
    int steps, more;                  // every walker takes `steps` steps, the first `more` of them one more
    int whole;                        // output chunks of 16 bytes are aligned and the offsets of 32 rows fit 31 bits
    uint32_t magic_image, magic_row;  // STRIDED: ceil(2^32 / d) of Ho * Wo and of Wo, 0 for d = 1
};

// waits until at most N requests to memory are outstanding; nothing that touches memory is moved across
template <int N> __device__ __forceinline__ void wait_requests() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// ... n, rounded down to one of the cases
__device__ __forceinline__ void wait_requests_at_most(int n)
{
    if (n >= 16) wait_requests<16>();
    else if (n >= 8) wait_requests<8>();
    else if (n >= 6) wait_requests<6>();
    else if (n >= 4) wait_requests<4>();
    else if (n >= 2) wait_requests<2>();
    else if (n >= 1) wait_requests<1>();
    else wait_requests<0>();
}

// ... of YOUNGER + min(step, LAST) * MOVES
template <int YOUNGER, int MOVES, int LAST> __device__ __forceinline__ void wait_requests_of_step(int step)
{
    if constexpr (LAST == 0) {
        wait_requests<YOUNGER>();
    } else {
        if (step >= LAST) wait_requests<YOUNGER + LAST * MOVES>();
        else wait_requests_of_step<YOUNGER, MOVES, LAST - 1>(step);
    }
}

// LDS layout of a block of 32 rows: CPR 16-byte chunks per row, a power of two (those beyond K hold zeros), chunk c of row r at
// place c ^ turn(r), so that the 16 rows that share a cycle of a 16-byte read fall into 16 different bank groups
constexpr int ring_chunks(int ks) { return ks <= 1 ? 2 : ks <= 2 ? 4 : ks <= 4 ? 8 : 16; }
template <int CPR> __device__ __forceinline__ int ring_place(int row, int c)
{
    constexpr int kShift = CPR == 16 ? 0 : CPR == 8 ? 1 : CPR == 4 ? 2 : 3;
    return c ^ ((row >> kShift) & (CPR - 1));
}

// Waves of a workgroup and its dynamic LDS: tables, output tiles of the waves, ring.  Two workgroups of four waves per CU, three or
// four of the forms that have the registers for it (us with two and with three or four: 401408 x 64 x 64 12.4 and 10.9, 100352 x 64 x
// 128 7.3 and 6.5, 401408 x 32 x 32 8.5 and 8.0; small launches and 128 columns level, 401408 x 32 x 128 13.7 and 14.6), with the
// pair table one of eight or sixteen waves; the ring has what is left of the LDS, up to eight blocks, and its first CW blocks (with
// the pair table: its place) are where the weights are exchanged before.
template <int NB, int KS, int ADD, bool WIDE, bool ZW> struct RingGeometry {
    static constexpr int kWaves = ADD == 3 ? 16 : ADD == 2 ? 8 : 4;
    static constexpr int kCw = ADD == 3 ? (WIDE ? 8 : 4) : (WIDE ? 4 : 1), kRw = kWaves / kCw; // waves side by side, and on other rows
    static constexpr int kResident = ADD >= 2 ? 1 : ADD || ZW ? 2 : KS <= 4 && NB * KS <= 4 ? (NB <= 2 ? 4 : 3) : NB == 2 && KS <= 4 ? 3 : 2; // workgroups per CU
    static constexpr int kPitch = 32 * NB + 32; // bytes per staged output row: the 8 rows a store instruction touches fall in distinct banks
    static constexpr int kPerSimd = ADD == 3 ? 4 : kResident; // waves that the registers have to hold, at least
    static constexpr int kTables = ADD >= 2 ? 65536 : (ADD == 1 ? 2048 : 0);
    static constexpr int kStage = kWaves * 32 * kPitch;
    static constexpr int kBlock = ring_chunks(KS) * 512; // 32 rows
    static constexpr int kFit = (160 * 1024 / kResident - kTables - kStage) / (kRw * kBlock);
    static constexpr int kDepth = kFit < 8 ? kFit : 8;
    static constexpr int kAhead = ADD >= 2 ? kDepth : kDepth - kCw; // blocks requested before the weights are in place
    static constexpr bool kFits = kDepth >= 2 && kAhead >= 1;
    static constexpr int kLds = kTables + kStage + kDepth * kRw * kBlock;
};

// ADD: the rescaling add with a residual tensor (g.R) is applied to the output tile on its way from LDS to global memory; the
// residual chunks of a row block are requested one step ahead.  1: through two 256-entry tables of rescaled codes.  2: the add is
// a function of two 8-bit codes, so the workgroup (8 waves here, to share it) first tabulates all 65536 results in LDS; combining
// a pair of codes is then one byte gather.  3: the same with 16 waves of half the columns, whose gathers, rescale
// and memory streams overlap better, for more reads of the ring: 200704 x 512 x 128 62 -> 60 us, but 50176 x 1024 x 256 42 -> 43 and
// 802816 x 256 x 64 level, so for 96 < K <= 128 only.  Which launches have the add here: launch_ring_add.
// ZW: per-column weight zero-points, as in shortk.h.  STRIDED: rows are the pixels of a strided 1x1 convolution.
// The set-up is kept short, small launches consist of it: 32-bit offsets, no division.
template <int NB, int KS, bool INT4, int ADD, bool WIDE, bool ZW, bool STRIDED>
__global__ void __launch_bounds__((RingGeometry<NB, KS, ADD, WIDE, ZW>::kWaves * 64), (RingGeometry<NB, KS, ADD, WIDE, ZW>::kPerSimd)) shortk_ring_kernel(const ShortKRingArgs ra)
{
    fetch_arguments<sizeof(ShortKRingArgs)>();
    using G = RingGeometry<NB, KS, ADD, WIDE, ZW>;
    constexpr int PITCH = G::kPitch, WAVES = G::kWaves, CPR = ring_chunks(KS), KP = CPR / 2, CW = G::kCw, RW = G::kRw, DEPTH = G::kDepth;
    extern __shared__ __attribute__((aligned(16))) uint8_t dyn_lds[];
    const ShortKArgs &s = ra.s;
    const IgemmArgs &g = s.g;
    uint8_t *const pair_tab = dyn_lds, *const stage_all = dyn_lds + G::kTables, *const ring = stage_all + G::kStage;
    constexpr bool use_pairs = ADD >= 2;
    int32_t *const tab = reinterpret_cast<int32_t *>(use_pairs ? stage_all : pair_tab);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t *const stage = stage_all + wave * (32 * PITCH);
    const int frow = lane & 31, fhalf = lane >> 5;

    // ---- workgroup -> (set of column groups y, walker): the grid is 8 x sets x walkers / 8, so that the sets of one walker's rows
    // run on one XCD and share them in its L2
    const int group = (int)blockIdx.y;
    const int walker = (int)(blockIdx.z * 8 + blockIdx.x);
    if (walker >= s.walkers) return; // the whole workgroup
    const int wc = wave % CW, wr = wave / CW;
    const bool active = group * CW + wc < s.col_groups; // the others only help with the copies and the barriers
    const int cg = active ? group * CW + wc : s.col_groups - 1;
    const int n0 = cg * 32 * NB;
    const int blocks_here = (g.N - n0 + 31) / 32 < NB ? (g.N - n0 + 31) / 32 : NB;
    const int M = (int)g.M; // (the dispatcher guarantees M < 2^30)
    const int steps = ra.steps + (walker < ra.more ? 1 : 0); // at least one

    // ---- rows of step `step` into block `at` of the ring, by buffer loads: offsets that do not change from step to step, rows
    // beyond M out of the resource's bounds, past the last step everything.  A wave copies the pieces of 1 KB wc, wc + CW, ... of
    // its 32 rows (the last one again where there are fewer: every wave issues PIECES of them, which the waits count).
    // (As global_load_lds the compiler takes a copy for a flat access and drains every request at the next use of a loaded
    // register, the residual's here.)
    constexpr uint32_t NOWHERE = 0x80000000u; // beyond the bounds of every buffer
    constexpr int PIECES = (KP + CW - 1) / CW; // KP pieces per 32 rows
    constexpr int BLOCK_BYTES = RW * G::kBlock;
    auto piece_of = [&](int i) { return KP % CW == 0 || wc + i * CW < KP ? wc + i * CW : KP - 1; };
    int piece_row[PIECES];
    uint32_t piece_k[PIECES];
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
        piece_row[i] = piece_of(i) * (64 / CPR) + lane / CPR;
        const int k = ring_place<CPR>(piece_row[i], lane % CPR) * 16; // (its own inverse)
        piece_k[i] = k < g.K ? (uint32_t)(k + (STRIDED ? 0 : piece_row[i] * (int)g.lda)) : NOWHERE;
    }
    auto request = [&](int step, int at) __attribute__((always_inline)) {
        const int first = ((walker + step * s.walkers) * RW + wr) * 32; // past the last step beyond M
        const int rows = M - first < 32 ? M - first : 32;
        uint8_t *const dst = ring + at * BLOCK_BYTES + wr * G::kBlock;
        if constexpr (STRIDED) {
            // relative to the image of the first row (the dispatcher has checked that 32 rows span less than 2 GiB)
            const uint32_t per_image = (uint32_t)g.Ho * (uint32_t)g.Wo;
            uint32_t rem, wo;
            const uint32_t img0 = ring_div((uint32_t)(first < M ? first : M - 1), per_image, ra.magic_image, rem);
            const uint8_t *const base = g.A + (int64_t)img0 * g.H * g.W * g.Cin;
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                int m = first + piece_row[i];
                m = m < M ? m : M - 1;
                const uint32_t img = ring_div((uint32_t)m, per_image, ra.magic_image, rem);
                const uint32_t ho = ring_div(rem, (uint32_t)g.Wo, ra.magic_row, wo);
                const uint32_t offset = (((img - img0) * (uint32_t)g.H + ho * (uint32_t)g.sh) * (uint32_t)g.W + wo * (uint32_t)g.sw) * (uint32_t)g.Cin;
                buffer_to_lds16(base, rows > 0 ? 0x7fffffff : 0, piece_k[i] == NOWHERE ? NOWHERE : offset + piece_k[i], dst + piece_of(i) * 1024);
            }
        } else {
            const uint8_t *const base = g.A + (int64_t)first * g.lda;
            const int bytes = rows > 0 ? (rows - 1) * (int)g.lda + g.K : 0;
#pragma unroll
            for (int i = 0; i < PIECES; ++i) buffer_to_lds16(base, bytes, piece_k[i], dst + piece_of(i) * 1024);
        }
    };
    auto read_rows = [&](int at, i32x4 (&fa)[KS]) __attribute__((always_inline)) {
        const uint8_t *const base = ring + at * BLOCK_BYTES + wr * G::kBlock + frow * (CPR * 16);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) fa[ks] = *reinterpret_cast<const i32x4 *>(base + ring_place<CPR>(frow, 2 * ks + fhalf) * 16);
    };

    // ---- set-up: parameters, weights (whole rows, 16 k per lane) and the first steps' rows are requested before any is waited for
    using Piece = std::conditional_t<INT4, u32x2, u32x4>;
    constexpr int PB = INT4 ? 8 : 16;
    int32_t p_bias[NB], p_mult[NB], p_shift[NB], p_zw[NB];
    const int32_t *const bias_or_any = g.bias ? g.bias : g.mult; // no branch around the load; the value is dropped below
    // (RW waves have the same columns: each loads its part of their NB * KP pieces of 1 KB)
    constexpr int LOADS = (NB * KP + RW - 1) / RW;
    Piece raw[LOADS];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        int n = n0 + j * 32 + frow;
        n = n < g.N ? n : g.N - 1;
        p_bias[j] = bias_or_any[n], p_mult[j] = g.mult[n], p_shift[j] = g.shift[n];
        p_zw[j] = ZW ? g.zw[n] : 0;
    }
    const int pitch_b = (int)(g.ldb >> (INT4 ? 1 : 0)); // bytes (the dispatcher guarantees that those of 128 rows fit 31 bits)
    const uint32_t weight_off = lane % CPR * 16 < g.K ? (uint32_t)(lane / CPR * pitch_b + lane % CPR * PB) : NOWHERE;
    auto load_of = [&](int l) { return l * RW + (RW > 1 ? wr : 0); }; // piece load `l` of this wave: 64 / CPR columns
    const int columns = g.N - n0 < 32 * NB ? g.N - n0 : 32 * NB; // those beyond N read as zero
    const uint8_t *const b_base = g.B + (int64_t)n0 * pitch_b;
#pragma unroll
    for (int l = 0; l < LOADS; ++l) {
        const uint32_t offset = weight_off + (uint32_t)(load_of(l) * (64 / CPR) * pitch_b);
        if constexpr (INT4) raw[l] = buffer_load8(b_base, columns * pitch_b, offset);
        else raw[l] = buffer_load16(b_base, columns * pitch_b, offset);
    }
    // With no more steps than blocks all rows are requested here and nothing later.  (The forms with the add keep issuing requests
    // past the end: behind a branch the compiler could not count what is younger than the residual.)
    constexpr int AHEAD = G::kAhead, FIRST = DEPTH - AHEAD; // FIRST: block of step 0
    const bool few = !ADD && steps <= DEPTH;
#pragma unroll
    for (int st = 0; st < AHEAD; ++st)
        if (!few || st < steps) request(st, FIRST + st);

    i32x4 fb[KS][NB];
    // where a piece's lane goes, and where a fragment is: column c of a block of 32, chunk p
    auto place_of = [&](int c, int p) { return (c * CPR + ring_place<CPR>(c, p)) * PB; };
    auto fragment = [&](const uint8_t *block, int ks) {
        const Piece v = *reinterpret_cast<const Piece *>(block + place_of(frow, 2 * ks + fhalf));
        if constexpr (INT4) return expand_int4(v);
        else return __builtin_bit_cast(i32x4, v);
    };
    constexpr int COLUMNS_BYTES = 32 * CPR * PB;
    if constexpr (RW > 1) {
        uint8_t *const exchange = (use_pairs ? pair_tab : ring) + wc * NB * COLUMNS_BYTES;
#pragma unroll
        for (int l = 0; l < LOADS; ++l) {
            const int c = load_of(l) * (64 / CPR) + lane / CPR;
            if (NB * KP % RW == 0 || load_of(l) < NB * KP) *reinterpret_cast<Piece *>(exchange + (c >> 5) * COLUMNS_BYTES + place_of(c & 31, lane % CPR)) = raw[l];
        }
        lds_barrier();
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) fb[ks][j] = fragment(exchange + j * COLUMNS_BYTES, ks);
    } else {
        static_assert(!use_pairs || WAVES * G::kBlock <= G::kTables, "the place of the pair table");
        uint8_t *const exchange = (use_pairs ? pair_tab : ring) + wave * G::kBlock; // one block of 32 columns after the other
#pragma unroll
        for (int j = 0; j < NB; ++j) {
#pragma unroll
            for (int i = 0; i < KP; ++i)
                *reinterpret_cast<Piece *>(exchange + place_of(i * (64 / CPR) + lane / CPR, lane % CPR)) = raw[j * KP + i];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) fb[ks][j] = fragment(exchange, ks);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
    ShortKColumn col[NB];
    bool range_ok = g.small_acc >= 2, fused_ok = true;
    const bool ties = rescale_ties(g.lo_rel);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        int32_t colsum = 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int d = 0; d < 4; ++d) colsum = __builtin_amdgcn_sdot4(fb[ks][j][d], 0x01010101, colsum, false);
        }
        colsum += __shfl_xor(colsum, 32);
        if (INT4) colsum >>= 4; // weights are kept times 16; exact
        const int32_t b = g.bias ? p_bias[j] : 0;
        shortk_column(col[j], g, colsum, b, p_mult[j], p_shift[j], p_zw[j], g.K); // (the sums of ZW run over K)
        range_ok = range_ok && rescale_in_range(p_shift[j]) && b > -(1 << 27) && b < (1 << 27);
        fused_ok = fused_ok && range_ok && channel_rescale_ok(p_mult[j], p_shift[j], ties);
    }
    const bool fused = __all(fused_ok), in_range = __all(range_ok), k_tail = g.K != KS * 32;
    const i32x4 ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    if constexpr (ADD) {
        lds_barrier(); // the exchange is over
        add_fill_tables(tab, g.add, threadIdx.x, WAVES * 64);
        lds_barrier();
        if constexpr (use_pairs) {
            fill_pair_table<WAVES>(pair_tab, tab, g.add);
            lds_barrier();
        }
    } else {
        lds_barrier(); // the exchange area becomes blocks of the ring
    }
    // the blocks of the exchange area; step st is in block (FIRST + st) % DEPTH
#pragma unroll
    for (int st = AHEAD; st < DEPTH; ++st)
        if (!few || st < steps) request(st, st - AHEAD);

    // ---- lane-invariant parts of the LDS and global addresses of the output tile.  Whole 16-byte chunks (`chunks_whole`) leave
    // by buffer stores: offsets that do not change from step to step, and what lies beyond the last row or column is dropped
    // by the bounds of the resource, without a branch, so that the number of requests per step is known to the waits.
    int st_lds[NB], st_row[NB];
    uint32_t st_off[NB], st_roff[NB];
    u32x4 rres[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int idx = i * 64 + lane;
        st_row[i] = idx / (2 * NB);
        const int col0 = n0 + (idx % (2 * NB)) * 16;
        st_lds[i] = st_row[i] * PITCH + (idx % (2 * NB)) * 16;
        st_off[i] = col0 < g.N && active ? (uint32_t)st_row[i] * (uint32_t)g.ldc + (uint32_t)col0 : NOWHERE;
        st_roff[i] = col0 < g.N && active ? (uint32_t)st_row[i] * (uint32_t)g.ldr + (uint32_t)col0 : NOWHERE;
        rres[i] = u32x4{0u, 0u, 0u, 0u};
    }
    // bytes of the rows of block rb (none: -1) that exist
    auto rows_bytes = [&](int64_t pitch, int rb) __attribute__((always_inline)) {
        const int left = rb < 0 ? 0 : (M - rb * 32 < 32 ? M - rb * 32 : 32);
        return left > 0 ? left * (int)pitch : 0;
    };
    const int put_base = (4 * fhalf + (lane & 3)) * PITCH + (frow & ~3);
    const bool chunks_whole = ra.whole && ((g.N & 15) == 0 || n0 + 32 * NB <= g.N);
    const int quad_lane = lane & 3;
    const uint32_t sel1 = (quad_lane & 1) ? 0x03070105u : 0x06020400u;
    const uint32_t sel2 = (quad_lane & 2) ? 0x03020706u : 0x05040100u;
    const int32_t lo_rel = g.lo_rel, hi_rel = g.hi_rel, z_out = g.z_out;
    auto load_res = [&](int rb) __attribute__((always_inline)) { // residual chunks of a row block: lanes and rows of its stores
        const uint8_t *const r_block = g.R + (int64_t)rb * 32 * g.ldr;
        const int bytes = rows_bytes(g.ldr, rb);
#pragma unroll
        for (int i = 0; i < NB; ++i) rres[i] = buffer_load16(r_block, bytes, st_roff[i]);
    };
    const AddOut ao = make_add_out(g.add);
    auto tile_fence = [] { // the tile is private to the wave and LDS operations of one wave complete in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // output tile of row block rb (none: -1), from the wave's LDS area to global memory, one step late (non-temporal: see
    // store_block of shortk.h)
    auto store_block = [&](int rb) __attribute__((always_inline)) {
        tile_fence();
        uint8_t *const c_block = g.C + (int64_t)(rb < 0 ? 0 : rb) * 32 * g.ldc;
        if (ADD || chunks_whole) { // (the launcher uses ADD only when every output chunk is a whole, aligned 16-byte chunk)
            const int bytes = rows_bytes(g.ldc, rb);
            auto chunk = [&](int i) { return *reinterpret_cast<const u32x4 *>(stage + st_lds[i]); };
            if constexpr (ADD) {
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    buffer_store16<false>(c_block, bytes, st_off[i], add_chunk<ADD>(chunk(i), rres[i], pair_tab, tab, ao));
                    __builtin_amdgcn_sched_barrier(0); // one chunk at a time: the table reads of all chunks at once would spill
                }
            } else if (s.stream_out) {
#pragma unroll
                for (int i = 0; i < NB; ++i) buffer_store16<true>(c_block, bytes, st_off[i], chunk(i));
            } else {
#pragma unroll
                for (int i = 0; i < NB; ++i) buffer_store16<false>(c_block, bytes, st_off[i], chunk(i));
            }
        } else if (rb >= 0) {
#pragma nounroll
            for (int i = 0; i < NB; ++i) {
                const int idx = i * 64 + lane;
                const int row = idx / (2 * NB), ch = idx % (2 * NB);
                const int n = n0 + ch * 16;
                if (rb * 32 + row >= M || n >= g.N || !active) continue;
                uint8_t *dst = c_block + (int64_t)row * g.ldc + n;
                const uint8_t *src = stage + row * PITCH + ch * 16;
#pragma nounroll
                for (int e = 0; e < 16 && n + e < g.N; ++e) dst[e] = src[e];
            }
        }
        tile_fence();
    };

    // ---- the steps.  Requests retire in order, so a block has landed when at most what was requested after it is outstanding:
    // the DEPTH - 2 blocks behind it and, where their number is known, the stores and residual chunks of the steps since, which
    // are those of DEPTH - 1 steps once the block is none of the set-up's.
    constexpr int MOVES = ADD ? 2 * NB : NB; // per step, besides PIECES
    constexpr int YOUNGER = (DEPTH - 2) * PIECES;
    static_assert(G::kFits && YOUNGER + PIECES + (DEPTH - 1) * MOVES < 64, "see RingGeometry");
    const bool counted = ADD || chunks_whole;
    auto walk = [&](auto mode_tag) {
        using Mode = RescaleModeTraits<decltype(mode_tag)::value>;
        i32x4 fa[KS];
        int at = FIRST, rb_stored = -1;
        if (few) wait_requests_at_most((steps - 1) * PIECES);
        else wait_requests<YOUNGER + PIECES>(); // step 0: DEPTH - 1 blocks behind it
        if constexpr (CW > 1) block_barrier();
        read_rows(at, fa);
        for (int st = 0; st < steps; ++st) {
            const int rb = (walker + st * s.walkers) * RW + wr;
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
                }
                // in registers from here on: the LDS read is over before the barrier below, behind which its block is refilled
                asm volatile("" : "+v"(xs));
                if constexpr (ZW) {
                    sums = __builtin_amdgcn_mfma_i32_32x32x32_i8(xs, ones, sums, 0, 0, 0);
                }
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xs, fb[ks][j], acc[j], 0, 0, 0); // columns past N: zeros, never stored
            }
            // Every wave has this step's fragments in registers (read one step ago): its block is free after the barrier.  Without
            // a branch for the last step, whose next one is a constant chunk: the compiler counts requests too.
            const int next = at + 1 < DEPTH ? at + 1 : 0;
            if (few) {
                if (st + 1 < steps) {
                    wait_requests_at_most((steps - 2 - st) * PIECES + (counted ? st * MOVES : 0));
                    if constexpr (CW > 1) block_barrier();
                    read_rows(next, fa);
                }
            } else {
                if (counted) wait_requests_of_step<YOUNGER, MOVES, DEPTH - 1>(st);
                else wait_requests<YOUNGER>();
                if constexpr (CW > 1) block_barrier();
                read_rows(next, fa);
                asm volatile("" ::: "memory");
                request(st + DEPTH, at);
            }
            at = next;
            store_block(rb_stored);
            if constexpr (ADD) load_res(rb); // used one step from now, when this block is stored
            auto put = [&](int j, int q, uint32_t x) { // 4x4 byte transposition inside each quad of lanes, see shortk.h
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
            tile_fence();
            rb_stored = rb;
        }
        store_block(rb_stored);
    };
    with_rescale_mode(fused, z_out, lo_rel, hi_rel, walk);
    // no copy into this workgroup's LDS may outlive it: the last stores alone are younger
    if (!few) {
        if (counted) wait_requests<NB>();
        else wait_requests<0>();
    }
}

} // namespace qnn
