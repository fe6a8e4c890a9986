// Depthwise convolution (one kh x kw kernel per channel), NHWC uint8 -> NHWC uint8.
//
// 18 integer operations per output byte: the kernel is bound by HBM traffic and by the
// vector ALU, not by the matrix cores, so it does not use MFMA.  Channels are the
// contiguous axis: one lane owns 4 consecutive channels (one dword of activations, one
// dword of weights per tap) and a small patch of output pixels, so that the input window is
// loaded and unpacked once and reused by every output of the patch; consecutive lanes own
// consecutive channel groups, which makes every load and store of a wave a contiguous run
// of channels.
//
//   acc[c] = sum_{a,b} (x[hi][wi][c] - z_x) * w[a][b][c]    taps outside the image skipped
//   out    = clamp(z_out + RESCALE(acc + bias[c]; mult[c], shift[c]))            (eq. 4-6, z_w = 0)
#include <cstdlib>
#include <type_traits>

#include "qnn_device.h"
#include "tuning.h"

namespace qnn {

struct DwArgs {
    const uint8_t *x;
    const int8_t *w;
    uint8_t *y;
    const int32_t *bias, *mult, *shift;
    const int32_t *zw; // per-channel weight zero-points, or nullptr
    int N, H, W, C, Ho, Wo, kh, kw, sh, sw, ph, pw;
    int32_t z_x, z_out, lo_rel, hi_rel;
    int64_t total_work; // lanes of work
    int wruns, hruns;   // patches of RW x RH output pixels per image row / column
    uint32_t magic_cgroups, shift_cgroups; // x / (C/4) = umulhi(x, magic) >> shift for x < 2^31
    int xcd_remap;      // renumber the workgroups (see xcd_neighbours)
};

// The hardware deals workgroups to the 8 XCDs (each with a private L2) round-robin by linear
// id, so spatial neighbours -- which re-read each other's halo rows and columns -- end up behind
// eight different L2s and every halo byte is fetched from the fabric twice.  This renumbering
// gives XCD k the k-th contiguous eighth of the (x fastest, then y, then z) order instead:
// workgroup lin runs on XCD lin % 8 as its (lin / 8)-th, and takes the place
// k * (total / 8) + min(k, total % 8) + lin / 8, a bijection of 0 .. total - 1.
__device__ __forceinline__ void xcd_neighbours(bool on, uint32_t &bx, uint32_t &by, uint32_t &bz)
{
    bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
    if (!on) return;
    const uint32_t gx = gridDim.x, gy = gridDim.y;
    const uint32_t total = gx * gy * gridDim.z; // the dispatcher keeps this below 2^31
    const uint32_t lin = bx + gx * (by + gy * bz);
    const uint32_t xcd = lin & 7u, per = total >> 3, rem = total & 7u;
    const uint32_t id = xcd * per + (xcd < rem ? xcd : rem) + (lin >> 3);
    const uint32_t t = id / gx;
    bx = id - t * gx;
    bz = t / gy;
    by = t - bz * gy;
}

__device__ __forceinline__ int32_t sbyte(uint32_t v, int j) { return (int32_t)(int8_t)(v >> (8 * j)); }
__device__ __forceinline__ int32_t ubyte(uint32_t v, int j) { return (int32_t)((v >> (8 * j)) & 0xffu); }

// One output as the definition has it, for any kernel size, stride, channel and weight zero-point (sums modulo 2^32).
__device__ __forceinline__ uint8_t dw_direct(const DwArgs &g, int n, int ho, int wo, int c)
{
    uint32_t acc = g.bias ? (uint32_t)g.bias[c] : 0u;
    const uint32_t zw = g.zw ? (uint32_t)g.zw[c] : 0u;
    for (int a = 0; a < g.kh; ++a) {
        const int hi = ho * g.sh - g.ph + a;
        if (hi < 0 || hi >= g.H) continue;
        for (int b = 0; b < g.kw; ++b) {
            const int wi = wo * g.sw - g.pw + b;
            if (wi < 0 || wi >= g.W) continue;
            const uint32_t xv = (uint32_t)((int32_t)g.x[(((int64_t)n * g.H + hi) * g.W + wi) * g.C + c] - g.z_x);
            acc += xv * ((uint32_t)(int32_t)g.w[((int64_t)a * g.kw + b) * g.C + c] - zw); // eq. 4 taken literally
        }
    }
    const RescaleParams rp = make_rescale(g.mult[c], g.shift[c]);
    return (uint8_t)(clamp_i32(g.lo_rel, g.hi_rel, rescale_general((int32_t)acc, rp)) + g.z_out);
}

// The 3x3 kernels take weight zero-points of a signed byte (what int8 weights have).  The values live on the device,
// so the kernels look themselves: outputs of channels with any other value are formed one by one, as defined.
__device__ __forceinline__ bool dw_zero_point_is_byte(int32_t zw) { return zw >= -128 && zw <= 127; }

// outputs ho0 .. ho1 - 1 x wo0 .. wo1 - 1 (step `step`) x c0 .. c1 - 1, cut at the output's edges
__device__ __forceinline__ void dw_direct_block(const DwArgs &g, int n, int ho0, int ho1, int wo0, int wo1, int step, int c0, int c1)
{
#pragma nounroll
    for (int ho = ho0; ho < ho1 && ho < g.Ho; ++ho)
#pragma nounroll
        for (int wo = wo0; wo < wo1 && wo < g.Wo; wo += step)
#pragma nounroll
            for (int c = c0; c < c1; ++c) g.y[(((int64_t)n * g.Ho + ho) * g.Wo + wo) * g.C + c] = dw_direct(g, n, ho, wo, c);
}

// One dword of the output.  NT: non-temporal.  What is left in the L2s is written back when the kernel ends, 10-15 % of a
// 12 us launch; but a cache line that several waves fill piece by piece goes out in pieces once much else passes
// through the caches (see dw_stream_out).
template <bool NT> __device__ __forceinline__ void dw_store(uint8_t *p, uint32_t v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<uint32_t *>(p));
    else *reinterpret_cast<uint32_t *>(p) = v;
}

// 3x3 kernel, stride S (same in h and w).  One lane owns 4 consecutive channels and an
// RH x RW patch of output pixels; the ((RH-1)S+3) x ((RW-1)S+3) input window is loaded once
// (one dword = 4 channels per pixel), each byte is unpacked once and multiplied into every
// output of the patch that uses it.  The accumulators start at bias - z_x * sum(w) and taps
// outside the image read as the code z_x, which is the expansion of eq. 5-6 (z_w = 0) with
// the border padded by the code of real zero.
template <int S, int RH, int RW>
__global__ void __launch_bounds__(256) dwconv3x3_kernel(const DwArgs g)
{
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= g.total_work) return;
    const int cgroups = g.C >> 2;
    const int cg = (int)(gid % cgroups);
    int64_t t = gid / cgroups;
    const int pw = (int)(t % g.wruns);
    t /= g.wruns;
    const int ph = (int)(t % g.hruns);
    const int n = (int)(t / g.hruns);
    const int c0 = cg * 4;
    const int ho0 = ph * RH, wo0 = pw * RW;

    // weights as sign-extended ints (less their zero-point), and their per-channel sums
    int32_t wt[3][3][4];
    int32_t wsum[4] = {0, 0, 0, 0}, zw[4] = {0, 0, 0, 0};
    if (g.zw) {
        bool byte = true;
#pragma unroll
        for (int j = 0; j < 4; ++j) zw[j] = g.zw[c0 + j], byte = byte && dw_zero_point_is_byte(zw[j]);
        if (!byte) return dw_direct_block(g, n, ho0, ho0 + RH, wo0, wo0 + RW, 1, c0, c0 + 4);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const uint32_t wv = *reinterpret_cast<const uint32_t *>(g.w + ((int64_t)a * 3 + b) * g.C + c0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                wt[a][b][j] = sbyte(wv, j) - zw[j];
                wsum[j] += wt[a][b][j];
            }
        }
    int32_t acc[RH][RW][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int32_t init = (g.bias ? g.bias[c0 + j] : 0) - g.z_x * wsum[j];
#pragma unroll
        for (int r = 0; r < RH; ++r)
#pragma unroll
            for (int p = 0; p < RW; ++p) acc[r][p][j] = init;
    }

    constexpr int ROWS = (RH - 1) * S + 3, COLS = (RW - 1) * S + 3;
    const int hi0 = ho0 * S - g.ph, wi0 = wo0 * S - g.pw;
    const uint8_t *img = g.x + (int64_t)n * g.H * g.W * g.C + c0;
    const uint32_t fill = (uint32_t)g.z_x * 0x01010101u;
#pragma unroll
    for (int row = 0; row < ROWS; ++row) {
        const int hi = hi0 + row;
        const bool row_ok = hi >= 0 && hi < g.H;
        const uint8_t *line = img + (int64_t)hi * g.W * g.C;
        uint32_t v[COLS];
#pragma unroll
        for (int col = 0; col < COLS; ++col) {
            const int wi = wi0 + col;
            v[col] = fill;
            if (row_ok && wi >= 0 && wi < g.W) v[col] = *reinterpret_cast<const uint32_t *>(line + (int64_t)wi * g.C);
        }
#pragma unroll
        for (int col = 0; col < COLS; ++col) {
            int32_t xv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) xv[j] = ubyte(v[col], j);
#pragma unroll
            for (int r = 0; r < RH; ++r) {
                const int a = row - r * S; // kernel row of this input row for output row r
                if (a < 0 || a > 2) continue;
#pragma unroll
                for (int p = 0; p < RW; ++p) {
                    const int b = col - p * S;
                    if (b < 0 || b > 2) continue;
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[r][p][j] += xv[j] * wt[a][b][j];
                }
            }
        }
    }

    RescaleParams rp[4];
    FusedRescale fr[4];
    bool fused_ok = true;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int32_t mu = g.mult[c0 + j], sf = g.shift[c0 + j];
        rp[j] = make_rescale(mu, sf);
        fused_ok = fused_ok && sf >= 1 && sf <= 20;
        fr[j] = make_fused(mu, sf, 0, g.z_out, g.lo_rel + g.z_out, g.hi_rel + g.z_out);
    }
    // |acc| <= |bias| + 2 * 9 * 255 * 255: the fused form needs |acc| < 2^29, i.e. a sane bias
    if (g.bias) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int32_t b = g.bias[c0 + j];
            fused_ok = fused_ok && b > -(1 << 28) && b < (1 << 28);
        }
    }
    const bool fused = __all(fused_ok);
#pragma unroll
    for (int r = 0; r < RH; ++r) {
        if (ho0 + r >= g.Ho) break;
        uint8_t *out = g.y + (((int64_t)n * g.Ho + ho0 + r) * g.Wo + wo0) * g.C + c0;
#pragma unroll
        for (int p = 0; p < RW; ++p) {
            if (wo0 + p >= g.Wo) break;
            uint32_t packed = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                int32_t y;
                if (fused) y = rescale_fused(acc[r][p][j], fr[j]);
                else y = clamp_i32(g.lo_rel, g.hi_rel, rescale_general(acc[r][p][j], rp[j])) + g.z_out;
                packed |= (uint32_t)y << (8 * j);
            }
            *reinterpret_cast<uint32_t *>(out + (int64_t)p * g.C) = packed;
        }
    }
}

// Weight zero-points on 8-bit multipliers.  The effective weight w' = w - z_w needs 9 bits; it is fed as two signed
// bytes, w' = w + (-z_w), of which the second is the same for all taps.  -z_w does not fit for z_w = -128; such a
// channel accumulates -w' = ~w + (-127) instead and its sum changes sign in the rescale's add (|sum| <= 9 * 255 * 255
// fits the 24-bit multiply-add that does both).  So weight zero-points cost one more dot product (or matrix
// instruction) per tap vector and nothing else.  (Only for z_w of a signed byte, see dw_zero_point_is_byte.)
struct DwZeroPoint {
    int32_t common; // the byte shared by all taps
    int32_t flip;   // all ones: taps enter complemented
    int32_t sign;   // of the accumulated sum
};
__device__ __forceinline__ DwZeroPoint dw_zero_point(int32_t zw)
{
    const bool low = zw == -128;
    return {low ? -127 : -zw, low ? -1 : 0, low ? -1 : 1};
}

// Same layer, multiply-accumulates on the 4-way int8 dot product instruction.
//
// In NHWC a dword holds 4 channels of one pixel, but the sum of a depthwise kernel runs over
// pixels of ONE channel.  Each input row of the window is therefore transposed in registers
// (byte permutes) into per-channel dwords of 4 consecutive pixels, x - 128 as signed bytes.
// One kernel row of one channel is the signed byte vector [w0, w1, w2, 0]: its dot product with
// pixels (p, p+1, p+2, p+3) is the row's contribution to output p, and the same vector shifted by
// one byte gives output p+1 from the same dword, so a row of 4 outputs costs 5 (stride 1) or
// 6 (stride 2) instructions per channel and kernel row instead of 12 multiply-adds plus the
// byte unpacking.  acc starts at bias + (128 - z_x) * sum(w); taps outside the image read as
// the code z_x.  One lane: 4 channels x RH x 4 outputs.
//
// Launch: grid.x covers (patch along W, channel group) lanes, grid.y the patches along H, grid.z
// the images, so that the image and the input rows of a workgroup are wave-uniform: row
// addresses and row bounds live in scalar registers, and a lane only keeps the byte offset and
// the in-image flag of its COLS window columns.  Every load is unconditional (from a clamped
// address) followed by a select of the padding code: no branches around memory operations.
// ZW: weight zero-points, see DwZeroPoint.  (One lane per output, as such layers ran before: 17.6 us on
// 16 x 14 x 14 x 512, 7.2 us here; 57 against 14.3 us on 16 x 112 x 112 x 32 with the matrix-unit kernel below.)
template <int S, int RH, bool ZW, bool NT>
__global__ void __launch_bounds__(256) dwconv3x3_dot_kernel(const DwArgs g)
{
    constexpr int RW = 4;
    constexpr int ROWS = (RH - 1) * S + 3, COLS = (RW - 1) * S + 3; // 6 or 9 input pixels per window row
    uint32_t bx, by, bz;
    xcd_neighbours(g.xcd_remap != 0, bx, by, bz);
    const uint32_t lane_x = bx * 256u + threadIdx.x;
    const uint32_t cgroups = (uint32_t)g.C >> 2;
    const uint32_t pw = cgroups == 1 ? lane_x : __umulhi(lane_x, g.magic_cgroups) >> g.shift_cgroups; // lane_x / cgroups
    const uint32_t cg = lane_x - pw * cgroups;
    if (pw >= (uint32_t)g.wruns) return;
    const int n = (int)bz, ph = (int)by; // wave-uniform
    const int c0 = (int)cg * 4;
    const int ho0 = ph * RH, wo0 = (int)pw * RW;

    // ---- Everything that the lane needs from memory is requested before anything is waited for: the window (whole where
    // the registers hold it; the tall patch of stride 2 goes row by row), the weights and the parameters of the
    // rescale.  As a chain of four round trips, weights, bias, window, rescale, a 14 x 14 x 512 layer took 4.3 us on one
    // image, 6.0 on 16 with weight zero-points and 7.6 on 64, now 3.8, 5.5 and 6.4.
    const int hi0 = ho0 * S - g.ph, wi0 = wo0 * S - g.pw;
    const uint8_t *img = g.x + (int64_t)n * g.H * g.W * g.C; // scalar
    const uint32_t fill = (uint32_t)g.z_x * 0x01010101u;
    // byte offset inside an image row and in-image flag of each window column (the dispatcher
    // guarantees W * C < 2^31)
    uint32_t col_off[COLS]; // unsigned: scalar base + 32-bit lane offset addressing
    bool col_ok[COLS];
#pragma unroll
    for (int col = 0; col < COLS; ++col) {
        const int wi = wi0 + col;
        col_ok[col] = wi >= 0 && wi < g.W;
        col_off[col] = (uint32_t)((col_ok[col] ? wi : 0) * g.C + c0);
    }
    constexpr bool AHEAD = ROWS * COLS <= 48;
    uint32_t ahead[AHEAD ? ROWS : 1][COLS];
    auto load_row = [&](int row, uint32_t (&v)[COLS]) __attribute__((always_inline)) {
        const int hi = hi0 + row;                // scalar
        const bool row_ok = hi >= 0 && hi < g.H; // scalar
        const uint8_t *line = img + (int64_t)(row_ok ? hi : 0) * g.W * g.C; // scalar, always inside the image
#pragma unroll
        for (int col = 0; col < COLS; ++col) v[col] = *reinterpret_cast<const uint32_t *>(line + col_off[col]);
    };
    if constexpr (AHEAD) {
#pragma unroll
        for (int row = 0; row < ROWS; ++row) load_row(row, ahead[row]);
    }
    uint32_t w_raw[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) w_raw[a][b] = *reinterpret_cast<const uint32_t *>(g.w + (a * 3 + b) * g.C + c0);
    int32_t mu[4], sf[4], bias[4], zps[4]; // 16 bytes each, from any address of a dword
    __builtin_memcpy(bias, (g.bias ? g.bias : g.mult) + c0, 16); // no branch around the load; the value is dropped below
    __builtin_memcpy(mu, g.mult + c0, 16);
    __builtin_memcpy(sf, g.shift + c0, 16);
    if constexpr (ZW) __builtin_memcpy(zps, g.zw + c0, 16);
    asm volatile("" ::: "memory"); // the loads stay here
#pragma unroll
    for (int j = 0; j < 4; ++j) bias[j] = g.bias ? bias[j] : 0;

    // ---- weights: wa[a][j] = [w(a,0), w(a,1), w(a,2), 0] of channel c0 + j
    uint32_t wa[3][4];
    int32_t wsum[4] = {0, 0, 0, 0};
    uint32_t wc[4];      // ZW: [c, c, c, 0], the byte that the taps share
    int32_t sign[4];     // ZW
    uint32_t flip = 0u;  // ZW: byte j all ones where channel c0 + j enters complemented
    bool zw_bytes = true; // looked at behind the loop: a branch here would wait for the zero-points (2 % of the launch)
    if constexpr (ZW) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int32_t zw = zps[j];
            zw_bytes = zw_bytes && dw_zero_point_is_byte(zw);
            const DwZeroPoint z = dw_zero_point(zw);
            wc[j] = ((uint32_t)z.common & 0xffu) * 0x00010101u;
            sign[j] = z.sign;
            flip |= (uint32_t)z.flip & (0xffu << (8 * j));
            wsum[j] = -9 * zw;
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const uint32_t(&wv)[3] = w_raw[a];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t t01 = __builtin_amdgcn_perm(wv[1], wv[0], 0x0c0c0000u | ((4u + j) << 8) | (uint32_t)j);
            wa[a][j] = __builtin_amdgcn_perm(wv[2], t01, 0x0c000100u | ((4u + j) << 16));
            wsum[j] = __builtin_amdgcn_sdot4((int)wa[a][j], 0x01010101, wsum[j], false);
            if constexpr (ZW) wa[a][j] ^= __builtin_amdgcn_perm(0u, flip, 0x0c000000u | (uint32_t)(0x00010101 * j));
        }
    }
    int32_t acc[RH][RW][4], init[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        init[j] = bias[j] + (128 - g.z_x) * wsum[j];
#pragma unroll
        for (int r = 0; r < RH; ++r)
#pragma unroll
            for (int p = 0; p < RW; ++p) acc[r][p][j] = ZW ? 0 : init[j];
    }

    // 4 pixel dwords (4 channels each) -> 4 channel dwords (4 pixels each)
    auto transpose4 = [](const uint32_t *v, uint32_t (&x)[4]) {
        const uint32_t lo01 = __builtin_amdgcn_perm(v[1], v[0], 0x05010400u), hi01 = __builtin_amdgcn_perm(v[1], v[0], 0x07030602u);
        const uint32_t lo23 = __builtin_amdgcn_perm(v[3], v[2], 0x05010400u), hi23 = __builtin_amdgcn_perm(v[3], v[2], 0x07030602u);
        x[0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
        x[1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
        x[2] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
        x[3] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
    };
    const uint32_t fill_s = fill ^ 0x80808080u;
#pragma unroll
    for (int row = 0; row < ROWS; ++row) {
        const int hi = hi0 + row;                // scalar
        const bool row_ok = hi >= 0 && hi < g.H; // scalar
        uint32_t v[COLS];
        if constexpr (AHEAD) {
#pragma unroll
            for (int col = 0; col < COLS; ++col) v[col] = ahead[row][col];
        } else {
            load_row(row, v);
        }
#pragma unroll
        for (int col = 0; col < COLS; ++col) v[col] = (row_ok && col_ok[col]) ? (v[col] ^ 0x80808080u) : fill_s; // signed (code - 128)
        uint32_t x0[4], x1[4], x2[4] = {0u, 0u, 0u, 0u};
        transpose4(v, x0);
        if constexpr (S == 1) { // pixels 4, 5 -> [p4, p5, 0, 0]
#pragma unroll
            for (int j = 0; j < 4; ++j) x1[j] = __builtin_amdgcn_perm(v[5], v[4], 0x0c0c0000u | ((4u + j) << 8) | (uint32_t)j);
        } else { // pixels 4..7, and pixel 8 alone
            transpose4(v + 4, x1);
#pragma unroll
            for (int j = 0; j < 4; ++j) x2[j] = (v[8] >> (8 * j)) & 0xffu;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // stride 1: pixels (2, 3, 4, 5) as one dword
            const uint32_t y = S == 1 ? __builtin_amdgcn_alignbyte(x1[j], x0[j], 2) : 0u;
#pragma unroll
            for (int r = 0; r < RH; ++r) {
                const int a = row - r * S; // kernel row of this input row for output row r
                if (a < 0 || a > 2) continue;
                auto taps = [&](uint32_t w) __attribute__((always_inline)) {
                if constexpr (S == 1) {
                    acc[r][0][j] = __builtin_amdgcn_sdot4((int)x0[j], (int)w, acc[r][0][j], false);
                    acc[r][1][j] = __builtin_amdgcn_sdot4((int)x0[j], (int)(w << 8), acc[r][1][j], false);
                    acc[r][2][j] = __builtin_amdgcn_sdot4((int)y, (int)w, acc[r][2][j], false);
                    acc[r][3][j] = __builtin_amdgcn_sdot4((int)y, (int)(w << 8), acc[r][3][j], false);
                } else { // output p uses pixels 2p, 2p+1, 2p+2
                    acc[r][0][j] = __builtin_amdgcn_sdot4((int)x0[j], (int)w, acc[r][0][j], false);
                    acc[r][1][j] = __builtin_amdgcn_sdot4((int)x0[j], (int)(w << 16), acc[r][1][j], false);
                    acc[r][1][j] = __builtin_amdgcn_sdot4((int)x1[j], (int)(w >> 16), acc[r][1][j], false);
                    acc[r][2][j] = __builtin_amdgcn_sdot4((int)x1[j], (int)w, acc[r][2][j], false);
                    acc[r][3][j] = __builtin_amdgcn_sdot4((int)x1[j], (int)(w << 16), acc[r][3][j], false);
                    acc[r][3][j] = __builtin_amdgcn_sdot4((int)x2[j], (int)(w >> 16), acc[r][3][j], false);
                }
                };
                taps(wa[a][j]);
                if constexpr (ZW) taps(wc[j]);
            }
        }
    }

    // ---- epilogue: the fused form of the rescale when every channel of the wave allows it, else the general form
    ChannelRescale cr[4];
    const bool ties = rescale_ties(g.lo_rel);
    bool range_ok = true, fused_ok = true;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        range_ok = range_ok && rescale_in_range(sf[j]) && bias[j] > -(1 << 28) && bias[j] < (1 << 28);
        fused_ok = fused_ok && range_ok && channel_rescale_ok(mu[j], sf[j], ties);
        cr[j] = make_channel_rescale(mu[j], sf[j], 0, g.z_out, g.lo_rel + g.z_out, g.hi_rel + g.z_out, ties);
    }
    if constexpr (ZW) {
        if (!zw_bytes) return dw_direct_block(g, n, ho0, ho0 + RH, wo0, wo0 + RW, 1, c0, c0 + 4);
#pragma unroll
        for (int r = 0; r < RH; ++r)
#pragma unroll
            for (int p = 0; p < RW; ++p)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[r][p][j] = __mul24(acc[r][p][j], sign[j]) + init[j];
    }
    const bool fused = __all(fused_ok), in_range = __all(range_ok);
    uint8_t *const out_img = g.y + (int64_t)n * g.Ho * g.Wo * g.C; // scalar
    const uint32_t out_off = (uint32_t)(wo0 * g.C + c0);            // inside an output row (Wo * C < 2^31)
    auto finish = [&](auto mode_tag) {
        using Mode = RescaleModeTraits<decltype(mode_tag)::value>;
#pragma unroll
        for (int r = 0; r < RH; ++r) {
            if (ho0 + r >= g.Ho) break; // scalar
            uint8_t *out = out_img + (int64_t)(ho0 + r) * g.Wo * g.C; // scalar
            // the four pixels of a channel share its shift and are packed together; the 4x4 bytes are transposed then
            uint32_t ch[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int32_t a[4] = {acc[r][0][j], acc[r][1][j], acc[r][2][j], acc[r][3][j]};
                if constexpr (Mode::kFused) ch[j] = channel_codes4<Mode::kTies, Mode::kFull>(a, cr[j]);
                else ch[j] = other_codes4(a, mu[j], sf[j], 0, in_range, g.z_out, g.lo_rel, g.hi_rel);
            }
            const uint32_t lo01 = __builtin_amdgcn_perm(ch[1], ch[0], 0x05010400u), hi01 = __builtin_amdgcn_perm(ch[1], ch[0], 0x07030602u);
            const uint32_t lo23 = __builtin_amdgcn_perm(ch[3], ch[2], 0x05010400u), hi23 = __builtin_amdgcn_perm(ch[3], ch[2], 0x07030602u);
            const uint32_t pixel[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100u), __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                                       __builtin_amdgcn_perm(hi23, hi01, 0x05040100u), __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
#pragma unroll
            for (int p = 0; p < RW; ++p)
                if (wo0 + p < g.Wo) dw_store<NT>(out + (out_off + (uint32_t)(p * g.C)), pixel[p]);
        }
    };
    static_assert(RW == 4, "four pixels of a channel are packed together");
    // (the code of the rare form behind the others: in front of them one-image layers took 0.07 us longer each)
    if (__builtin_expect(!fused, 0)) finish(RescaleTag<RESCALE_GENERAL>{});
    else with_rescale_mode(true, g.z_out, g.lo_rel, g.hi_rel, finish);
}

// Depthwise 3x3 with the multiplies on the matrix unit.
//
// The layer moves 2-5 bytes per output, and on the vector ALU it costs about 16 instructions per
// output byte (the dot products need pixels in the bytes of a dword while NHWC puts channels there,
// so every input byte goes through byte permutes first): the vector ALU, not HBM, sets the pace.
// v_mfma_i32_32x32x32_i8 takes the transposition away.  For a block of 32 channels and one kernel tap,
//   D[pixel][c] += sum_c' A[pixel][c'] * B[c'][c],   B[c'][c] = w[tap][c] if c' == c else 0
// is that tap's contribution to 32 pixels x 32 channels.  A's fragment is what NHWC memory holds:
// lane (pixel, half) takes the 16 contiguous channel bytes of its pixel -- no byte shuffling at all;
// B's fragment is a diagonal matrix built once per wave from the weights.  The unit runs at 1/32
// of its density and that is fine: nine of these instructions per output row of a wave take fewer
// issue cycles than the rescale of the same outputs, and they run beside it.  The layer stays
// HBM-bound and is graded against HBM; the matrix unit only replaces the byte transposition.
//
// A wave owns TP = 30 output pixels of one image row x 32 channels and walks down a segment of output
// rows.  Its input rows -- 32 pixels (stride 1) or 64 pixels (stride 2) x 32 channel bytes, one or
// two 1 KB copies -- go straight from global memory into a ring of LDS rows that belongs to the wave
// alone (global_load_lds_dwordx4, RING - 1 rows ahead of the row in use; no barrier anywhere: waves
// share nothing).  A row is read back three times as fragments (window columns 0, 1, 2 = the same
// pixels shifted by one); it is kernel row 0, 1 and 2 of three consecutive output rows (stride 1;
// stride 2: two rows per output row, the odd one shared), whose accumulators form a ring of their
// own.  An output row that has received its last kernel row is rescaled (all 16 values of a lane
// belong to ONE channel, so the constants are per lane), its bytes are transposed across the four
// lanes of a quad into NHWC order and stored.  acc starts at bias + (128 - z_x) * sum(w); codes are
// offset by 128 (xor) to be signed; taps outside the image hold the code z_x.
//
// vmcnt bookkeeping: every wave issues exactly DPW copies per input row, rows
// past the end of the segment repeat the last one, "at most (RING - 2) x DPW outstanding" means
// the oldest row has landed, and the output stores can only make that wait stricter.
// (Measured: a wait that also allows for the stores issued since -- possible in the steady state, where their
// number is known -- and even no wait at all leave the time of a launch unchanged.)
using dw_i32x4 = int32_t __attribute__((ext_vector_type(4)));
using dw_i32x16 = int32_t __attribute__((ext_vector_type(16)));

template <int S, int MODE, bool ZW, bool NT> // ZW: weight zero-points, see DwZeroPoint; NT: see dw_store
__global__ void __launch_bounds__(256, 2) dwconv3x3_mfma_kernel(const DwArgs g, const int seg_rows, const int tiles_w,
                                                                const int cblocks)
{
    constexpr int SLOTS = S == 1 ? 3 : 2, TP = 30, DPW = S, ROW_BYTES = DPW * 1024, RING = S == 1 ? 12 : 8, D = RING - 1;
    __shared__ __attribute__((aligned(16))) uint8_t lds[4 * RING * ROW_BYTES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t bx, by, bz;
    xcd_neighbours(g.xcd_remap != 0, bx, by, bz);
    const int wave_lin = (int)bx * 4 + wave; // scalar
    const int tile_w = wave_lin / cblocks, cblk = wave_lin - tile_w * cblocks;
    if (tile_w >= tiles_w) return; // whole wave; waves share nothing
    uint8_t *const ring = lds + wave * (RING * ROW_BYTES);
    const int n = (int)bz;
    const int hb = (int)by * seg_rows;
    const int rows = (g.Ho - hb) < seg_rows ? (g.Ho - hb) : seg_rows;
    const int li = lane & 31, half = lane >> 5;
    const int w0 = tile_w * TP;

    // ---- input rows: copy j of a row moves, per lane, 16 channel bytes of pixel wi0 + (j * 64 + lane) / 2
    // (clamped into the image row; pixels outside are replaced after the read-back) to LDS offset
    // (j * 64 + lane) * 16, i.e. an LDS row is [pixel][32 channel bytes]
    const int wi0 = w0 * S - g.pw;
    const int64_t row_bytes = (int64_t)g.W * g.C;
    const uint8_t *img = g.x + (int64_t)n * g.H * row_bytes;    // scalar
    uint32_t src_off[DPW];
#pragma unroll
    for (int j = 0; j < DPW; ++j) {
        int wi = wi0 + ((j * 64 + lane) >> 1);
        wi = wi < 0 ? 0 : (wi >= g.W ? g.W - 1 : wi);
        int c16 = cblk * 32 + 16 * (lane & 1);
        c16 = c16 + 16 <= g.C ? c16 : g.C - 16; // blocks that stick out of C: any valid bytes (B is zero there)
        src_off[j] = (uint32_t)(wi * g.C + c16);
    }
    // ---- the row pipeline: input row t of the segment is image row hi_first + t, t = 0 .. steps - 1
    const int hi_first = hb * S - g.ph;
    const int steps = S == 1 ? rows + 2 : 2 * rows + 1;
    int issue_t = 0, issue_slot = 0; // next row to copy and the ring row it goes to (scalar)
    int read_t = 0, read_slot = 0;   // next row to consume
    auto issue_row = [&]() __attribute__((always_inline)) {
        const int t = issue_t < steps ? issue_t : steps - 1; // past the end: repeat the last row (nobody reads that ring row)
        int hi = hi_first + t;
        hi = hi < 0 ? 0 : (hi >= g.H ? g.H - 1 : hi);        // rows outside the image: any row inside (replaced by the padding code)
        const uint8_t *line = img + (int64_t)hi * row_bytes;
        uint8_t *dst = ring + issue_slot * ROW_BYTES;
#pragma unroll
        for (int j = 0; j < DPW; ++j)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(line + src_off[j]),
                                             (__attribute__((address_space(3))) void *)(dst + j * 1024), 16, 0, 0);
        ++issue_t;
        issue_slot = issue_slot + 1 == RING ? 0 : issue_slot + 1;
    };
    for (int d = 0; d < D; ++d) issue_row(); // D rows in flight before anything else: their latency covers the set-up below

    // ---- B fragments: the diagonal of tap (a, b) for the channels of this block.  Lane (column li, half)
    // holds rows k = 16 half .. 16 half + 15 of column li: only row k = li is non-zero.
    const int ch = cblk * 32 + li;                  // the channel this lane accumulates and rescales
    const bool ch_ok = ch < g.C;
    const bool diag_here = ch_ok && (li >> 4) == half;
    auto diagonal = [&](int32_t w) { // the byte w of this lane's channel in its place
        const uint32_t placed = diag_here ? ((uint32_t)(w & 0xff) << (8 * (li & 3))) : 0u;
        const int d = (li >> 2) & 3;
        return dw_i32x4{d == 0 ? (int32_t)placed : 0, d == 1 ? (int32_t)placed : 0, d == 2 ? (int32_t)placed : 0,
                        d == 3 ? (int32_t)placed : 0};
    };
    dw_i32x4 wq[3][3], wc = {0, 0, 0, 0};
    int32_t wsum = 0;
    DwZeroPoint zp = {0, 0, 1};
    bool zw_bytes = true;
    if constexpr (ZW) {
        const int32_t zw = ch_ok ? g.zw[ch] : 0;
        zw_bytes = dw_zero_point_is_byte(zw);
        zp = dw_zero_point(zw);
        wsum = -9 * zw;
        wc = diagonal(zp.common);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const int32_t w = ch_ok ? (int32_t)g.w[(a * 3 + b) * g.C + ch] : 0;
            wsum += w;
            wq[a][b] = diagonal(w ^ zp.flip);
        }
    const int32_t bias = (ch_ok && g.bias) ? g.bias[ch] : 0;
    const int32_t init = bias + (128 - g.z_x) * wsum;

    // ---- epilogue constants of this lane's channel
    using Mode = RescaleModeTraits<MODE>;
    const int32_t mu = ch_ok ? g.mult[ch] : 1 << 30, sf = ch_ok ? g.shift[ch] : 1;
    const bool range_ok = rescale_in_range(sf) && bias > -(1 << 28) && bias < (1 << 28);
    const ChannelRescale cr = make_channel_rescale(mu, sf, init, g.z_out, g.lo_rel + g.z_out, g.hi_rel + g.z_out, Mode::kTies);
    const bool in_range = __all(range_ok), fused = __all(range_ok && channel_rescale_ok(mu, sf, Mode::kTies)); // wave-uniform
    if (ZW && !__all(zw_bytes)) { // the whole wave: its lanes share the matrix instructions
        dw_direct_block(g, n, hb, hb + rows, w0 + half, w0 + TP, 2, ch, ch_ok ? ch + 1 : ch);
        __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8)); // vmcnt(0): no copy may land in LDS after the wave is gone
        return;
    }

    // read-back of window column b: pixel li * S + b of the LDS row, 16 channel bytes of this lane's half
    uint32_t l_off[3];
    bool a_ok[3], all_ok = true;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const int wi = wi0 + li * S + b;
        a_ok[b] = wi >= 0 && wi < g.W;
        all_ok = all_ok && a_ok[b];
        const int lp = li < TP ? li : TP - 1; // lanes 30, 31 own no output pixel: they re-read the last one, inside the row
        l_off[b] = (uint32_t)((lp * S + b) * 32 + 16 * half);
    }
    const bool wave_interior = __all(all_ok);
    const int32_t fill_s = (int32_t)(((uint32_t)g.z_x * 0x01010101u) ^ 0x80808080u);

    // ---- output addressing: after the quad transposition lane (li, half) stores, for q = 0..3, the 4 channels
    // (li & ~3) .. + 3 of pixel w0 + 8q + 4 half + (li & 3)
    const int quad_lane = li & 3;
    const uint32_t sel1 = (quad_lane & 1) ? 0x03070105u : 0x06020400u;
    const uint32_t sel2 = (quad_lane & 2) ? 0x03020706u : 0x05040100u;
    const int64_t out_row_bytes = (int64_t)g.Wo * g.C;
    int64_t out_row = ((int64_t)n * g.Ho + hb) * out_row_bytes; // scalar: byte offset of the output row that finishes next
    const int out_c = cblk * 32 + (li & ~3);
    uint32_t o_off[4];
    bool o_ok[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int p = 8 * q + 4 * half + quad_lane; // pixel of the tile
        const int wo = w0 + p;
        o_ok[q] = p < TP && wo < g.Wo && out_c < g.C;
        o_off[q] = (uint32_t)((o_ok[q] ? wo : 0) * g.C + (out_c < g.C ? out_c : 0));
    }

    // accumulators start at zero (an inline constant of the matrix instruction); bias and zero-point term join in
    // the addend of the rescale
    dw_i32x16 acc[SLOTS];
    auto reset = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[slot][r] = 0;
    };
    auto finish = [&](int slot) __attribute__((always_inline)) {
        // wave-uniform row base (scalar registers) + 32-bit lane offsets
        auto signed_sum = [&](int32_t a) { return ZW ? __mul24(a, zp.sign) : a; };
        const int64_t row_off = ((int64_t)__builtin_amdgcn_readfirstlane((int)(out_row >> 32)) << 32) |
                                (uint32_t)__builtin_amdgcn_readfirstlane((int)out_row);
        uint8_t *out = g.y + row_off;
        uint32_t x[4];
        if (fused) { // one test per output row; the forms below are the rare case
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                int32_t a[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = signed_sum(acc[slot][4 * q + e]);
                x[q] = channel_codes4<Mode::kTies, Mode::kFull>(a, cr);
            }
        } else if (in_range) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                int32_t a[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = signed_sum(acc[slot][4 * q + e]);
                x[q] = other_codes4(a, mu, sf, init, true, g.z_out, g.lo_rel, g.hi_rel);
            }
        } else {
#pragma nounroll
            for (int q = 0; q < 4; ++q) {
                int32_t a[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = signed_sum(acc[slot][4 * q + e]);
                x[q] = other_codes4(a, mu, sf, init, false, g.z_out, g.lo_rel, g.hi_rel);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            // 4 pixels of one channel -> 4 channels of one pixel, across the quad (two exchanges + byte permutes)
            uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)x[q], 0xB1, 0xF, 0xF, true);
            uint32_t v = __builtin_amdgcn_perm(o, x[q], sel1);
            o = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);
            v = __builtin_amdgcn_perm(o, v, sel2);
            if (o_ok[q]) dw_store<NT>(out + o_off[q], v);
        }
        out_row += out_row_bytes;
    };

    dw_i32x4 fa[3], fn[3];
    // requests the LDS read-back of input row read_t into fn (after its copy has landed) and the copy of row read_t + D
    auto fetch_row = [&]() __attribute__((always_inline)) {
        constexpr int N = (D - 1) * DPW;
        __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8)); // vmcnt only
        asm volatile("" ::: "memory");
        const uint8_t *src = ring + read_slot * ROW_BYTES;
#pragma unroll
        for (int b = 0; b < 3; ++b) fn[b] = *reinterpret_cast<const dw_i32x4 *>(src + l_off[b]);
        asm volatile("" ::: "memory");
        issue_row(); // into the ring row that was consumed one step ago
    };
    // fn (raw codes of row read_t) -> fa (signed, padding replaced)
    auto take_row = [&]() __attribute__((always_inline)) {
        const int hi = hi_first + read_t;
        const bool row_ok = hi >= 0 && hi < g.H; // scalar
        if (!row_ok) {
#pragma unroll
            for (int b = 0; b < 3; ++b) fa[b] = dw_i32x4{fill_s, fill_s, fill_s, fill_s};
        } else if (wave_interior) { // the common case: twelve xors
#pragma unroll
            for (int b = 0; b < 3; ++b) fa[b] = fn[b] ^ (int32_t)0x80808080; // signed (code - 128)
        } else {
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const dw_i32x4 t = fn[b] ^ (int32_t)0x80808080;
                const bool ok = a_ok[b];
                fa[b] = dw_i32x4{ok ? t.x : fill_s, ok ? t.y : fill_s, ok ? t.z : fill_s, ok ? t.w : fill_s};
            }
        }
        ++read_t;
        read_slot = read_slot + 1 == RING ? 0 : read_slot + 1;
    };
    // one window column of the current row into one accumulator set (the caller interleaves the sets, so that
    // consecutive matrix instructions do not depend on each other)
    auto mac1 = [&](int a, int b, int slot) __attribute__((always_inline)) {
        acc[slot] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[b], wq[a][b], acc[slot], 0, 0, 0);
        if constexpr (ZW) acc[slot] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[b], wc, acc[slot], 0, 0, 0);
    };

    // Steady state of the row pipeline, free of run-time conditions: every output row involved exists and every
    // input row lies inside the image, so a step is LDS read-back, sign flip (EDGE: plus the padding selects of
    // the window columns that stick out of the image), nine matrix instructions -- the first one of a new output
    // row takes the constant zero as its accumulator input, which replaces the reset -- and one rescale.
    const dw_i32x16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    auto take_inside = [&](auto edge) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const dw_i32x4 t = fn[b] ^ (int32_t)0x80808080;
            if constexpr (decltype(edge)::value) {
                const bool ok = a_ok[b];
                fa[b] = dw_i32x4{ok ? t.x : fill_s, ok ? t.y : fill_s, ok ? t.z : fill_s, ok ? t.w : fill_s};
            } else {
                fa[b] = t;
            }
        }
        ++read_t;
        read_slot = read_slot + 1 == RING ? 0 : read_slot + 1;
    };
    auto mac0 = [&](int b, int slot) __attribute__((always_inline)) { // kernel row 0: window column 0 opens the accumulator set
        acc[slot] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[b], wq[0][b], b == 0 ? zero16 : acc[slot], 0, 0, 0);
        if constexpr (ZW) acc[slot] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[b], wc, acc[slot], 0, 0, 0);
    };

    if constexpr (S == 1) {
        // row t is kernel row 0 of output k = t, kernel row 1 of k = t - 1, kernel row 2 of k = t - 2; output k lives
        // in accumulator set k % 3
        auto steady3 = [&](auto edge) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                fetch_row();
                take_inside(edge);
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    mac1(2, b, (u + 1) % 3);
                    mac1(1, b, (u + 2) % 3);
                    mac0(b, u);
                }
                finish((u + 1) % 3);
            }
        };
        for (int t0 = 0; t0 < steps; t0 += 3) {
            // rows t0 .. t0 + 2: all three outputs of every step exist and all three input rows are inside the image
            if (t0 >= 2 && t0 + 2 < rows && hi_first + t0 >= 0 && hi_first + t0 + 2 < g.H) { // scalar
                if (wave_interior) steady3(std::false_type{});
                else steady3(std::true_type{});
                continue;
            }
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const int t = t0 + u;
                if (t >= steps) break; // scalar
                fetch_row();
                take_row();
                const bool has0 = t < rows, has1 = t >= 1 && t - 1 < rows, has2 = t >= 2; // scalar
                if (has0) reset(u);
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    if (has2) mac1(2, b, (u + 1) % 3);
                    if (has1) mac1(1, b, (u + 2) % 3);
                    if (has0) mac1(0, b, u);
                }
                if (has2) finish((u + 1) % 3);
            }
        }
    } else {
        // output k uses rows 2k, 2k + 1, 2k + 2 of the segment; row 2k + 2 is also the first row of output k + 1;
        // output k lives in accumulator set k % 2
        fetch_row();
        take_row();
        reset(0);
#pragma unroll
        for (int b = 0; b < 3; ++b) mac1(0, b, 0);
        auto steady2 = [&](auto edge) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                fetch_row();
                take_inside(edge);
#pragma unroll
                for (int b = 0; b < 3; ++b) mac1(1, b, u);
                fetch_row();
                take_inside(edge);
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    mac1(2, b, u);
                    mac0(b, u ^ 1);
                }
                finish(u);
            }
        };
        for (int k0 = 0; k0 < rows; k0 += 2) {
            // outputs k0, k0 + 1 and k0 + 2 exist and input rows 2 k0 + 1 .. 2 k0 + 4 are inside the image
            if (k0 + 2 < rows && hi_first + 2 * k0 + 1 >= 0 && hi_first + 2 * k0 + 4 < g.H) { // scalar
                if (wave_interior) steady2(std::false_type{});
                else steady2(std::true_type{});
                continue;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k = k0 + u;
                if (k >= rows) break; // scalar
                fetch_row();
                take_row();
#pragma unroll
                for (int b = 0; b < 3; ++b) mac1(1, b, u);
                fetch_row();
                take_row();
                const bool more = k + 1 < rows; // scalar
                if (more) reset(u ^ 1);
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    mac1(2, b, u);
                    if (more) mac1(0, b, u ^ 1);
                }
                finish(u);
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8)); // vmcnt(0): no copy may land in LDS after the wave is gone
}

// any kernel size / stride / channel count: one lane per output element
__global__ void __launch_bounds__(256) dwconv_generic_kernel(const DwArgs g)
{
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= g.total_work) return;
    const int c = (int)(gid % g.C);
    int64_t t = gid / g.C;
    const int wo = (int)(t % g.Wo);
    t /= g.Wo;
    const int ho = (int)(t % g.Ho);
    const int n = (int)(t / g.Ho);
    g.y[gid] = dw_direct(g, n, ho, wo, c);
}

} // namespace qnn

using namespace qnn;

// Non-temporal output stores?  A wave of the matrix-unit kernel writes 32 channels of its pixels, one of the patch kernel
// 256: with just as many channels in a pixel (or fewer) it fills whole cache lines, else these stores pay only while
// input and output together are small enough that the other waves' pieces come in time.  Measured, non-temporal over
// plain time, inputs from the cache / from HBM, outputs of 4, 16, 32 and 80 MB:
//   matrix unit, 56x56x32: 0.99/0.94, 0.96/0.93, 0.92/0.95, 0.96/0.93;  112x112x64: 0.99/0.93, 0.93/0.93, 0.93/0.92, 1.04/1.02
//                56x56x128: 0.98/0.93, 0.93/0.93, 1.03/1.04, 1.29/1.27;  112x112x128, stride 2: 0.98/0.98, 1.05/1.05, 1.15/1.16, 1.24/1.28
//   patch, 28x28x256: 0.97/0.92, 0.90/0.90, 0.95/0.91, 0.98/0.95;  28x28x144, stride 2: 0.98/0.97, 1.00/1.01, 1.01/1.04, 1.05/1.05
static bool dw_stream_out(const DwArgs &g, bool matrix_unit)
{
    const int64_t mb = ((int64_t)g.N * g.C * ((int64_t)g.H * g.W + (int64_t)g.Ho * g.Wo)) >> 20;
    if (matrix_unit) return g.C <= 32 || mb < (g.C <= 64 ? 128 : 42);
    return g.C >= 256 || mb < 128;
}

static qnn_status qdwconv2d_impl(const uint8_t *x, int N, int H, int W, int C, int32_t z_x, const int8_t *w, int kh, int kw,
                                 int stride_h, int stride_w, int pad_h, int pad_w, const int32_t *bias, const int32_t *mult,
                                 const int32_t *shift, int32_t z_out, int32_t act_min, int32_t act_max, uint8_t *y,
                                 void *stream, const int32_t *z_w)
{
    if (N < 0 || H <= 0 || W <= 0 || C <= 0 || kh <= 0 || kw <= 0 || kh > 7 || kw > 7) return QNN_EINVAL;
    if (stride_h <= 0 || stride_w <= 0 || pad_h < 0 || pad_w < 0) return QNN_EINVAL;
    if (H + 2 * (int64_t)pad_h < kh || W + 2 * (int64_t)pad_w < kw) return QNN_EINVAL;
    if (z_x < 0 || z_x > 255 || bad_out_range(z_out, act_min, act_max)) return QNN_EINVAL;
    if (N == 0) return QNN_OK; // an empty batch: nothing to compute, no pointer is looked at
    if (!x || !w || !mult || !shift || !y) return QNN_EINVAL;
    DwArgs g = {};
    g.x = x, g.w = w, g.y = y, g.bias = bias, g.mult = mult, g.shift = shift, g.zw = z_w;
    g.N = N, g.H = H, g.W = W, g.C = C, g.kh = kh, g.kw = kw;
    g.sh = stride_h, g.sw = stride_w, g.ph = pad_h, g.pw = pad_w;
    g.Ho = (H + 2 * pad_h - kh) / stride_h + 1;
    g.Wo = (W + 2 * pad_w - kw) / stride_w + 1;
    g.z_x = z_x, g.z_out = z_out, g.lo_rel = act_min - z_out, g.hi_rel = act_max - z_out;
    const hipStream_t s = as_stream(stream);
    auto al4 = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 3) == 0; };
    const bool c4 = (C % 4 == 0) && al4(x) && al4(w) && al4(y) && kh == 3 && kw == 3 && stride_h == stride_w &&
                    (stride_h == 1 || stride_h == 2);
    constexpr int RH = 2, RW = 4;
    if (c4) {
        g.wruns = (g.Wo + RW - 1) / RW;
        g.hruns = (g.Ho + RH - 1) / RH;
        g.total_work = (int64_t)N * g.hruns * g.wruns * (C / 4);
    } else {
        g.total_work = (int64_t)N * g.Ho * g.Wo * C;
    }
    const int64_t blocks = (g.total_work + 255) / 256;
    if (blocks > 0x7fffffff) return QNN_EINVAL;
    const bool old_form = tuning().dw_mad != 0; // tuning aid: the multiply-add form
    const int64_t lanes_x = (int64_t)g.wruns * (C / 4);
    const bool dot_ok = c4 && !old_form && N <= 65535 && g.hruns <= 65535 && lanes_x < (1ll << 31) - 256 &&
                        (int64_t)W * C < (1ll << 31) && (int64_t)g.Wo * C < (1ll << 31);
    if (dot_ok) {
        fast_division((uint32_t)(C / 4), g.magic_cgroups, g.shift_cgroups);
        const int variant = tuning().dw_variant; // tuning aid: 0 = patch kernel, 3 = matrix-unit kernel, -1 = by shape
        // matrix-unit kernel: whole 16-byte channel chunks, rows of at least 24 outputs (narrower images waste
        // most of the 32-pixel tile and stay with the patch kernel)
        if ((variant == 3 || variant < 0) && (C % 16) == 0 && (reinterpret_cast<uintptr_t>(x) % 16) == 0 &&
            (int64_t)H * W * C < (1ll << 31) && (int64_t)g.Ho * g.Wo * C < (1ll << 31) &&
            // measured: ahead of the patch kernel on stride-2 layers from 56 x 56 inputs up (+15 % at 112 x 112 and
            // at 56 x 56), by 5 % on stride-1 layers at least 48 pixels wide, and once a launch has more than ~10^8 outputs
            // (+25 %: 0.40 against 0.32 of HBM); behind it on the small layers, whose image rows fill less than
            // half of the 30-pixel tile
            // (and never below 2^21 outputs: a few dozen waves walking their segments row by row take longer than the
            // patch kernel's thousands of independent lanes -- 9 against 4 us on one 112 x 112 x 32 image)
            (variant == 3 ||
             ((int64_t)N * g.Ho * g.Wo * C >= (1ll << 21) && ((stride_h == 2 && g.Wo >= 24) || (stride_h == 1 && g.Wo >= 48))) ||
             (int64_t)N * g.Ho * g.Wo * C >= (100ll << 20))) {
            const int tiles_w = (g.Wo + 29) / 30, cblocks = (C + 31) / 32; // 30 output pixels per wave
            const int64_t waves_x = (int64_t)tiles_w * cblocks;
            int seg_rows = tuning().dw_rh > 0 ? tuning().dw_rh : 0;
            if (seg_rows <= 0) {
                const int64_t target = 2048; // waves: 2 per SIMD of the chip
                int64_t segs = (target + waves_x * N - 1) / (waves_x * N);
                const int64_t most = (g.Ho + 7) / 8; // at least 8 output rows per segment (each re-reads 2 input rows)
                segs = segs < 1 ? 1 : (segs > most ? most : segs);
                seg_rows = (int)((g.Ho + segs - 1) / segs);
            }
            if (seg_rows > g.Ho) seg_rows = g.Ho;
            const int segs = (g.Ho + seg_rows - 1) / seg_rows;
            const dim3 grid((unsigned)((waves_x + 3) / 4), (unsigned)segs, (unsigned)N);
            g.xcd_remap = tuning().dw_xcd != 0 && (int64_t)grid.x * grid.y * grid.z < (1ll << 31);
            auto launch = [&](auto zw, auto nt) {
                constexpr bool ZW = decltype(zw)::value, NT = decltype(nt)::value;
                with_rescale_mode(true, g.z_out, g.lo_rel, g.hi_rel, [&](auto mode) {
                    constexpr int MODE = decltype(mode)::value;
                    if constexpr (MODE != RESCALE_GENERAL) { // (channels that need that form are found in the kernel)
                        if (stride_h == 1) hipLaunchKernelGGL((dwconv3x3_mfma_kernel<1, MODE, ZW, NT>), grid, dim3(256), 0, s, g, seg_rows, tiles_w, cblocks);
                        else hipLaunchKernelGGL((dwconv3x3_mfma_kernel<2, MODE, ZW, NT>), grid, dim3(256), 0, s, g, seg_rows, tiles_w, cblocks);
                    }
                });
            };
            if (dw_stream_out(g, true)) z_w ? launch(std::true_type{}, std::true_type{}) : launch(std::false_type{}, std::true_type{});
            else z_w ? launch(std::true_type{}, std::false_type{}) : launch(std::false_type{}, std::false_type{});
            return launch_status(hipGetLastError());
        }
        // taller patches (4 output rows per lane) reuse more of the window, but need enough lanes to
        // give the chip something to do (tiny layers keep 2-row patches: twice the lanes)
        const int tall_env = tuning().dw_rh; // tuning aid: 2 or 4 forces the patch height
        const int64_t lanes_tall = lanes_x * ((g.Ho + 3) / 4) * N;
        const bool tall = tall_env ? tall_env == 4 : lanes_tall >= 16384;
        if (tall) g.hruns = (g.Ho + 3) / 4;
        const dim3 grid((unsigned)((lanes_x + 255) / 256), (unsigned)g.hruns, (unsigned)N);
        g.xcd_remap = tuning().dw_xcd != 0 && (int64_t)grid.x * grid.y * grid.z < (1ll << 31);
        auto launch = [&](auto zw, auto nt) {
            constexpr bool ZW = decltype(zw)::value, NT = decltype(nt)::value;
            if (tall && stride_h == 1) hipLaunchKernelGGL((dwconv3x3_dot_kernel<1, 4, ZW, NT>), grid, dim3(256), 0, s, g);
            else if (tall) hipLaunchKernelGGL((dwconv3x3_dot_kernel<2, 4, ZW, NT>), grid, dim3(256), 0, s, g);
            else if (stride_h == 1) hipLaunchKernelGGL((dwconv3x3_dot_kernel<1, RH, ZW, NT>), grid, dim3(256), 0, s, g);
            else hipLaunchKernelGGL((dwconv3x3_dot_kernel<2, RH, ZW, NT>), grid, dim3(256), 0, s, g);
        };
        if (dw_stream_out(g, false)) z_w ? launch(std::true_type{}, std::true_type{}) : launch(std::false_type{}, std::true_type{});
        else z_w ? launch(std::true_type{}, std::false_type{}) : launch(std::false_type{}, std::false_type{});
    } else if (c4 && stride_h == 1)
        hipLaunchKernelGGL((dwconv3x3_kernel<1, RH, RW>), dim3((unsigned)blocks), dim3(256), 0, s, g);
    else if (c4)
        hipLaunchKernelGGL((dwconv3x3_kernel<2, RH, RW>), dim3((unsigned)blocks), dim3(256), 0, s, g);
    else
        hipLaunchKernelGGL(dwconv_generic_kernel, dim3((unsigned)blocks), dim3(256), 0, s, g);
    return launch_status(hipGetLastError());
}

extern "C" qnn_status qnn_qdwconv2d(const uint8_t *x, int N, int H, int W, int C, int32_t z_x, const int8_t *w, int kh,
                                    int kw, int stride_h, int stride_w, int pad_h, int pad_w, const int32_t *bias,
                                    const int32_t *mult, const int32_t *shift, int32_t z_out, int32_t act_min,
                                    int32_t act_max, uint8_t *y, void *stream)
{
    return qdwconv2d_impl(x, N, H, W, C, z_x, w, kh, kw, stride_h, stride_w, pad_h, pad_w, bias, mult, shift, z_out, act_min,
                          act_max, y, stream, nullptr);
}

extern "C" qnn_status qnn_qdwconv2d_asym(const uint8_t *x, int N, int H, int W, int C, int32_t z_x, const int8_t *w, int kh,
                                         int kw, const int32_t *z_w, int stride_h, int stride_w, int pad_h, int pad_w,
                                         const int32_t *bias, const int32_t *mult, const int32_t *shift, int32_t z_out,
                                         int32_t act_min, int32_t act_max, uint8_t *y, void *stream)
{
    if (!z_w) return QNN_EINVAL;
    return qdwconv2d_impl(x, N, H, W, C, z_x, w, kh, kw, stride_h, stride_w, pad_h, pad_w, bias, mult, shift, z_out, act_min,
                          act_max, y, stream, z_w);
}
