// Operands whose rows are no whole, aligned 16-byte chunks (odd K, odd pitches, odd channel counts), copied once per
// call into the caller's workspace in rows padded with zeros, so that the pipelined kernels apply.
//
// Bound by memory: one 16-byte chunk per lane, consecutive lanes on consecutive chunks of a row.  The padded
// copies are M*K + N*K bytes written and read again next to 2*M*N*K operations: 1021 x 1001 x 1027 spends 2 us on
// it, while its byte-wise staged loads took 100 us.
#include "igemm_launch.h"
#include "smallk.h"

namespace qnn {

struct RepackPart {
    const uint8_t *src;
    uint8_t *dst;
    int64_t pitch;          // source row pitch in bytes
    int32_t len;            // source row length in bytes
    uint32_t cpr;           // chunks per padded row
    uint32_t magic, shift;  // x / cpr = umulhi(x, magic) >> shift for x < 2^31, cpr >= 2
    uint32_t chunks;        // rows * cpr
};

__global__ void __launch_bounds__(256) repack_kernel(const RepackPart a, const RepackPart b)
{
    uint32_t i = blockIdx.x * 256u + threadIdx.x;
    const bool second = i >= a.chunks;
    const RepackPart &p = second ? b : a;
    if (second) i -= a.chunks;
    if (i >= p.chunks) return;
    const uint32_t row = p.cpr == 1 ? i : __umulhi(i, p.magic) >> p.shift;
    const uint32_t c = i - row * p.cpr;
    const u32x4 v = load_tail16(p.src + (int64_t)row * p.pitch, (int)(c * 16), p.len);
    *reinterpret_cast<u32x4 *>(p.dst + (uint64_t)i * 16) = v;
}

static RepackPart make_part(const uint8_t *src, int64_t pitch, int64_t rows, int len, int padded, uint8_t *dst)
{
    RepackPart p = {};
    p.src = src, p.dst = dst, p.pitch = pitch, p.len = len;
    const uint32_t d = (uint32_t)(padded / 16);
    p.cpr = d;
    fast_division(d, p.magic, p.shift);
    p.chunks = (uint32_t)(rows * d);
    return p;
}

static size_t round256(size_t n) { return (n + 255) / 256 * 256; }

int repack_length(int length, int weight_bits) { return weight_bits == 4 ? (length + 31) / 32 * 32 : (length + 15) / 16 * 16; }

size_t repack_bytes(int64_t rows_a, int64_t rows_b, int length, int weight_bits)
{
    const int64_t padded = repack_length(length, weight_bits);
    if ((rows_a + rows_b) * (padded / 16) >= ((int64_t)1 << 31)) return 0; // beyond the kernel's chunk index
    return round256((size_t)(rows_a * padded)) + round256((size_t)(rows_b * (padded * weight_bits / 8)));
}

qnn_status launch_repack(IgemmArgs &g, int a_mode, int weight_bits, int kh, void *workspace, hipStream_t s)
{
    const bool conv = a_mode == A_CONV;
    const int length = conv ? g.Cin : g.K, padded = repack_length(length, weight_bits);
    const int64_t rows_a = conv ? g.M / ((int64_t)g.Ho * g.Wo) * g.H * g.W : g.M;
    const int64_t rows_b = conv ? (int64_t)g.N * kh * g.kw : g.N;
    uint8_t *const a2 = static_cast<uint8_t *>(workspace);
    uint8_t *const b2 = a2 + round256((size_t)(rows_a * padded));
    const RepackPart pa = make_part(g.A, conv ? g.Cin : g.lda, rows_a, length, padded, a2);
    const RepackPart pb = make_part(g.B, (conv ? g.Cin : g.ldb) * weight_bits / 8, rows_b, length * weight_bits / 8, padded * weight_bits / 8, b2);
    const uint64_t chunks = (uint64_t)pa.chunks + pb.chunks;
    hipLaunchKernelGGL(repack_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, s, pa, pb);
    g.A = a2, g.B = b2;
    if (conv) {
        g.Cin = padded;
        g.magic_cin = magic_for((uint32_t)padded);
        g.K = kh * g.kw * padded;
        g.ldb = g.K;
    } else {
        g.K = padded;
        g.lda = g.ldb = padded;
    }
    return launch_status(hipGetLastError());
}

} // namespace qnn
