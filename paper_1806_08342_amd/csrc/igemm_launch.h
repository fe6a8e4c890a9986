// Host-side launch routines of the dense quantized layers; each kernel family is compiled in a
// translation unit of its own (igemm_*.hip) and called from the dispatcher in igemm.hip.
#pragma once

#include <atomic>
#include <cstdint>
#include <cstdlib>

#include "igemm.h"

namespace qnn {

// magic number for dividing by d with a multiply-high (see the kernels that take it)
inline uint32_t magic_for(uint32_t d) { return d <= 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d); }

// Kernels that use more than 64 KB of dynamic LDS must opt in once per device.  One object per kernel
// instantiation (a function-local static); safe to call from several threads (setting the attribute
// twice is harmless).
struct LdsOptIn {
    std::atomic<int> enabled[64] = {}; // bytes enabled so far, per device
    hipError_t ensure(const void *kernel, int bytes)
    {
        int dev = 0;
        if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
        if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
        if (enabled[dev].load(std::memory_order_acquire) >= bytes) return hipSuccess;
        if (hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); e != hipSuccess) return e;
        enabled[dev].store(bytes, std::memory_order_release);
        return hipSuccess;
    }
};

inline bool aligned_to(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Short reduction (K <= 256): weight-stationary kernel of shortk.h.  `strided`: rows are the pixels
// of a strided 1x1 convolution.  Not eligible when the operands miss its alignment rules.
bool shortk_eligible(const IgemmArgs &g, int b_mode, bool strided);
qnn_status launch_shortk(IgemmArgs &g, int b_mode, bool strided, hipStream_t s);

// Few rows, and launches that are small altogether: kernel of smallk.h.  Returns false if the shape does not fit.
bool small_shape(int64_t M, int64_t N, int64_t K, bool conv, bool int4); // sizes only
bool try_small(const IgemmArgs &g, int a_mode, int b_mode, hipStream_t s, qnn_status *status);

// Medium reduction, few output channels: weight-resident kernel of bres.h.  Returns false when the
// shape or the alignment does not fit (the caller then takes the tiled route).
bool try_bres(IgemmArgs &g, int a_mode, int b_mode, hipStream_t s, qnn_status *status);

// Network stems (very few input channels): kernels of stemwave.h / stemconv.h.  `g` carries the
// convolution geometry; returns false if the layer is not a stem these kernels cover.
bool stem_shape(int64_t W, int Cin, int Cout, int kh, int kw, int stride_w, int weight_bits);
bool try_stem(IgemmArgs &g, int batch, int kh, int stride_h, int stride_w, int weight_bits, hipStream_t s, qnn_status *status);

struct SplitK;
// Pipelined tiles bm x bn for K % 64 != 0 (igemm_tail.hip)
hipError_t launch_tail_tile(const IgemmArgs &g, int bm, int bn, bool mat, bool i4, const SplitK &sk, hipStream_t s);

// 64x64 tiles for few output tiles, any K of whole chunks; g.zw and sk (8-bit weights) as set
hipError_t launch_tile64(const IgemmArgs &g, bool mat, bool i4, const SplitK &sk, hipStream_t s);

// Zero-padded copies of operands that are no whole, aligned 16-byte chunks (igemm_repack.hip).  `length`: K of a
// matrix, Cin of a convolution.  launch_repack points g at the copies in `workspace` (repack_bytes of it).
int repack_length(int length, int weight_bits);
size_t repack_bytes(int64_t rows_a, int64_t rows_b, int length, int weight_bits);
qnn_status launch_repack(IgemmArgs &g, int a_mode, int weight_bits, int kh, void *workspace, hipStream_t s);

// Register-staged tiles of igemm.h (any alignment, any weight layout): 64x64 or 128x128.
void launch_plain_tile(bool big, const IgemmArgs &g, int a_mode, int b_mode, int vec, hipStream_t s);
// the 64x64 tile with per-column weight zero-points (g.zw set)
void launch_plain_tile_zw(const IgemmArgs &g, int a_mode, int b_mode, int vec, hipStream_t s);

} // namespace qnn
