// 16-byte buffer accesses: a base and a size that are the same in the whole wave, a 32-bit offset per lane; what lies beyond the
// size is dropped (stores), reads as zero (loads) and costs no traffic.  And the division for the rows that such offsets address.  The bodies exist in the device pass only: the
// resource type does.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace qnn {

using buf16 = uint32_t __attribute__((ext_vector_type(4)));

// NT: non-temporal
template <bool NT> __device__ __forceinline__ void buffer_store16(uint8_t *base, int bytes, uint32_t offset, buf16 v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_buffer_store_b128(v, __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000), (int)offset, 0, NT ? 2 : 0);
#else
    (void)base, (void)bytes, (void)offset, (void)v;
#endif
}

__device__ __forceinline__ buf16 buffer_load16(const uint8_t *base, int bytes, uint32_t offset)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base), 0, bytes, 0x00020000), (int)offset, 0, 0);
#else
    (void)base, (void)bytes, (void)offset;
    return buf16{0u, 0u, 0u, 0u};
#endif
}

using buf8 = uint32_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ buf8 buffer_load8(const uint8_t *base, int bytes, uint32_t offset)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_raw_buffer_load_b64(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base), 0, bytes, 0x00020000), (int)offset, 0, 0);
#else
    (void)base, (void)bytes, (void)offset;
    return buf8{0u, 0u};
#endif
}

// 16 bytes per lane to 1024 consecutive bytes of LDS in lane order; `lds` is the same in the whole wave
__device__ __forceinline__ void buffer_to_lds16(const uint8_t *base, int bytes, uint32_t offset, uint8_t *lds)
{
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base), 0, bytes, 0x00020000),
                                             (__attribute__((address_space(3))) void *)lds, 16, (int)offset, 0, 0, 0);
#else
    (void)base, (void)bytes, (void)offset, (void)lds;
#endif
}

// m / d for m < 2^31: the product with ceil(2^32 / d) is at most one too high (magic 0: d = 1)
__device__ __forceinline__ uint32_t ring_div(uint32_t m, uint32_t d, uint32_t magic, uint32_t &rem)
{
    uint32_t q = __umulhi(m, magic) + (magic == 0 ? m : 0u);
    rem = m - q * d;
    const uint32_t high = rem >> 31;
    rem += high * d;
    return q - high;
}

} // namespace qnn
