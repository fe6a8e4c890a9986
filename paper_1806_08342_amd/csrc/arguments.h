// Kernel arguments are read by scalar loads from memory that no cache holds when a kernel starts, 200 cycles a line in a replayed
// graph and 600 in a launch, and the compiler places each load where its value is first needed: a chain of four to eight such
// round trips at the head of a launch that takes 10 000 cycles in all.  fetch_arguments, as a kernel's first statement, reads one
// word of every 64-byte line at once; what follows finds the lines in the scalar cache.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace qnn {

template <int BYTES> __device__ __forceinline__ void fetch_arguments()
{
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(BYTES <= 512, "at most eight lines");
    constexpr int last = (BYTES - 4) & ~3;
    uint32_t t0, t1, t2, t3, t4, t5, t6, t7;
    asm volatile("s_load_dword %0, %8, %9\n\t"
                 "s_load_dword %1, %8, %10\n\t"
                 "s_load_dword %2, %8, %11\n\t"
                 "s_load_dword %3, %8, %12\n\t"
                 "s_load_dword %4, %8, %13\n\t"
                 "s_load_dword %5, %8, %14\n\t"
                 "s_load_dword %6, %8, %15\n\t"
                 "s_load_dword %7, %8, %16\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&s"(t0), "=&s"(t1), "=&s"(t2), "=&s"(t3), "=&s"(t4), "=&s"(t5), "=&s"(t6), "=&s"(t7)
                 : "s"(__builtin_amdgcn_kernarg_segment_ptr()), "n"(0), "n"(last < 64 ? last : 64), "n"(last < 128 ? last : 128), "n"(last < 192 ? last : 192),
                   "n"(last < 256 ? last : 256), "n"(last < 320 ? last : 320), "n"(last < 384 ? last : 384), "n"(last));
#endif
}

} // namespace qnn
