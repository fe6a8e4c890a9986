// Waits and barriers of the kernels that copy their operands into an LDS ring.
#pragma once

#include <hip/hip_runtime.h>

namespace qnn {

template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    // gfx9 encoding: vmcnt = {imm[15:14], imm[3:0]}, expcnt = imm[6:4], lgkmcnt = imm[11:8]
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// workgroup barrier that the compiler may not move memory operations across; unlike
// __syncthreads() it does not wait for outstanding global loads (the LDS DMA pipeline
// must stay in flight across it)
__device__ __forceinline__ void block_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// barrier over the LDS traffic of the workgroup: what was written is visible, what was read may be overwritten;
// requests to memory stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

} // namespace qnn
