// Launch templates of the weight-resident kernels, for the two files that instantiate them (8- and 4-bit weights).
#pragma once

#include "igemm_launch.h"
#include "bres_ring.h"

namespace qnn {

template <int NB, int KC, bool INT4, bool CONV, bool PAD = false>
inline hipError_t launch_bres_one(const BResArgs &a, unsigned blocks, int lds, hipStream_t s)
{
    auto kernel = bres_kernel<NB, KC, INT4, CONV, PAD>;
    static LdsOptIn opt_in; // per instantiation
    if (hipError_t e = opt_in.ensure(reinterpret_cast<const void *>(kernel), lds); e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(512), lds, s, a);
    return hipGetLastError();
}

template <int NB, bool INT4, bool CONV>
inline hipError_t launch_bres_kc(const BResArgs &a, unsigned blocks, int lds, hipStream_t s)
{
    // A fragments travel in chunks of KC K sub-steps; a chunk size that divides K / 32 wastes no MFMA
    const int ks = a.g.K / 32;
    if (ks % 8 == 0) return launch_bres_one<NB, 8, INT4, CONV>(a, blocks, lds, s);
    if (ks % 6 == 0) return launch_bres_one<NB, 6, INT4, CONV>(a, blocks, lds, s);
    if (ks % 4 == 0) return launch_bres_one<NB, 4, INT4, CONV>(a, blocks, lds, s);
    return launch_bres_one<NB, 6, INT4, CONV, true>(a, blocks, lds, s); // last chunk padded with zero operands
}

// the form with its rows through an LDS ring of RING slots per wave
template <int NB, int RING, bool INT4> inline hipError_t launch_ring_one(const BResArgs &a, unsigned blocks, int lds, hipStream_t s)
{
    auto kernel = bres_ring_kernel<NB, RING, INT4>;
    static LdsOptIn opt_in; // per instantiation
    if (hipError_t e = opt_in.ensure(reinterpret_cast<const void *>(kernel), lds); e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(512), lds, s, a);
    return hipGetLastError();
}

// slots: of the ring per wave that the weights leave room for (0: fragments from global memory)
template <int NB, bool INT4> inline hipError_t launch_bres_nb(const BResArgs &a, bool conv, int slots, unsigned blocks, int lds, hipStream_t s)
{
    if (slots >= 6) return launch_ring_one<NB, 6, INT4>(a, blocks, lds + 6 * 8 * 2048, s);
    if (slots >= 3) return launch_ring_one<NB, 3, INT4>(a, blocks, lds + 3 * 8 * 2048, s);
    return conv ? launch_bres_kc<NB, INT4, true>(a, blocks, lds, s) : launch_bres_kc<NB, INT4, false>(a, blocks, lds, s);
}

template <bool INT4> inline hipError_t launch_bres(const BResArgs &a, int nb, bool conv, int slots, unsigned blocks, int lds, hipStream_t s)
{
    if (nb == 4) return launch_bres_nb<4, INT4>(a, conv, slots, blocks, lds, s);
    if (nb == 2) return launch_bres_nb<2, INT4>(a, conv, slots, blocks, lds, s);
    return launch_bres_nb<1, INT4>(a, conv, slots, blocks, lds, s);
}

hipError_t launch_bres_int8(const BResArgs &a, int nb, bool conv, int slots, unsigned blocks, int lds, hipStream_t s);
hipError_t launch_bres_int4(const BResArgs &a, int nb, bool conv, int slots, unsigned blocks, int lds, hipStream_t s);

} // namespace qnn
