// The weight-resident kernels for 4-bit weights.
#include "bres_launch.h"

namespace qnn {

hipError_t launch_bres_int4(const BResArgs &a, int nb, bool conv, int slots, unsigned blocks, int lds, hipStream_t s) { return launch_bres<true>(a, nb, conv, slots, blocks, lds, s); }

} // namespace qnn
