// The instantiations of the ring kernel.  They are compiled in translation units of their own (ring_kernels.hip, once for every
// pair of cell format and lanes per machine), side by side: together they take minutes.
#pragma once

#include "kernel_ring.h"

namespace dagsched_dev {

using RingKernel = void (*)(RingParams);
// HALF and SUB as in kernel_ring.h; NULL where the shape is not built
template <int HALF, int SUB>
RingKernel ring_kernel_pick(int ring, int feeders, int pib_lds, int kind);
// window mode's ingest launch
RingKernel ring_ingest_kernel(int kind);


}  // namespace dagsched_dev
