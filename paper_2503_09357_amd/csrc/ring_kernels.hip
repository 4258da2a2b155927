// One translation unit of the ring kernel's instantiations: DAGSCHED_RING_HALF and DAGSCHED_RING_SUB say which.
#include <hip/hip_runtime.h>

#include "ring_kernels.h"

namespace dagsched_dev {

// The instantiated shapes: placement bytes in LDS with 4 or 8 ring slots, as nibbles in LDS likewise, in L2 with 8, 16
// or 32; one to four feeders where that was ever measured useful; each in the three kinds of the kernel.
#define DAGSCHED_RING_CASES(PIB, RING, F)                                                         \
  case 0 * 10000 + PIB * 1000 + RING * 10 + F: return relax_ring_kernel<RING, F, HALF, PIB, 0, 0, SUB>;    \
  case 1 * 10000 + PIB * 1000 + RING * 10 + F: return relax_ring_kernel<RING, F, HALF, PIB, 1, 0, SUB>;    \
  case 2 * 10000 + PIB * 1000 + RING * 10 + F: return relax_ring_kernel<RING, F, HALF, PIB, 2, 0, SUB>;
// the one-predecessor kind: 16-bit cells only
#define DAGSCHED_RING_CASES_ONE(PIB, RING, F)                                                     \
  case 3 * 10000 + PIB * 1000 + RING * 10 + F: return relax_ring_kernel<RING, F, HALF, PIB, 3, 0, SUB>;
// window mode: the relaxation launch (PHASE = 2) in the shapes that large layered problems get, and the ingest launch
#define DAGSCHED_WIN_CASES(RING, F)                                                               \
  case 0 * 10000 + RING * 10 + F: return relax_ring_kernel<RING, F, HALF, 0, 0, 2>;               \
  case 1 * 10000 + RING * 10 + F: return relax_ring_kernel<RING, F, HALF, 0, 1, 2>;               \
  case 2 * 10000 + RING * 10 + F: return relax_ring_kernel<RING, F, HALF, 0, 2, 2>;

template <int HALF, int SUB>
RingKernel ring_kernel_pick(int ring, int feeders, int pib_lds, int kind) {
  if constexpr (SUB > 1) {                                      // several lanes per machine
    if constexpr (HALF == 0) {
      switch (kind * 10000 + pib_lds * 1000 + ring * 10 + feeders) {
        DAGSCHED_RING_CASES_ONE(1, 4, 1) DAGSCHED_RING_CASES_ONE(1, 4, 2) DAGSCHED_RING_CASES_ONE(1, 8, 1) DAGSCHED_RING_CASES_ONE(1, 8, 2)
        DAGSCHED_RING_CASES_ONE(2, 8, 1) DAGSCHED_RING_CASES_ONE(2, 8, 2) DAGSCHED_RING_CASES_ONE(0, 8, 1) DAGSCHED_RING_CASES_ONE(0, 8, 2)
      }
    }
    if constexpr (SUB == 2) {
      switch (kind * 10000 + pib_lds * 1000 + ring * 10 + feeders) {
        DAGSCHED_RING_CASES(1, 4, 3) DAGSCHED_RING_CASES(1, 8, 3) DAGSCHED_RING_CASES(0, 8, 3)
        DAGSCHED_RING_CASES(0, 16, 1) DAGSCHED_RING_CASES(0, 16, 2) DAGSCHED_RING_CASES(0, 16, 3)
      }
    }
    switch (kind * 10000 + pib_lds * 1000 + ring * 10 + feeders) {
      DAGSCHED_RING_CASES(1, 4, 1) DAGSCHED_RING_CASES(1, 4, 2) DAGSCHED_RING_CASES(1, 8, 1) DAGSCHED_RING_CASES(1, 8, 2)
      DAGSCHED_RING_CASES(2, 8, 1) DAGSCHED_RING_CASES(2, 8, 2) DAGSCHED_RING_CASES(0, 8, 1) DAGSCHED_RING_CASES(0, 8, 2)
      default: return nullptr;
    }
  } else if constexpr (HALF == 5) {                                    // window mode with 32-bit end times: fewer shapes
    if (pib_lds != 0) return nullptr;
    switch (kind * 10000 + ring * 10 + feeders) {
      DAGSCHED_WIN_CASES(8, 2) DAGSCHED_WIN_CASES(16, 2) DAGSCHED_WIN_CASES(16, 3)
      default: return nullptr;
    }
  } else if constexpr (HALF == 4) {
    if (pib_lds != 0) return nullptr;
    switch (kind * 10000 + ring * 10 + feeders) {
      DAGSCHED_WIN_CASES(8, 1) DAGSCHED_WIN_CASES(8, 2) DAGSCHED_WIN_CASES(8, 3)
      DAGSCHED_WIN_CASES(16, 2) DAGSCHED_WIN_CASES(16, 3) DAGSCHED_WIN_CASES(16, 4)
      default: return nullptr;
    }
  } else if constexpr (HALF == 2) {                             // 32-bit end times: the shapes that large problems get
    switch (kind * 10000 + pib_lds * 1000 + ring * 10 + feeders) {
      DAGSCHED_RING_CASES(1, 8, 1) DAGSCHED_RING_CASES(1, 8, 2) DAGSCHED_RING_CASES(1, 8, 3)
      DAGSCHED_RING_CASES(2, 8, 2) DAGSCHED_RING_CASES(2, 8, 3)
      DAGSCHED_RING_CASES(0, 8, 2) DAGSCHED_RING_CASES(0, 16, 2) DAGSCHED_RING_CASES(0, 16, 3) DAGSCHED_RING_CASES(0, 16, 4)
      default: return nullptr;
    }
  } else if constexpr (HALF == 3) {                      // ... and wide ops (no nibbles)
    switch (kind * 10000 + pib_lds * 1000 + ring * 10 + feeders) {
      DAGSCHED_RING_CASES(1, 8, 1) DAGSCHED_RING_CASES(1, 8, 2) DAGSCHED_RING_CASES(1, 8, 3)
      DAGSCHED_RING_CASES(0, 8, 2) DAGSCHED_RING_CASES(0, 16, 2) DAGSCHED_RING_CASES(0, 16, 3) DAGSCHED_RING_CASES(0, 16, 4)
      default: return nullptr;
    }
  } else {
  switch (kind * 10000 + pib_lds * 1000 + ring * 10 + feeders) {
    DAGSCHED_RING_CASES(1, 4, 1) DAGSCHED_RING_CASES(1, 4, 2)
    DAGSCHED_RING_CASES(1, 8, 1) DAGSCHED_RING_CASES(1, 8, 2) DAGSCHED_RING_CASES(1, 8, 3) DAGSCHED_RING_CASES(1, 8, 4)
    DAGSCHED_RING_CASES(2, 4, 1) DAGSCHED_RING_CASES(2, 4, 2)
    DAGSCHED_RING_CASES(2, 8, 1) DAGSCHED_RING_CASES(2, 8, 2) DAGSCHED_RING_CASES(2, 8, 3)
    DAGSCHED_RING_CASES(0, 8, 1) DAGSCHED_RING_CASES(0, 8, 2) DAGSCHED_RING_CASES(0, 8, 3)
    DAGSCHED_RING_CASES(0, 16, 1) DAGSCHED_RING_CASES(0, 16, 2) DAGSCHED_RING_CASES(0, 16, 3) DAGSCHED_RING_CASES(0, 16, 4)
    DAGSCHED_RING_CASES(0, 32, 1) DAGSCHED_RING_CASES(0, 32, 2) DAGSCHED_RING_CASES(0, 32, 3)
    DAGSCHED_RING_CASES_ONE(1, 4, 1) DAGSCHED_RING_CASES_ONE(1, 4, 2)
    DAGSCHED_RING_CASES_ONE(1, 8, 1) DAGSCHED_RING_CASES_ONE(1, 8, 2) DAGSCHED_RING_CASES_ONE(1, 8, 3)
    DAGSCHED_RING_CASES_ONE(2, 8, 1) DAGSCHED_RING_CASES_ONE(2, 8, 2) DAGSCHED_RING_CASES_ONE(2, 8, 3)
    DAGSCHED_RING_CASES_ONE(0, 8, 2) DAGSCHED_RING_CASES_ONE(0, 8, 3) DAGSCHED_RING_CASES_ONE(0, 16, 2) DAGSCHED_RING_CASES_ONE(0, 16, 3)
    default: return nullptr;
  }
  }
}

#if DAGSCHED_RING_HALF == 4
RingKernel ring_ingest_kernel(int kind) {
  return kind == 0 ? relax_ring_kernel<8, 2, 4, 0, 0, 1> : kind == 1 ? relax_ring_kernel<8, 2, 4, 0, 1, 1> : relax_ring_kernel<8, 2, 4, 0, 2, 1>;
}
#endif

template RingKernel ring_kernel_pick<DAGSCHED_RING_HALF, DAGSCHED_RING_SUB>(int, int, int, int);

}  // namespace dagsched_dev
