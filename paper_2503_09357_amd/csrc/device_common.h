// Shared device-side definitions of the dagsched kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dagsched.h"

namespace dagsched_dev {

constexpr int kWave = 64;

// bits collected per candidate while it is being evaluated; turned into one DAGSCHED_FLAG_* at the end
constexpr int kBitCyclic = 1, kBitBadPlacement = 2, kBitBadRank = 4, kBitInternal = 8, kBitOverMemory = 16;
constexpr int kBitOtherPlacement = 64;   // the candidate does not use the shared placement: another kernel evaluates it

__device__ __forceinline__ int flag_from_bits(int bits) {
  return (bits & kBitBadPlacement) ? DAGSCHED_FLAG_BAD_PLACEMENT
       : (bits & kBitBadRank)      ? DAGSCHED_FLAG_BAD_RANK
       : (bits & kBitInternal)     ? DAGSCHED_FLAG_INTERNAL
       : (bits & kBitCyclic)       ? DAGSCHED_FLAG_CYCLIC
       : (bits & kBitOverMemory)   ? DAGSCHED_FLAG_OVER_MEMORY
                                   : DAGSCHED_FLAG_OK;
}

// Loads/stores that must observe data written earlier in the same kernel by other lanes go to L2
// (agent scope) so that a stale line in the per-CU vector cache can never be returned.
__device__ __forceinline__ int32_t ld_agent(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(int32_t *p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The same for data that only the wavefronts of one workgroup exchange (they share the CU's vector cache): a plain load or
// store that the compiler neither caches nor drops.  An agent-scope load leaves the XCD (700 ns against 120).
__device__ __forceinline__ int32_t ld_group(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void st_group(int32_t *p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// LDS pointers with an explicit address space: volatile accesses through generic pointers would be
// compiled to flat loads, these compile to ds_read/ds_write.
#define DAGSCHED_LDS __attribute__((address_space(3)))
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef DAGSCHED_LDS unsigned char lds_byte_t;
typedef DAGSCHED_LDS volatile uint32_t lds_vu32_t;
typedef DAGSCHED_LDS volatile uint64_t lds_vu64_t;
typedef DAGSCHED_LDS volatile uint16_t lds_vu16_t;
typedef DAGSCHED_LDS volatile int32_t lds_vi32_t;
typedef DAGSCHED_LDS const uint8_t lds_cu8_t;
typedef DAGSCHED_LDS volatile u32x4_t lds_vu32x4_t;

// A lane's bit of a mask kept in scalar registers, as a condition (the mask itself is combined with scalar instructions).
__device__ __forceinline__ bool lane_bit(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// (lower / upper half of x) << 2 in one instruction
__device__ __forceinline__ uint32_t lo16_x4(uint32_t x) {
  uint32_t r;
  asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(r) : "v"(2u), "v"(x));
  return r;
}
__device__ __forceinline__ uint32_t hi16_x4(uint32_t x) {
  uint32_t r;
  asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(r) : "v"(2u), "v"(x));
  return r;
}

// Where the outputs of one evaluate call go.
struct OutPtrs {
  int32_t *makespan;
  int64_t *bubble;
  int64_t *peak_mem;
  int32_t *flags;
  int64_t peak_stride_c, peak_stride_j;   // peak_mem[c*peak_stride_c + j*peak_stride_j]
};

}  // namespace dagsched_dev
