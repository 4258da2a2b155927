// Small helper kernels: layout conversion, counter reset, missing-channel flags.
#pragma once

#include "device_common.h"

namespace dagsched_dev {

// Two arrays [rows][cols] int32 -> [cols][rows], 64x64 tiles through LDS (both sides coalesced), one array per blockIdx.z; the sixteen
// loads of a thread are all on their way before the first is stored.  The evaluation of 2051 candidates of 3001
// operations: 131 us with a launch for each array and its loads one after the other, 119 with this.
__global__ __launch_bounds__(256) void transpose_i32_kernel(const int32_t *__restrict__ in0, const int32_t *__restrict__ in1, int32_t *__restrict__ out0,
                                                             int32_t *__restrict__ out1, int64_t rows, int64_t cols) {
  __shared__ int32_t tile[64][65];
  const int32_t *__restrict__ const in = blockIdx.z ? in1 : in0;
  int32_t *__restrict__ const out = blockIdx.z ? out1 : out0;
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  int32_t x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t r = r0 + ty + 4 * i, c = c0 + tx;
    x[i] = in[(r < rows ? r : rows - 1) * cols + (c < cols ? c : cols - 1)];
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) tile[ty + 4 * i][tx] = x[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t c = c0 + ty + 4 * i, r = r0 + tx;
    if (r < rows && c < cols) out[c * rows + r] = tile[tx][ty + 4 * i];
  }
}

// A fill kernel instead of a memset node: safe to record into a captured graph.
__global__ void reset_counter_kernel(int32_t *counter) {        // two words: the lists of the first and second fallback
  if (threadIdx.x == 0 && blockIdx.x == 0) { counter[0] = 0; counter[1] = 0; }
}

// Missing channels (Sec. III eqs. (9)-(10)), run after the evaluation when the cluster graph lacks some pair: one
// workgroup per candidate copies the candidate's placement into LDS as bytes (one coalesced pass over the row) and
// walks the edge list (u | v << 16, one coalesced dword per edge); an edge whose ends sit on machines a != b with
// bit b of no_channel[a] set makes the candidate NO_CHANNEL, unless it is malformed already (then its placement
// may not even be in range).  placement is candidate-major, N entries per candidate.  Dynamic LDS: 512 + N bytes;
// any workgroup size that is a multiple of 64.
// cand_list: only the candidates cand_list[0 .. *cand_count), in turn, whatever the grid.  Where the evaluation was told the placement that the
// candidates share, and that one keeps to the channels, these are the ones that place differently: looking at all 4096 candidates of 768
// operations took 8 us of every 78 us of a search over orders (ten steps 801 us then; about 700 with this, with 16-byte accesses in the proposals and three copies
// fewer around them; ten steps with 256 candidates of the MoE graph 2253 and 2087).
__global__ __launch_bounds__(1024) void channel_flag_kernel(int32_t N, int32_t E, int32_t P,
                                                            const uint32_t *__restrict__ edges,
                                                            const uint64_t *__restrict__ no_channel,
                                                            const int32_t *__restrict__ placement, int32_t C,
                                                            const int32_t *__restrict__ cand_list, const int32_t *__restrict__ cand_count, OutPtrs out) {
  extern __shared__ __align__(16) unsigned char channel_lds[];
  uint64_t *mask = reinterpret_cast<uint64_t *>(channel_lds);
  uint8_t *machine = channel_lds + DAGSCHED_MAX_DEVICES * sizeof(uint64_t);
  const int32_t todo = cand_list ? *cand_count : C;
  for (int32_t at = (int32_t)blockIdx.x; at < todo; at += (int32_t)gridDim.x) {
    const int64_t c = cand_list ? cand_list[at] : at;
    const int32_t before = out.flags[c];
    if (before == DAGSCHED_FLAG_BAD_PLACEMENT || before == DAGSCHED_FLAG_BAD_RANK) continue;   // uniform over the workgroup
    __syncthreads();                                        // (the candidate before may still be looked at)
    if ((int)threadIdx.x < DAGSCHED_MAX_DEVICES) mask[threadIdx.x] = (int)threadIdx.x < P ? no_channel[threadIdx.x] : 0;
    const int32_t *pl = placement + c * N;
    for (int32_t v = threadIdx.x; v < N; v += blockDim.x) machine[v] = (uint8_t)pl[v];
    __syncthreads();
    int found = 0;
#pragma unroll 4
    for (int32_t k = threadIdx.x; k < E; k += blockDim.x) {
      const uint32_t e = edges[k];
      const uint32_t a = machine[e & 0xFFFFu], b = machine[e >> 16];
      found |= (a != b) && ((mask[a] >> b) & 1u);
    }
    if (!__syncthreads_or(found)) continue;
    if (threadIdx.x == 0) {
      out.flags[c] = DAGSCHED_FLAG_NO_CHANNEL;
      out.makespan[c] = -1;
      out.bubble[c] = -1;
    }
    if ((int)threadIdx.x < P) out.peak_mem[c * out.peak_stride_c + threadIdx.x * out.peak_stride_j] = -1;
  }
}

}  // namespace dagsched_dev
