// Pipeline kernel: candidates that share one placement (as for kernel_static.h) on a graph where every operation waits
// for at most one operation whose end time has to be looked up.
//
// With the allocation known, an edge between two operations of one machine needs no end time: the machine runs them
// one after the other, so eqs. (11)-(13) hold exactly when the order has them the right way round, and a candidate
// that has not is cyclic.  Of a pipeline's edges the ones that other paths imply are dropped, and what is left is one
// edge per operation that crosses machines, so
//
//   relaxers   (waves 0 .. W-1) read one cell a step: x = max(e_chainpred, cell + K), one addition and one maximum
//              (K: delay and the number of the cell's user that is waited for, see share_cells.h), and keep the machine's memory
//              level and its peak (eqs. (17)-(19)) as its operations pass
//   checkers   (the other waves) look the ranks of operations that share a machine up again and compare them with B
//
// A candidate's cells are few (zero-bubble pipeline: 34 words instead of 768 half words), so two workgroups fit a CU and one
// relaxes while the other reads its next candidates; the rows of a workgroup's next batch are on their way while it relaxes.
//
// What bounds it: HBM traffic, part of it of its own making.  Zero-bubble pipeline, 768 operations, 65536 candidates: 124 us in the kernel, 594 MB by the counters,
// 4.8 TB/s, what a copy reaches; 408 MB would do.  The rest is a second read of nearly every rank row: the checkers come to it after the next
// batch's rows have pushed it out of the L2.  The LDS is busy 59 % of the time (47 % of that bank conflicts of the 16-byte gathers), the VALU 57 %.
// The step is written out in assembly because what a lane does only when its operation has run (most lanes wait in most steps)
// is done under the lanes' mask, without a branch and without a wait: the cell is written, the next operation moves up
// and the one after it is requested by those lanes only; the decisions between two blocks of steps are part of it.
// The same batch, whole evaluation: 291 us with kernel_static.h (one workgroup of four relaxers a CU), 161 with this kernel while accountants took the
// levels through the LDS and the decisions were the compiler's, 130 now.
#pragma once

#include "device_common.h"

namespace dagsched_dev {

struct PipelineParams {
  int32_t N, P, Pseg, log_pseg, G, W, C;   // G candidates per relaxer, W relaxers per workgroup
  const uint4 *ops;          // [N + 1] x = K, y = duration + (own user << T), z = offset of the cell read | of the own cell << 16,
                             //         w = A_i / mem_scale; entry N: never ready, ends every machine's list
  const uint8_t *machine;    // [N rounded up to 4] the shared placement
  const int32_t *off;        // [Pseg + 1] operations on the machines before machine j
  const uint32_t *pairs;     // [n_pairs] u | v << 16: edges of B inside a machine that no cell stands for
  int32_t n_pairs;
  int64_t mem_scale;         // common factor of the A_i
  const int64_t *base;       // [P] static memory on each machine under the shared placement (eq. (16)), or NULL
  const int64_t *mem_limit;  // [P] or NULL
  int64_t sum_dur;           // original units
  int32_t time_scale;
  uint32_t limit;            // 1 << T
  const int32_t *placement, *rank;   // [C][N]
  int32_t *fb_count, *fb_list;       // candidates with another placement
  uint32_t n_cells;                  // cell 0 (always 0), the shared ones, one that nobody reads
  uint32_t o_mach, o_cand, cand_stride, o_list, o_book, total;   // LDS: ops at 0; per candidate cells, then list
  OutPtrs out;
};

// One step of the relaxer, for all lanes whose machine can go on.  e: the cell that the operation at work waits for; v[44:45]: its K and D;
// v[40:43]: the next operation; idn: number of the one after it; lp: where the list goes on.  Order of the LDS accesses: own cell, cell
// waited for, next operation, list.  The first wait is for the cell (two accesses after it may be on their way), the
// second for next operation and list, which the access before them has had a whole step to let through.  list_address: instructions that
// work out where the list goes on, list: the register that holds it.
#define DAGSCHED_PIPELINE_STEP(list_address, list)                                                                              \
  "s_waitcnt lgkmcnt(2)\n\t"                                                                                                    \
  "v_add_u32 %[x], %[e], v44\n\t"                                                                                              \
  "v_max_u32 %[x], %[xa], %[x]\n\t"                                                                                             \
  "v_cmp_gt_u32 vcc, %[lim], %[x]\n\t"                                                                                          \
  "v_add_u32 %[y], %[x], v45\n\t"                                                                                              \
  "s_mov_b64 exec, vcc\n\t"                                                                                                    \
  "ds_write_b32 %[own], %[y]\n\t"                                                                                               \
  "s_waitcnt lgkmcnt(1)\n\t"                                                                                                    \
  "v_add_u32_sdwa %[at], %[cb], v42 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"                     \
  "s_mov_b64 exec, %[all]\n\t"                                                                                                  \
  "ds_read_b32 %[e], %[at]\n\t"                                                                                                 \
  "s_mov_b64 exec, vcc\n\t"                                                                                                     \
  "v_and_b32 %[xa], %[tm], %[y]\n\t"                                                                                            \
  "v_add_u32_sdwa %[own], %[cb], v42 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"                    \
  "v_mov_b64 v[44:45], v[40:41]\n\t"                                                                                           \
  "v_add_u32 %[lvl], %[lvl], v43\n\t"                                                                                          \
  "v_max_i32 %[pk], %[pk], %[lvl]\n\t"                                                                                         \
  "v_lshl_add_u32 %[x], %[idn], 4, %[ob]\n\t"                                                                                   \
  list_address                                                                                                                  \
  "ds_read_b128 v[40:43], %[x]\n\t"                                                                                             \
  "ds_read_u16 %[idn], " list "\n\t"                                                                                           \
  "v_add_u32 %[lp], 2, %[lp]\n\t"                                                                                               \
  "s_mov_b64 exec, %[all]\n\t"
#define DAGSCHED_FUSED_STEP DAGSCHED_PIPELINE_STEP("", "%[lp]")
#define DAGSCHED_STREAM_STEP DAGSCHED_PIPELINE_STEP("v_and_or_b32 %[y], %[lp], 63, %[ring]\n\t", "%[y]")   // lp: bytes of the order loaded so far
// Blocks of eight steps as long as some lane is not through and something ran in a block's last step, at most `turns` of them.
#define DAGSCHED_PIPELINE_LOOP                                                                                                  \
  "s_waitcnt lgkmcnt(0)\n"                                                                                                      \
  ".Lpipeline%=:\n\t"                                                                                                           \
  DAGSCHED_FUSED_STEP DAGSCHED_FUSED_STEP DAGSCHED_FUSED_STEP DAGSCHED_FUSED_STEP                                               \
  DAGSCHED_FUSED_STEP DAGSCHED_FUSED_STEP DAGSCHED_FUSED_STEP DAGSCHED_FUSED_STEP                                               \
  "s_mov_b64 %[moved], vcc\n\t"                                                                                                \
  "v_cmp_ne_u32 vcc, %[lp], %[end]\n\t"                                                                                        \
  "s_sub_u32 %[turns], %[turns], 1\n\t"                                                                                        \
  "s_cbranch_vccz .Lpipeline_end%=\n\t"                                                                                        \
  "s_cmp_eq_u64 %[moved], 0\n\t"                                                                                               \
  "s_cbranch_scc1 .Lpipeline_end%=\n\t"                                                                                        \
  "s_cmp_lg_u32 %[turns], 0\n\t"                                                                                               \
  "s_cbranch_scc1 .Lpipeline%=\n"                                                                                              \
  ".Lpipeline_end%=:\n\t"                                                                                                       \
  "s_waitcnt lgkmcnt(0)"

constexpr int kPipelineWavesPerSimd = 4;                     // (128 registers: the rows on their way take 48 of them)

__global__ __launch_bounds__(512, kPipelineWavesPerSimd) void relax_pipeline_kernel(PipelineParams p) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int T = (int)blockDim.x;                            // at least 128 * W
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = p.N, P = p.P, Pseg = p.Pseg, G = p.G, W = p.W;
  const int GW = G * W;                                     // candidates per batch, at most 64
  const int n_batches = (int)(((int64_t)p.C + GW - 1) / GW);
  lds_byte_t *const ldsb = (lds_byte_t *)lds;
  uint4 *const opsw = (uint4 *)lds;
  uint32_t *const machw = (uint32_t *)(lds + p.o_mach);     // [N / 4 rounded up] the shared placement, four machines per word
  int32_t *const flagw = (int32_t *)(lds + p.o_book);       // [64]
  uint32_t *const pairw = (uint32_t *)(lds + p.o_book + 256);   // [64] start of machine j in every list | operations << 16
  int32_t *const cycw = (int32_t *)(lds + p.o_book + 512);  // [64] 1 = an order contradicts B inside a machine
  uint16_t *const idle_list = (uint16_t *)(lds + p.o_book + 768);   // four entries that name operation N

  const int tpc = T / GW, team = tid / tpc, tt = tid - team * tpc;   // ingest: a team of consecutive threads per candidate
  constexpr int kChunk = 6;
  const bool vec_ok = ((N & 3) == 0) && ((((uintptr_t)p.placement) | ((uintptr_t)p.rank)) & 15) == 0;
  const int nq = N >> 2;
  const int n_list = N + P + 3;                             // entries: a terminal per machine, three more at the end
  const int cwords = (int)p.n_cells, lwords = (n_list + 1) / 2;

  for (int i = tid; i <= N; i += T) opsw[i] = p.ops[i];
  for (int i = tid; i < (N + 3) / 4; i += T) machw[i] = ((const uint32_t *)p.machine)[i];
  if (tid < 64) pairw[tid] = tid < P ? (uint32_t)(p.off[tid] + tid) | ((uint32_t)(p.off[tid + 1] - p.off[tid]) << 16) : 0u;
  if (tid < 4) idle_list[tid] = (uint16_t)N;

  const bool lane_on = lane < G * Pseg;
  const int ql = lane_on ? lane : 0;
  const int g = ql >> p.log_pseg, j = ql & (Pseg - 1);
  const int gi = wave < W ? wave * G + g : 0;               // candidate slot of this lane (relaxers)

  int4 a4[kChunk], r4[kChunk];                              // rows on their way
  // (one base per batch and row in scalar registers, and offsets worked out at the loads from a number the compiler cannot
  // see through: carried along from batch to batch they would not fit the registers)
  auto request = [&](int b, int q0) {
    const int64_t bs = __builtin_amdgcn_readfirstlane(b);
    if (!vec_ok || team >= GW || bs >= n_batches || bs * GW + team >= p.C) return;
    const char *const base_pl = (const char *)(p.placement + bs * GW * N), *const base_rk = (const char *)(p.rank + bs * GW * N);
    asm volatile("" : "+v"(q0));
    const uint32_t row = (uint32_t)team * (uint32_t)N * 4u;
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const uint32_t at = row + (uint32_t)min(q0 + u * tpc, nq - 1) * 16u;
      a4[u] = *(const int4 *)(base_pl + at);
      r4[u] = *(const int4 *)(base_rk + at);
    }
  };
  request((int)blockIdx.x, tt);

  for (int b = (int)blockIdx.x; b < n_batches; b += (int)gridDim.x) {
    const int64_t c0 = (int64_t)b * GW;
    const int ng = (int)min((int64_t)GW, (int64_t)p.C - c0);
    // ---------------------------------------------------------------- ingest
    const bool mine = team < ng;
    if (tid < 64) { flagw[tid] = 0; cycw[tid] = 0; }
    if (team < GW) {
      uint32_t *const w = (uint32_t *)(lds + p.o_cand + team * p.cand_stride);
      for (int i = tt; i < cwords + lwords; i += tpc) w[i] = i < cwords ? 0u : 0xFFFFFFFFu;   // (the list follows the cells)
    }
    __syncthreads();
    // x as promised (else: another kernel's candidate), ranks inside the machine's range (eqs. (6)-(8))
    if (mine) {
      const int32_t *const pl = p.placement + (c0 + team) * N, *const rk = p.rank + (c0 + team) * N;
      uint16_t *const list = (uint16_t *)(lds + p.o_cand + team * p.cand_stride + p.o_list);
      for (int m = tt; m < P; m += tpc) list[(pairw[m] & 0xFFFFu) + (pairw[m] >> 16)] = (uint16_t)N;
      if (tt < 3) list[N + P + tt] = (uint16_t)N;
      int bits = 0;
      // (without a branch, so that the LDS reads of a round are all in flight together: an operation that cannot be put into
      // its list goes to the last entry, which nobody reads)
      const uint32_t dump = (uint32_t)n_list - 1u;
      auto place = [&](int v, bool live, int32_t a, int32_t r, uint32_t m, uint32_t pair) {
        const bool bad_pl = (uint32_t)a >= (uint32_t)P, other = (uint32_t)a != m, bad_rk = (uint32_t)r >= (pair >> 16);
        bits |= (live && bad_pl) ? kBitBadPlacement : 0;
        bits |= (live && !bad_pl && other) ? kBitOtherPlacement : 0;
        bits |= (live && !other && bad_rk) ? kBitBadRank : 0;
        list[live && !other && !bad_rk ? (pair & 0xFFFFu) + (uint32_t)r : dump] = (uint16_t)v;
      };
      if (vec_ok) {
        for (int q0 = tt; q0 < nq; q0 += kChunk * tpc) {
          if (q0 != tt) request(b, q0);                     // (the first of them were requested a batch ago)
          int qs = q0;
          asm volatile("" : "+&v"(qs));
          uint32_t mw[kChunk];
#pragma unroll
          for (int u = 0; u < kChunk; ++u) mw[u] = machw[min(qs + u * tpc, nq - 1)];
#pragma unroll
          for (int half = 0; half < kChunk; half += 2) {
            uint32_t pr[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
              for (int e = 0; e < 4; ++e) pr[u][e] = pairw[(mw[half + u] >> (8 * e)) & 0xFF];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const int q = qs + (half + u) * tpc;
              const int32_t av[4] = {a4[half + u].x, a4[half + u].y, a4[half + u].z, a4[half + u].w};
              const int32_t rv[4] = {r4[half + u].x, r4[half + u].y, r4[half + u].z, r4[half + u].w};
#pragma unroll
              for (int e = 0; e < 4; ++e) place(4 * q + e, q < nq, av[e], rv[e], (mw[half + u] >> (8 * e)) & 0xFF, pr[u][e]);
            }
          }
        }
      } else {
        for (int v = tt; v < N; v += tpc) {
          const uint32_t m = (machw[v >> 2] >> ((v & 3) << 3)) & 0xFF;
          place(v, true, pl[v], rk[v], m, pairw[m]);
        }
      }
      if (bits) atomicOr(&flagw[team], bits);
    }
    __syncthreads();
    // N operations into N slots: no slot left unwritten <=> every (machine, rank) slot hit exactly once
    if (mine && !(flagw[team] & (kBitBadPlacement | kBitOtherPlacement))) {
      const uint32_t *const lw = (const uint32_t *)(lds + p.o_cand + team * p.cand_stride + p.o_list);
      bool hole = false;
      const int nw = (N + P + 1) / 2;                       // (entry N + P is a terminal)
      for (int i0 = tt; i0 < nw; i0 += 8 * tpc) {
        uint32_t w[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) w[u] = lw[min(i0 + u * tpc, nw - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) hole |= (w[u] & 0xFFFFu) == 0xFFFFu || (w[u] >> 16) == 0xFFFFu;
      }
      if (hole) atomicOr(&flagw[team], kBitBadRank);
    }
    __syncthreads();

    request(b + (int)gridDim.x, tt);                         // the next batch's rows: on their way while this one is relaxed
    const bool ok = wave < W && lane_on && gi < ng && flagw[gi] == 0 && j < P;
    int32_t z = 0, peak = 0;
    if (wave < W) {
      // -------------------------------------------------------------- relaxer
      const uint32_t pair = ok ? pairw[j] : 0u, n_ops = pair >> 16;
      const uint32_t cb = (uint32_t)(uintptr_t)(ldsb + p.o_cand + (uint32_t)(gi < GW ? gi : 0) * p.cand_stride);
      auto ld16 = [](uint32_t a) -> uint32_t { return (uint32_t)*(lds_vu16_t *)(uintptr_t)a; };
      const uint32_t ob = (uint32_t)(uintptr_t)ldsb;
      const uint32_t l0 = ok ? cb + p.o_list + 2u * (pair & 0xFFFFu) : ob + p.o_book + 768u;
      const u32x4_t first = *(lds_vu32x4_t *)(uintptr_t)(ob + ld16(l0) * 16u);
      u32x4_t next = *(lds_vu32x4_t *)(uintptr_t)(ob + ld16(l0 + 2) * 16u);
      typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
      u32x2_t kd = {first.x, first.y};
      uint32_t idn = ld16(l0 + 4), lp = l0 + 6;
      uint32_t end = l0 + 6 + 2 * n_ops;                     // where lp is when the machine is through (or given up)
      uint32_t x = 0, y = 0, xa = 0, own = cb + (first.z >> 16), at = cb + (first.z & 0xFFFFu);
      int32_t lvl = (int32_t)first.w, pk = max(0, lvl);      // (an operation counts as it moves up: the order is all that matters)
      uint32_t e = *(lds_vu32_t *)(uintptr_t)at;
      const uint64_t seg0 = (Pseg == kWave) ? ~0ull : ((1ull << Pseg) - 1ull);
      const uint32_t seg_shift = (uint32_t)(g * Pseg);
      const uint32_t tm = p.limit - 1u;
      const uint64_t all = ~0ull;
      __builtin_amdgcn_s_setprio(3);
      // (every round completes an operation or gives up a candidate)
      const uint32_t max_rounds = (uint32_t)N * (uint32_t)G + (uint32_t)G + 2u;
      for (uint32_t round = 0; round < max_rounds; ++round) {
        uint64_t moved = 0;
        uint32_t turns = 16;
        asm volatile(DAGSCHED_PIPELINE_LOOP
                     : [x] "+&v"(x), [y] "+&v"(y), [e] "+&v"(e), [xa] "+&v"(xa), [own] "+&v"(own), [at] "+&v"(at), [idn] "+&v"(idn), [lp] "+&v"(lp),
                       [lvl] "+&v"(lvl), [pk] "+&v"(pk), "+&{v[40:43]}"(next), "+&{v[44:45]}"(kd), [moved] "+&s"(moved), [turns] "+&s"(turns)
                     : [cb] "v"(cb), [end] "v"(end), [lim] "s"(p.limit), [tm] "s"(tm), [ob] "s"(ob), [all] "s"(all)
                     : "vcc", "scc", "memory");
        const bool open = lp != end;
        if (__ballot(open) == 0) break;
        if (open && ((moved >> seg_shift) & seg0) == 0) {    // nothing of this candidate ran in the last step: a cycle
          atomicOr(&flagw[gi], kBitCyclic);
          end = lp;
        }
      }
      if (lp != end) atomicOr(&flagw[gi], kBitInternal);     // the bound on the rounds ran out: never expected
      __builtin_amdgcn_s_setprio(0);
      z = (int32_t)xa;
      peak = pk;
    } else {
      // -------------------------------------------------------------- checkers: a wavefront goes along the pairs for four candidates at a time
      const int n_check = (T >> 6) - W;
      for (int s0 = (wave - W) * 4; s0 < ng; s0 += n_check * 4) {
        for (int k0 = lane; k0 < p.n_pairs; k0 += kWave) {
          const uint32_t uv = p.pairs[k0];
          int32_t ru[4], rv[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int32_t *const rk = p.rank + (c0 + min(s0 + u, ng - 1)) * N;
            ru[u] = rk[uv & 0xFFFFu];
            rv[u] = rk[uv >> 16];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (ru[u] > rv[u]) cycw[min(s0 + u, ng - 1)] = 1;
        }
      }
    }
    __syncthreads();
    // ---------------------------------------------------------------- reductions and outputs
    if (wave < W) {
      const int64_t peak64 = peak * p.mem_scale + (p.base && j < P ? p.base[j] : 0);
      uint32_t over = ok && p.mem_limit && peak64 > p.mem_limit[j] ? 1u : 0u;
      for (int s = 1; s < Pseg; s <<= 1) { z = max(z, __shfl_xor(z, s, Pseg)); over |= __shfl_xor(over, s, Pseg); }
      if (lane_on && gi < ng && j < P) {
        const int64_t c = c0 + gi;
        const int bits = flagw[gi] | (over ? kBitOverMemory : 0) | (cycw[gi] ? kBitCyclic : 0);
        if ((bits & kBitOtherPlacement) && !(bits & kBitBadPlacement)) {
          if (j == 0) { const int slot = atomicAdd(p.fb_count, 1); p.fb_list[slot] = (int32_t)c; }   // the general kernel writes this candidate
        } else {
          const int flag = flag_from_bits(bits);
          const int64_t zz = (int64_t)z * p.time_scale;
          p.out.peak_mem[c * p.out.peak_stride_c + j * p.out.peak_stride_j] = flag ? -1 : peak64;
          if (j == 0) {
            p.out.makespan[c] = flag ? -1 : (int32_t)zz;
            p.out.bubble[c] = flag ? -1 : (int64_t)P * zz - p.sum_dur;
            p.out.flags[c] = flag;
          }
        }
      }
    }
    __syncthreads();                                         // the flags are reset by the next batch
  }
}
#undef DAGSCHED_FUSED_STEP
#undef DAGSCHED_PIPELINE_LOOP

// ---------------------------------------------------------------------------------------------------------------------
// The same for problems whose order lists do not fit the LDS beside the operations (bidirectional pipeline: 6144 operations, 98 KB
// of them): two launches.  The first reads the candidates' rows and writes the orders to a workspace, a segment of a multiple of
// eight entries per machine; the second keeps the operations and the cells of up to eight relaxers' candidates in the LDS (one
// workgroup per CU, 32 candidates of the bidirectional pipeline where the ring kernel holds eight) and streams the orders past
// them: a thread per machine copies eight entries at a time into a ring of 32.
// Bidirectional pipeline, 6144 operations, 16384 candidates: 1180 us with the ring kernel (two relaxers a CU, fed
// by wavefronts that look up placements and delays), 418 here: ingest 183 us (806 MB read and 206 written, 5.5 TB/s), relaxation 234 in two rounds, in
// which the LDS that eight relaxers and four feeders share is busy 58 % of the time (40 % of that bank conflicts) and the VALU 51 %.

struct PipelineIngest {
  int32_t N, P, C;
  const uint8_t *machine;              // [N rounded up to 4] the shared placement
  const int32_t *seg;                  // [P + 1] first entry of machine j's segment, a multiple of 8
  const int32_t *count;                // [P] its operations
  const uint32_t *pairs;               // as in PipelineParams
  int32_t n_pairs;
  const int32_t *placement, *rank;     // [C][N]
  uint16_t *lists;                     // [C][row]
  int64_t row;
  int32_t *bad;                        // [C] flag bits
  int32_t *fb_count;                   // two words, set to 0 for the launches behind (as a launch of its own that took 4 us)
  uint32_t o_rank, team_stride, o_book, total;      // LDS: per candidate its lists and at o_rank its ranks, then the rest
};

// Workgroups of T threads, K candidates each, a team of T / K threads to a candidate.  What bounds it is HBM for large candidates and the workgroups
// themselves for small ones: with 256 threads to every candidate, 240 operations take 2.6 ns a candidate (at 5 TB/s 0.4).  So T and K follow
// the number of operations.
// Both launches, us, 256 threads to a candidate and this shape: 4 operations on 2 machines, 262144 candidates 564 and 34 (ring kernel 71); 64 on 4, 65536: 164 and 35
// (65); 240 on 2, 65536: 180 and 80 (146).  T = 64, 128, 256: 768 on 8, 65536: 193, 225, 284; 1200 on 8, 20000: 120, 121, 138; 1536 on 8, 20000: 151, 149, 168;
// 3072 on 16, 20000: 347, 314, 314; 3840 on 16, 20000: 443, 400, 390; 6144 on 16, 4096: 197, 172, 158.
struct PipelineIngestShape { int threads, teams; };
inline PipelineIngestShape pipeline_ingest_shape(int N, int C) {   // (few candidates: 1024 operations on 32 machines, 1024 candidates 30.3 us with 64, 29.0 with 256)
  return N > 3072 || (N > 768 && C <= 1280) ? PipelineIngestShape{256, 1}
       : N > 1280 ? PipelineIngestShape{128, 1} : PipelineIngestShape{64, N > 128 ? 1 : N > 64 ? 2 : N > 32 ? 4 : N > 16 ? 8 : 16};
}

template <int T, int K>
__global__ __launch_bounds__(T) void pipeline_ingest_kernel(PipelineIngest p) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int kTeam = T / K, kChunk = 4;
  const int tid = threadIdx.x, team = K == 1 ? 0 : tid / kTeam, tt = K == 1 ? tid : tid % kTeam;
  const int N = p.N, P = p.P, row = (int)p.row;
  uint16_t *const list = (uint16_t *)(lds + team * p.team_stride), *const rank16 = (uint16_t *)(lds + team * p.team_stride + p.o_rank);
  int32_t *const seg = (int32_t *)(lds + p.o_book), *const count = seg + 64, *const flag = count + 64 + team;
  const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;   // (a grid of one dimension holds fewer than 2^32 threads)
  const int64_t c = block * K + team;
  if (K == 1 && c >= p.C) return;
  const bool on = K == 1 || c < p.C;                        // (a team without a candidate goes along for the barriers)
  const int32_t *const pl = p.placement + (on ? c : 0) * N, *const rk = p.rank + (on ? c : 0) * N;
  const bool vec = ((N & 3) == 0) && ((((uintptr_t)p.placement) | ((uintptr_t)p.rank)) & 15) == 0;
  const int nq = N >> 2;
  const uint32_t *const machw = (const uint32_t *)p.machine;
  int4 a4[kChunk], r4[kChunk];
  auto request = [&](int q0) {
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      a4[u] = ((const int4 *)pl)[min(q0 + u * kTeam, nq - 1)];
      r4[u] = ((const int4 *)rk)[min(q0 + u * kTeam, nq - 1)];
    }
  };
  if (vec) request(tt);
  if (tid < 64) { seg[tid] = tid < P ? p.seg[tid] : 0; count[tid] = tid < P ? p.count[tid] : 0; }
  if (tt == 0) *flag = 0;
  if (tid < 2 && block == 0) p.fb_count[tid] = 0;
  for (int i = tt; i < row / 2; i += kTeam) ((uint32_t *)list)[i] = 0xFFFFFFFFu;
  __syncthreads();
  int bits = 0;
  if (on) {
    auto place = [&](int v, int32_t a, int32_t r, uint32_t m) {
      const bool bad_pl = (uint32_t)a >= (uint32_t)P, other = (uint32_t)a != m, bad_rk = (uint32_t)r >= (uint32_t)count[m];
      bits |= bad_pl ? kBitBadPlacement : other ? kBitOtherPlacement : bad_rk ? kBitBadRank : 0;
      rank16[v] = (uint16_t)r;
      if (!other && !bad_rk) list[seg[m] + r] = (uint16_t)v;
    };
    if (vec) {
      for (int q0 = tt; q0 < nq; q0 += kChunk * kTeam) {
        int4 a[kChunk], r[kChunk];
#pragma unroll
        for (int u = 0; u < kChunk; ++u) { a[u] = a4[u]; r[u] = r4[u]; }
        if (q0 + kChunk * kTeam < nq) request(q0 + kChunk * kTeam);
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
          const int q = q0 + u * kTeam;
          if (q >= nq) break;
          const uint32_t m = machw[q];
          place(4 * q, a[u].x, r[u].x, m & 0xFF); place(4 * q + 1, a[u].y, r[u].y, (m >> 8) & 0xFF);
          place(4 * q + 2, a[u].z, r[u].z, (m >> 16) & 0xFF); place(4 * q + 3, a[u].w, r[u].w, m >> 24);
        }
      }
    } else {
      for (int v = tt; v < N; v += kTeam) place(v, pl[v], rk[v], (machw[v >> 2] >> ((v & 3) << 3)) & 0xFF);
    }
    for (int j = tt; j < P; j += kTeam)                     // behind a machine's operations: the one that is never ready
      for (int i = seg[j] + count[j]; i < (j + 1 < P ? seg[j + 1] : row); ++i) list[i] = (uint16_t)N;
    if (bits) atomicOr(flag, bits);
  }
  __syncthreads();
  if (on && !(*flag & (kBitBadPlacement | kBitOtherPlacement | kBitBadRank))) {
    // N operations into N slots: no slot left unwritten <=> every (machine, rank) slot hit exactly once
    bits = 0;
    uint4 *const out = (uint4 *)(p.lists + c * p.row);
    for (int i = tt; i < row / 8; i += kTeam) {
      const uint4 w = ((const uint4 *)list)[i];
      auto hole = [](uint32_t x) { return (x & 0xFFFFu) == 0xFFFFu || (x >> 16) == 0xFFFFu; };
      if (hole(w.x) || hole(w.y) || hole(w.z) || hole(w.w)) bits |= kBitBadRank;
      out[i] = w;
    }
    // operations of one machine in the order of B
#pragma unroll 4
    for (int k = tt; k < p.n_pairs; k += kTeam) {
      const uint32_t uv = p.pairs[k];
      if (rank16[uv & 0xFFFFu] > rank16[uv >> 16]) bits |= kBitCyclic;
    }
    if (bits) atomicOr(flag, bits);
  }
  __syncthreads();
  if (on && tt == 0) p.bad[c] = *flag;
}

struct PipelineStream {
  int32_t N, P, Pseg, log_pseg, G, W, feeders, C;
  const uint4 *ops;                    // [N + 1] as in PipelineParams
  const int32_t *seg, *count;          // as in PipelineIngest
  const uint16_t *lists;
  int64_t row;
  const int32_t *bad;
  int64_t mem_scale;
  const int64_t *base, *mem_limit;
  int64_t sum_dur;
  int32_t time_scale;
  uint32_t limit, spin_cap;
  int32_t *fb_count, *fb_list;
  uint32_t cell_stride, o_cells, o_ring, o_fed, o_loaded, o_book, total;   // LDS: operations at 0, then these
  OutPtrs out;
};

constexpr uint32_t kPipelineRing = 64;                      // bytes of a lane's ring: 32 entries

// Eight steps where the entries for them are there, else two, one block after the other (at most `turns`) as long as there are entries and
// something ran in a block's last step.
#define DAGSCHED_STREAM_LOOP                                                                                                    \
  "s_waitcnt lgkmcnt(0)\n"                                                                                                      \
  ".Lstream%=:\n\t"                                                                                                             \
  "v_sub_u32 %[x], %[fed], %[lp]\n\t"                                                                                          \
  "v_cmp_gt_i32 vcc, 16, %[x]\n\t"                                                                                             \
  "s_cbranch_vccz .Lstream_eight%=\n\t"                                                                                        \
  "v_cmp_gt_i32 vcc, 4, %[x]\n\t"                                                                                              \
  "s_cbranch_vccnz .Lstream_end%=\n\t"                                                                                         \
  "ds_read_b32 %[fed], %[fedat]\n\t" DAGSCHED_STREAM_STEP DAGSCHED_STREAM_STEP                                                 \
  "s_branch .Lstream_done%=\n"                                                                                                 \
  ".Lstream_eight%=:\n\t"                                                                                                       \
  "ds_read_b32 %[fed], %[fedat]\n\t"                                                                                           \
  DAGSCHED_STREAM_STEP DAGSCHED_STREAM_STEP DAGSCHED_STREAM_STEP DAGSCHED_STREAM_STEP                                           \
  DAGSCHED_STREAM_STEP DAGSCHED_STREAM_STEP DAGSCHED_STREAM_STEP DAGSCHED_STREAM_STEP                                           \
  ".Lstream_done%=:\n\t"                                                                                                        \
  "s_mov_b64 %[moved], vcc\n\t"                                                                                                \
  "ds_write_b32 %[loadedat], %[lp]\n\t"                                                                                        \
  "s_sub_u32 %[turns], %[turns], 1\n\t"                                                                                        \
  "s_cmp_eq_u64 %[moved], 0\n\t"                                                                                               \
  "s_cbranch_scc1 .Lstream_end%=\n\t"                                                                                          \
  "s_cmp_lg_u32 %[turns], 0\n\t"                                                                                               \
  "s_cbranch_scc1 .Lstream%=\n"                                                                                                \
  ".Lstream_end%=:\n\t"                                                                                                         \
  "s_waitcnt lgkmcnt(0)"

__global__ __launch_bounds__(1024) void relax_stream_kernel(PipelineStream p) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int T = (int)blockDim.x;                            // 64 * (W + feeders)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = p.N, P = p.P, Pseg = p.Pseg, G = p.G, W = p.W;
  lds_byte_t *const ldsb = (lds_byte_t *)lds;
  const uint32_t ob = (uint32_t)(uintptr_t)ldsb;
  constexpr uint32_t kAll = 0x40000000u;
  const int64_t c0 = (int64_t)blockIdx.x * G * W;
  const int g = lane >> p.log_pseg, j = lane & (Pseg - 1);
  // machine of relaxer w's lane: its candidate is there and well-formed, and it has operations
  auto count_of = [&](int w) -> int32_t {
    const int64_t c = c0 + (int64_t)w * G + g;
    return lane < G * Pseg && j < P && c < p.C && p.bad[c] == 0 ? p.count[j] : 0;
  };
  for (int i = tid; i <= N; i += T) ((uint4 *)lds)[i] = p.ops[i];
  for (int i = tid; i < (int)(G * W * p.cell_stride / 4); i += T) ((uint32_t *)(lds + p.o_cells))[i] = 0;
  for (int w = wave; w < W; w += T >> 6) {
    ((uint32_t *)(lds + p.o_fed))[w * kWave + lane] = count_of(w) ? 0u : kAll;
    ((uint32_t *)(lds + p.o_loaded))[w * kWave + lane] = 0u;
  }
  if (tid < 4) ((uint16_t *)(lds + p.o_book))[tid] = (uint16_t)N;   // an order for lanes without one
  if (tid == 0) *(uint32_t *)(lds + p.o_book + 8) = kAll;           // ... of which all is there
  __syncthreads();

  if (wave < W) {
    // ---------------------------------------------------------------- relaxer
    const int32_t n_ops = count_of(wave);
    const bool ok = n_ops > 0;
    const bool lane_on = lane < G * Pseg;
    const uint32_t cb = ob + p.o_cells + (uint32_t)(wave * G + (lane_on ? g : 0)) * p.cell_stride;
    const uint32_t ring = ob + p.o_ring + (uint32_t)(wave * kWave + lane) * kPipelineRing;   // (a multiple of its size)
    uint32_t fedat = ob + p.o_fed + (uint32_t)(wave * kWave + lane) * 4u, loadedat = ob + p.o_loaded + (uint32_t)(wave * kWave + lane) * 4u;
    auto ld16 = [](uint32_t a) -> uint32_t { return (uint32_t)*(lds_vu16_t *)(uintptr_t)a; };
    uint32_t fed = 0, round = 0;
    for (;; ++round) {                                       // the first entries of every lane
      fed = *(lds_vu32_t *)(uintptr_t)fedat;
      if (__ballot(fed < 16u) == 0 || round >= p.spin_cap) break;
      __builtin_amdgcn_s_sleep(1);
    }
    const uint32_t l0 = ok ? ring : ob + p.o_book;
    const u32x4_t first = *(lds_vu32x4_t *)(uintptr_t)(ob + ld16(l0) * 16u);
    u32x4_t next = *(lds_vu32x4_t *)(uintptr_t)(ob + ld16(l0 + 2) * 16u);
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    u32x2_t kd = {first.x, first.y};
    uint32_t idn = ld16(l0 + 4), lp = 6u, end = 6u + 2u * (uint32_t)n_ops;
    uint32_t x = 0, y = 0, xa = 0, own = cb + (first.z >> 16), at = cb + (first.z & 0xFFFFu);
    int32_t lvl = (int32_t)first.w, pk = max(0, lvl);        // (an operation counts as it moves up: the order is all that matters)
    uint32_t e = *(lds_vu32_t *)(uintptr_t)at;
    const uint64_t segmask = ((Pseg == kWave) ? ~0ull : ((1ull << Pseg) - 1ull)) << ((lane_on ? g : 0) * Pseg);
    const uint32_t tm = p.limit - 1u;
    const uint64_t all = ~0ull;
    int halted = 0;
    bool expired = true;
    __builtin_amdgcn_s_setprio(3);
    for (; round < p.spin_cap; ++round) {
      uint64_t moved = ~0ull;
      uint32_t turns = 32;
      asm volatile(DAGSCHED_STREAM_LOOP
                   : [x] "+&v"(x), [y] "+&v"(y), [e] "+&v"(e), [xa] "+&v"(xa), [own] "+&v"(own), [at] "+&v"(at), [idn] "+&v"(idn), [lp] "+&v"(lp),
                     [lvl] "+&v"(lvl), [pk] "+&v"(pk), [fed] "+&v"(fed), "+&{v[40:43]}"(next), "+&{v[44:45]}"(kd), [moved] "+&s"(moved), [turns] "+&s"(turns)
                   : [cb] "v"(cb), [ring] "v"(ring), [fedat] "v"(fedat), [loadedat] "v"(loadedat), [lim] "s"(p.limit), [tm] "s"(tm), [ob] "s"(ob), [all] "s"(all)
                   : "vcc", "scc", "memory");
      const bool open = lp != end;
      if (__ballot(open) == 0) { expired = false; break; }
      // in the last step nothing of the candidate ran although some machine is not through: a cycle.  (moved stays all ones where
      // there was no step.)  Its feeders are told that everything has been taken.
      if (open && (moved & segmask) == 0) {
        halted = kBitCyclic;
        end = lp;
        *(lds_vu32_t *)(uintptr_t)loadedat = kAll;
        fedat = ob + p.o_book + 8u;
        loadedat = ob + p.o_book + 12u;
      }
      if (__ballot((int32_t)(fed - lp) < 4) != 0) fed = *(lds_vu32_t *)(uintptr_t)fedat;   // (it came out for want of entries, perhaps)
    }
    if (expired && lp != end) { halted = kBitInternal; *(lds_vu32_t *)(uintptr_t)loadedat = kAll; }   // never expected
    __builtin_amdgcn_s_setprio(0);
    // ---------------------------------------------------------------- reductions and outputs
    int32_t z = (int32_t)xa;
    const int64_t peak64 = pk * p.mem_scale + (p.base && j < P ? p.base[j] : 0);
    uint32_t bits = (uint32_t)halted | (lane_on && j < P && p.mem_limit && peak64 > p.mem_limit[j] ? (uint32_t)kBitOverMemory : 0u);
    for (int s = 1; s < Pseg; s <<= 1) { z = max(z, __shfl_xor(z, s, Pseg)); bits |= __shfl_xor(bits, s, Pseg); }
    const int64_t c = c0 + (int64_t)wave * G + g;
    if (lane_on && c < p.C && j < P) {
      bits |= (uint32_t)p.bad[c];
      if ((bits & kBitOtherPlacement) && !(bits & kBitBadPlacement)) {
        if (j == 0) { const int slot = atomicAdd(p.fb_count, 1); p.fb_list[slot] = (int32_t)c; }   // the general kernel writes this candidate
      } else {
        const int flag = flag_from_bits((int)bits);
        const int64_t zz = (int64_t)z * p.time_scale;
        p.out.peak_mem[c * p.out.peak_stride_c + j * p.out.peak_stride_j] = flag ? -1 : peak64;
        if (j == 0) {
          p.out.makespan[c] = flag ? -1 : (int32_t)zz;
          p.out.bubble[c] = flag ? -1 : (int64_t)P * zz - p.sum_dur;
          p.out.flags[c] = flag;
        }
      }
    }
  } else {
    // ---------------------------------------------------------------- feeders: relaxers f, f + feeders, a thread per lane
    constexpr int kPer = 2;
    const int f = wave - W;
    uint32_t k[kPer], n[kPer];                               // next chunk of eight entries, and how many there are
    const uint4 *from[kPer];
    uint4 held[kPer];
    bool asked[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int w = f + u * p.feeders;
      const bool on = w < W && count_of(w < W ? w : 0) > 0;
      k[u] = 0;
      n[u] = on ? (uint32_t)((j + 1 < P ? p.seg[j + 1] : (int32_t)p.row) - p.seg[j]) / 8u : 0u;
      from[u] = (const uint4 *)(p.lists + (on ? (c0 + (int64_t)w * G + g) * p.row + p.seg[j] : 0));
      held[u] = make_uint4(0, 0, 0, 0);
      asked[u] = false;
    }
    for (uint32_t it = 0; it < p.spin_cap; ++it) {
      bool any = false;
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const uint32_t at = (uint32_t)((f + u * p.feeders) * kWave + lane);
        if (asked[u]) {
          *(lds_vu32x4_t *)(ldsb + p.o_ring + at * kPipelineRing + ((k[u] * 16u) & (kPipelineRing - 1u))) = u32x4_t{held[u].x, held[u].y, held[u].z, held[u].w};
          ++k[u];
          *(lds_vu32_t *)(ldsb + p.o_fed + at * 4u) = k[u] == n[u] ? kAll : k[u] * 16u;   // after the entries
        }
        asked[u] = k[u] < n[u] && (int32_t)((k[u] + 1u) * 16u - *(lds_vu32_t *)(ldsb + p.o_loaded + at * 4u)) <= (int32_t)kPipelineRing;
        if (asked[u]) held[u] = from[u][k[u]];
        any = any || k[u] < n[u];
      }
      if (__ballot(any) == 0) break;
      if (__ballot(asked[0] || asked[kPer - 1]) == 0) __builtin_amdgcn_s_sleep(2);
    }
  }
}
#undef DAGSCHED_STREAM_STEP
#undef DAGSCHED_PIPELINE_STEP
#undef DAGSCHED_STREAM_LOOP

}  // namespace dagsched_dev
