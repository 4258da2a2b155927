// Start and end times of ONE schedule (dagsched_schedule), any problem the library takes: one workgroup, one launch.
//
// What bounds it is the dependent chain: one candidate has as many sequential steps as its combined graph (DAG edges
// plus chain edges) has operations on its longest path, and nothing else on the GPU can help.  So one wavefront, the
// RELAXER, steps as fast as an LDS round trip allows and never touches anything but LDS, and eight HELPER wavefronts
// look up in time what it needs (order list, predecessors, placements, delays: four dependent L2 round trips).
//
//   relaxer   R = min(4, 64 / P rounded up to a power of two) lanes per machine (beyond 32 machines two, in two wavefronts of 32
//             machines each, which see of each other what the end times say), which hold consecutive operations of it, each polling
//             up to four predecessors of its own.  The end of one goes on to the next through a DPP move within the step, so that a
//             machine runs up to R operations a step (as the ring kernel's lanes do: the head's x_acc is finite, the others' kNever or more).
//             Operations with more predecessors are split into consecutive parts.
//   helpers   a team of 512 / Pseg threads per machine packs the next operations of its list into the machine's ring.
//
// They meet at one barrier per phase of 8 to 64 steps (schedule_steps) and hand over counts only: how many parts of a
// machine's stream the relaxer has taken, how many the helpers have put into the ring (both kept twice, by the parity
// of the phase, so that nobody writes what somebody still reads).  16 steps of 270 cycles are longer than the helpers' chain of loads
// (about 2500), so one relaxer hardly ever waits where operations have one part; the 8 steps of two relaxers are a little shorter than that chain.
//
// us, while the lanes of a machine (up to eight) polled the predecessors of one operation together, and now: MoE graph, 11712 operations on
// 32 machines 265, 212 (1760 steps of 311 cycles then); its 30-layer form on 8: 353, 132; zero-bubble pipeline, 768 on 8: 48, 19;
// bidirectional pipeline, 6144 on 16: 146, 58; random graphs, 3001 on 11 and 6000 on 40: 66, 33 and 63, 49; layered graph, 50000 on 64,
// end times in the L2: 752, 647 (one lane per machine there before).  The one-wavefront int32 kernel, which polled one edge per step
// through the L2, took 4940 us for the first.
#pragma once

#include <type_traits>

#include "device_common.h"

namespace dagsched_dev {

constexpr int kBitNoChannel = 32;                          // (the evaluations leave this flag to a pass of its own)
constexpr int kScheduleHelpers = 8;                        // wavefronts
constexpr int schedule_threads(int relaxers) { return (relaxers + 1 + kScheduleHelpers) * kWave; }   // relaxers, accountant, helpers
// Steps of a phase: what the helpers need to bring the next operations, a thread each.  16; beyond 32 machines, with two relaxers, 8 unless most operations have several
// parts; more where they have many, for a helper looks up an operation's parts a few at a time.  Random graphs, us: 24000 operations of three
// predecessors on 64 machines, 8 steps 219; 2000 of eight on 64, 8 steps 77, 16 57; 2000 of 16 on 32, 16 steps 214, 32 152; 3000 of 16 on 64, 16 steps 137, 32 103;
// 2000 of 40 on 8, 16 steps 775, 32 432, 64 476; 2000 of 80 on 8, 32 steps 1428, 64 1242; 3000 of 200 on 5, 32 steps 15100, 64 11550.
inline int32_t schedule_steps(int relaxers, int32_t n_nodes, int32_t n_red) {
  const int64_t n = n_nodes;
  return n_red > 64 * n ? 64 : n_red > 8 * n ? 32 : relaxers == 1 || n_red > 4 * n ? 16 : 8;
}

struct ScheduleParams {
  int32_t N, P, Pseg, n_red;
  int32_t slots;                       // ring slots per lane: 8, 16 or 32
  int32_t steps;                       // of a phase, a multiple of 8 (with one relaxer of 16)
  const int32_t *pred_ptr, *pred_idx;  // predecessor CSR of B (for the channels)
  const int32_t *red_ptr, *red_idx;    // [N + 1], [n_red] the same without the edges that other paths imply
  const int32_t *dur, *comm;           // [N], [P*P] (0 where the pair has no channel)
  const uint64_t *no_channel;          // [P] bit b of word a: no channel a -> b, or NULL
  const int64_t *mem_delta, *weight, *mem_limit;
  const int32_t *placement, *rank;     // [N]
  int32_t *list;                       // [N] scratch: order lists, machine after machine
  int32_t *cells;                      // [N] scratch for the end times when they do not fit the LDS
  int32_t *start, *end, *flag;         // outputs
  uint32_t o_ring, o_comm, o_book;     // LDS: end times (or nothing) at 0, then these
};

// bytes of dynamic LDS: end times, rings, delays, bookkeeping
constexpr uint32_t kScheduleBook = 64 * 4 * 7 + 64;
inline uint32_t schedule_lds(ScheduleParams *p, bool lds_cells, int relaxers) {
  uint32_t at = lds_cells ? ((uint32_t)p->N + 2u + 3u) / 4u * 16u : 16u;
  p->o_ring = at;
  at += (uint32_t)p->slots * (uint32_t)(relaxers * kWave) * 32u;
  p->o_comm = at;
  at += ((uint32_t)p->P * (uint32_t)p->P + 3u) / 4u * 16u;
  p->o_book = at;
  return at + kScheduleBook;
}

// R lanes per machine, RW relaxers; LDSC: end times in LDS, else in the scratch row (L2)
template <int R, bool LDSC, int RW>
__global__ __launch_bounds__(schedule_threads(RW)) void schedule_kernel(ScheduleParams p) {
  extern __shared__ __align__(16) unsigned char lds[];
  lds_byte_t *const ldsb = (lds_byte_t *)lds;
  const int tid = threadIdx.x, lane = tid & 63, T = schedule_threads(RW);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = p.N, P = p.P, Pseg = p.Pseg;
  constexpr uint32_t kNever = 0x80000000u;
  int32_t *const comm = (int32_t *)(lds + p.o_comm);
  int32_t *const cnt = (int32_t *)(lds + p.o_book);          // [64] operations per machine
  int32_t *const off = cnt + 64;                             // [64] start of the machine in the list
  uint32_t *const taken = (uint32_t *)(off + 64);            // [2][64] parts the relaxer has taken from the ring
  uint32_t *const fed = taken + 128;                         // [2][64] parts in the ring so far, | 0x80000000: that is all
  int32_t *const s_flag = (int32_t *)(fed + 128);
  int32_t *const s_done = s_flag + 1;                        // [2][2] of a relaxer: 1 = through, 2 = stuck, 3 = the bound on the phases, 0 = on its way; + kMoved
  constexpr int kMoved = 4;                                  // ... something has run in this phase, or was taken
  constexpr uint32_t kRow = RW * kWave * 16u;                // bytes of a ring slot of all lanes, in either plane
  uint32_t *const seen = (uint32_t *)(lds + p.o_ring);       // [N bits] ingest only
  uint32_t *const cellw = (uint32_t *)lds;                   // [N + 2] end times; N: "ended at 0", N + 1: trash

  // ---------------------------------------------------------------- ingest
  if (tid < 64) { cnt[tid] = 0; taken[tid] = taken[64 + tid] = fed[tid] = fed[64 + tid] = 0; }
  if (tid == 0) { *s_flag = 0; s_done[0] = s_done[1] = s_done[2] = s_done[3] = 0; }
  for (int i = tid; i < (N + 31) / 32; i += T) seen[i] = 0;
  for (int i = tid; i < P * P; i += T) comm[i] = (i / P != i % P) ? p.comm[i] : 0;
  if (LDSC) { for (int i = tid; i < N + 2; i += T) cellw[i] = i < N ? kNever : 0u; }
  else { for (int i = tid; i < N; i += T) st_group(&p.cells[i], (int32_t)kNever); }
  // What the helpers will look up at random is read once in order, so that it waits in this XCD's L2 when they do (the
  // workgroup may land on any XCD): a helper's chain of loads took 7500 cycles without this, longer than a phase.
  {
    auto touch = [&](const int32_t *q, int n) {
      int32_t sink = 0;
#pragma unroll 8
      for (int i = tid * 32; i < n; i += T * 32) sink |= q[i];   // a word of every 128-byte line
      asm volatile("" ::"v"(sink));
    };
    touch(p.red_ptr, N + 1);
    touch(p.dur, N);
    touch(p.red_idx, p.n_red);
  }
  __syncthreads();
  // (the rows are read kBatch entries per thread at a time: a lone workgroup waits out every trip to memory)
  constexpr int kBatch = 8;
  for (int v0 = tid; v0 < N; v0 += kBatch * T) {
    int32_t m[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) m[u] = p.placement[min(v0 + u * T, N - 1)];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (v0 + u * T < N) {
        if ((uint32_t)m[u] >= (uint32_t)P) atomicOr(s_flag, kBitBadPlacement);
        else atomicAdd(&cnt[m[u]], 1);
      }
  }
  __syncthreads();
  if (wave == 0) {
    const int my = cnt[lane];
    int incl = my;
    for (int d = 1; d < kWave; d <<= 1) {
      const int t = __shfl_up(incl, d, kWave);
      if (lane >= d) incl += t;
    }
    off[lane] = incl - my;
  }
  __syncthreads();
  int bits = *s_flag;                                        // the same for every thread
  __syncthreads();
  if (!bits) {
    // every (machine, rank) slot hit exactly once: a bit per slot, over the rings
    for (int v0 = tid; v0 < N; v0 += kBatch * T) {
      int32_t m[kBatch], r[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) { const int v = min(v0 + u * T, N - 1); m[u] = p.placement[v]; r[u] = p.rank[v]; }
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (v0 + u * T < N) {
          const uint32_t slot = (uint32_t)(off[m[u]] + r[u]), bit = 1u << (slot & 31u);
          if ((uint32_t)r[u] >= (uint32_t)cnt[m[u]] || (atomicOr(&seen[slot >> 5], bit) & bit)) atomicOr(s_flag, kBitBadRank);
          else st_group(&p.list[slot], v0 + u * T);
        }
    }
    __syncthreads();
    bits = *s_flag;
    __syncthreads();
    if (!bits && p.no_channel) {                             // eqs. (9)-(10)
      for (int v = tid; v < N; v += T) {
        const int32_t b = p.placement[v];
        for (int k = p.pred_ptr[v]; k < p.pred_ptr[v + 1]; ++k) {
          const int32_t a = p.placement[p.pred_idx[k]];
          if (a != b && ((p.no_channel[a] >> b) & 1ull)) atomicOr(s_flag, kBitNoChannel);
        }
      }
      __syncthreads();
      bits = *s_flag;
      __syncthreads();
    }
  }

  // ---------------------------------------------------------------- relaxation
  if (!bits) {
    const int ring_mask = p.slots - 1;
    // how a phase has ended: 0 it goes on, 1 through, 2 nothing moved anywhere, 3.  (What a stuck relaxer waits for may have run in this very
    // phase, in the other relaxer's last step before that one was through.)
    auto phase_end = [&](uint32_t phase) -> int {
      const int a = s_done[(phase & 1) * 2], b = RW == 2 ? s_done[(phase & 1) * 2 + 1] : 1;
      const int end = (a & 3) && (b & 3) ? max(a & 3, b & 3) : 0;
      return end == 2 && ((a | b) & kMoved) ? 0 : end;
    };
    // (every phase completes a part, or takes one, or the helpers bring one)
    const uint32_t max_phases = 4u * ((uint32_t)N + (uint32_t)p.n_red) + 64u;
    int64_t level = 0, peak = 0, base = 0;
    if (wave < RW) {
      __builtin_amdgcn_s_setprio(3);
      const int place = wave * kWave + lane, m = place / R, sub = place % R;   // machines beyond P have no operations
      auto before = [](uint32_t v) -> uint32_t {             // what the lane before works out, in a ring of R
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, R == 4 ? 0x93 : 0xB1, 0xF, 0xF, true);
      };
      const bool mine = place < Pseg * R;
      lds_byte_t *const ring_lane = ldsb + p.o_ring + (uint32_t)place * 16u;   // two planes of [slot][lane] of 16 bytes
      const uint32_t plane = (uint32_t)p.slots * kRow;
      // (the end times are the first thing in the workgroup's LDS, and the kernel has no static LDS: cell v is at byte 4 v)
      auto cell = [&](uint32_t v4) -> uint32_t {
        if (LDSC) return *(lds_vu32_t *)(uintptr_t)v4;
        return (v4 >> 2) < (uint32_t)N ? (uint32_t)ld_group(&p.cells[v4 >> 2]) : 0u;
      };
      const uint32_t trash = ((uint32_t)N + 1u) * 4u;
      uint32_t t = 0, x_acc = sub == 0 ? 0u : kNever;
      uint64_t have = 0;                                     // lanes that hold an operation
      bool all_fed = !mine;
      u32x4_t a = {(uint32_t)N * 0x10001u, (uint32_t)N * 0x10001u, 0u, trash}, d = {0u, 0u, 0u, 0u};
      u32x4_t na = a, nd = d;                                // content of ring slot t
      uint32_t e0 = 0, e1 = 0, e2 = 0, e3 = 0;
      int idle_phases = 0;
      for (uint32_t phase = 0; ; ++phase) {
        const uint32_t f = fed[((phase + 1) & 1) * 64 + (mine ? m : 0)];
        const uint32_t avail = mine ? ((f & 0x7FFFFFFFu) + (uint32_t)(R - 1 - sub)) / R : 0u;   // parts of this lane in its ring
        all_fed = !mine || (f >> 31);
        uint64_t moved = 0;
        if (have | __ballot(t < avail)) {
          {
            lds_byte_t *const sp = ring_lane + (t & (uint32_t)ring_mask) * kRow;
            na = *(lds_vu32x4_t *)sp; nd = *(lds_vu32x4_t *)(sp + plane);
          }
          constexpr int kUnroll = RW == 1 ? 16 : 8;          // (the jump back costs 1 %)
          for (int i = 0; i < p.steps; i += kUnroll) {
#pragma unroll
            for (int step = 0; step < kUnroll; ++step) {
              // (a time of kNever or more plus a delay and the durations of R operations stays below 2^32: the library accepts no
              // problem whose times could pass INT32_MAX)
              const uint32_t polled = max(max(max(e0 + d.x, e1 + d.y), e2 + d.z), e3 + d.w);
              const uint32_t at = lane_bit(have) ? polled : kNever;
              uint32_t b = x_acc, y = max(at, b) + a.z;
#pragma unroll
              for (int k = 1; k < R; ++k) { b = min(b, before(y)); y = max(at, b) + a.z; }
              const uint64_t ran_m = __ballot(y < kNever);
              const bool ran = lane_bit(ran_m);
              // the machine is busy until y (chain edge, eq. (7))
              const uint32_t last = before(y);
              x_acc = ran ? max(x_acc, last) : b;
              if (LDSC) *(lds_vu32_t *)(uintptr_t)(ran ? a.w : trash) = y;
              else if (ran && a.w != trash) st_group(&p.cells[a.w >> 2], (int32_t)y);
              const uint64_t take_m = (ran_m | ~have) & __ballot(t < avail);
              const bool take = lane_bit(take_m);
              have = (have & ~ran_m) | take_m;
              moved |= ran_m | take_m;
              // the end times for the next step are requested first, everything else happens while they are on their way
              a.x = take ? na.x : a.x; a.y = take ? na.y : a.y;
              e0 = cell(lo16_x4(a.x)); e1 = cell(hi16_x4(a.x)); e2 = cell(lo16_x4(a.y)); e3 = cell(hi16_x4(a.y));
              __builtin_amdgcn_sched_barrier(0);
              a.z = take ? na.z : a.z; a.w = take ? na.w : a.w;
              d.x = take ? nd.x : d.x; d.y = take ? nd.y : d.y; d.z = take ? nd.z : d.z; d.w = take ? nd.w : d.w;
              t += take ? 1u : 0u;
              lds_byte_t *const sp = ring_lane + (t & (uint32_t)ring_mask) * kRow;
              na = *(lds_vu32x4_t *)sp; nd = *(lds_vu32x4_t *)(sp + plane);
            }
          }
        }
        uint32_t next = t * R + (uint32_t)sub;                 // the first part of the machine that has not been taken
#pragma unroll
        for (int s = 1; s < R; s <<= 1) next = min(next, __shfl_xor(next, s, kWave));
        if (mine && sub == 0) taken[(phase & 1) * 64 + m] = next;
        const bool held = lane_bit(have), through = !held && all_fed && t == avail;
        int done = 0;
        if (__ballot(!through) == 0) done = 1;
        // nothing moved in a whole phase, here and in the other relaxer, although every unfinished machine holds an operation: a cycle.  (End times in
        // the L2: seen in two phases on end, so that a store on its way is never taken for one)
        else if (moved == 0 && __ballot(!through && !held) == 0) { if (++idle_phases >= (LDSC ? 1 : 2)) done = 2; }
        else idle_phases = 0;
        if (!done && phase >= max_phases) done = 3;
        if (lane == 0) s_done[(phase & 1) * 2 + wave] = done | (moved ? kMoved : 0);
        __syncthreads();
        if (const int end = phase_end(phase)) {
          if (tid == 0 && end > 1) *s_flag = end == 2 ? kBitCyclic : kBitInternal;
          break;
        }
        if (RW == 2 && (s_done[(phase & 1) * 2 + (wave ^ 1)] & kMoved)) idle_phases = 0;
      }
      __builtin_amdgcn_s_setprio(0);
    } else if (wave == RW) {
      // accountant: peak of the running memory level (eqs. (17)-(19)), only asked for when there are limits
      int k = off[lane];
      const int kend = p.mem_limit ? k + cnt[lane] : k;
      auto walk = [&](int steps) {
        for (int s = 0; s < steps && __ballot(k < kend); ++s) {
          int32_t id[4];
          int64_t md[4], wt[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) id[u] = k + u < kend ? ld_group(&p.list[k + u]) : 0;
#pragma unroll
          for (int u = 0; u < 4; ++u) { md[u] = p.mem_delta[id[u]]; wt[u] = p.weight ? p.weight[id[u]] : 0; }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (k + u < kend) { level += md[u]; peak = max(peak, level); base += wt[u]; }
          k += 4;
        }
      };
      for (uint32_t phase = 0; ; ++phase) {
        walk(2);
        __syncthreads();
        if (phase_end(phase)) break;
      }
      walk(N);
      if (p.mem_limit && lane < P && base + peak > p.mem_limit[lane]) atomicOr(s_flag, kBitOverMemory);
    } else {
      const int h = tid - (RW + 1) * kWave;
      const int team = (kScheduleHelpers * kWave) / Pseg >= kWave ? kWave : (kScheduleHelpers * kWave) / Pseg;   // threads per machine, 8 .. 64
      const int m = h / team, i = h - m * team;
      const bool on = m < P;
      const uint64_t all = (team == kWave ? ~0ull : ((1ull << team) - 1ull)) << (lane & ~(team - 1));   // the lanes of this team
      const uint64_t upto = all & ((2ull << lane) - 1ull);   // ... up to this one
      int pos = on ? off[m] : 0;                             // list position of the team's next operation
      const int pend = on ? pos + cnt[m] : 0;
      uint32_t f = 0, part0 = 0;                             // parts put into the ring; parts of the operation at pos among them
      for (uint32_t phase = 0; ; ++phase) {
        const uint32_t tk = on ? taken[((phase + 1) & 1) * 64 + m] : 0u;
        const uint32_t room = on ? (uint32_t)p.slots * R - (f - tk) : 0u;
        const int k = pos + i;
        const bool valid = on && k < pend;
        const int v = valid ? ld_group(&p.list[k]) : 0;
        const int lo = valid ? p.red_ptr[v] : 0, hi = valid ? p.red_ptr[v + 1] : 0;
        const uint32_t parts = valid ? (uint32_t)max(1, (hi - lo + 3) / 4) : 0u;
        const uint32_t first = i == 0 ? part0 : 0u;
        const uint32_t n_mine = parts - (valid ? first : 0u);
        // inclusive prefix over the team, from ballots of the two low bits where those are all (a shuffle is an LDS trip)
        uint32_t incl, total;
        if (__ballot(n_mine > 3u) == 0) {
          const uint64_t b0 = __ballot(n_mine & 1u), b1 = __ballot(n_mine & 2u);
          incl = (uint32_t)(__popcll(b0 & upto) + 2 * __popcll(b1 & upto));
          total = (uint32_t)(__popcll(b0 & all) + 2 * __popcll(b1 & all));
        } else {
          incl = n_mine;
          for (int s = 1; s < team; s <<= 1) {
            const uint32_t o = __shfl_up(incl, s, team);
            if (i >= s) incl += o;
          }
          total = __shfl(incl, team - 1, team);
        }
        const uint32_t excl = incl - n_mine;
        const uint32_t n_put = excl >= room ? 0u : min(n_mine, room - excl);
        // `count` parts from the q0-th on, looked up together: each is two trips to memory, one behind the other
        auto put = [&](uint32_t q0, auto count) {
          constexpr uint32_t kTogether = decltype(count)::value;
          if (q0 >= n_put) return;
          uint32_t u[kTogether][4], dl[kTogether][4];
#pragma unroll
          for (uint32_t b = 0; b < kTogether; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int kk = lo + (int)(first + q0 + b) * 4 + e;
              u[b][e] = kk < hi ? (uint32_t)p.red_idx[kk] : (uint32_t)N;
            }
#pragma unroll
          for (uint32_t b = 0; b < kTogether; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) dl[b][e] = u[b][e] < (uint32_t)N ? (uint32_t)p.placement[u[b][e]] : 64u;
#pragma unroll
          for (uint32_t b = 0; b < kTogether; ++b)
            if (q0 + b < n_put) {
              const uint32_t part = first + q0 + b, seq = f + excl + q0 + b, slot = (seq / R) & (uint32_t)ring_mask;
              const bool last = part + 1 == parts;
              const uint32_t tail_z = last ? (uint32_t)p.dur[v] : 0u, tail_w = (last ? (uint32_t)v : (uint32_t)N + 1u) * 4u;
              uint32_t d[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) d[e] = dl[b][e] < 64u ? (uint32_t)comm[dl[b][e] * P + m] : 0u;
              lds_byte_t *const sp = ldsb + p.o_ring + slot * kRow + ((uint32_t)(m * R) + seq % R) * 16u;
              const u32x4_t wa = {u[b][0] | (u[b][1] << 16), u[b][2] | (u[b][3] << 16), tail_z, tail_w}, wd = {d[0], d[1], d[2], d[3]};
              *(lds_vu32x4_t *)sp = wa;
              *(lds_vu32x4_t *)(sp + (uint32_t)p.slots * kRow) = wd;
            }
        };
        put(0, std::integral_constant<uint32_t, 1>());
        if (__ballot(n_put > 1u) != 0) {
          if (__ballot(n_put > 2u) == 0) put(1, std::integral_constant<uint32_t, 1>());
          else put(1, std::integral_constant<uint32_t, 4>());
          for (uint32_t q = 5; __ballot(n_put > q) != 0; q += 8) put(q, std::integral_constant<uint32_t, 8>());
        }
        // how far the team got: operations that are in with all their parts, and the parts of the one that is not
        const bool whole = n_put == n_mine && valid;
        const uint32_t n_whole = (uint32_t)__popcll(__ballot(whole) & all), n_total = min(room, total);
        const uint64_t cut = __ballot(valid && !whole && n_put) & all;   // at most one thread of the team
        const uint32_t in_cut = __shfl(first + n_put, cut ? __builtin_ctzll(cut) : 0, kWave);
        const uint32_t part_next = cut ? in_cut : 0u;
        f += n_total;
        part0 = n_whole ? part_next : part0 + n_total;       // (n_whole == 0: only the team's first operation can be partly in)
        pos += (int)n_whole;
        if (i == 0) fed[(phase & 1) * 64 + m] = f | (pos >= pend ? 0x80000000u : 0u);
        __syncthreads();
        if (phase_end(phase)) break;
      }
    }
    __syncthreads();
    bits = *s_flag;
  }

  // ---------------------------------------------------------------- outputs
  // (looked for only where placement and ranks are well-formed, and then nothing was relaxed: the only bit there is)
  const int flag = bits & kBitNoChannel ? DAGSCHED_FLAG_NO_CHANNEL : flag_from_bits(bits);
#pragma unroll 4
  for (int v = tid; v < N; v += T) {
    const int32_t e = flag ? -1 : LDSC ? (int32_t)cellw[v] : ld_group(&p.cells[v]);
    const int32_t d = p.dur[v];
    p.end[v] = e;
    p.start[v] = flag ? -1 : e - d;
  }
  if (tid == 0) *p.flag = flag;
}

}  // namespace dagsched_dev
