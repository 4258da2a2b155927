// Evaluation with channel contention (Sec. III, eqs. (11)-(15)) for candidates whose channel orders follow their
// producers: the fast path beside kernel_contended.h, which takes the rest.
//
// Every transfer of a channel (a, b) is produced by an operation of machine a, and machine a runs its operations one
// after the other.  Where the transfers of every channel are ranked in the order in which machine a produces them (first
// come, first served; the messages of one operation over the same channel by the index of their edge), a transfer can be
// completed the moment its producer has ended:
//   d_k = max(e_u, free(a, b)) + comm[a][b],  free(a, b) = d_k       (eqs. (11), (13)-(15))
// so nothing ever waits for a channel (an edge inside a machine is a message over a channel of its own without delay).
// What is left is the evaluation without contention with the roles turned round: instead of polling its predecessors, an
// operation waits until the number of messages still on their way to it is 0, and whoever completes a transfer takes the
// maximum into the receiver's arrival time and one off its count (eq. (12)).
//
// One workgroup = G candidates, R lanes (g, j, r) for machine j of candidate g, arrival times and counts in LDS.  An ITEM
// is an operation together with its first R messages, or its next R messages; each lane of the machine sends one of them.
// Items are constants of the problem; a candidate orders them.
//   ingest    (all wavefronts) checks placement and ranks and writes the order of every machine's items to a workspace row.
//   RELAXER   wave 0: per step at most one item per machine.  An item is ready when its operation's count is 0 (at once when
//             it holds no operation).
//   ACCOUNTANTS two or four waves: go along the same streams 64 messages at a time: memory levels (eqs. (16)-(19)), and whether every
//             channel's transfers are ranked 0, 1, 2, ... as they come; a candidate where they are not is left to the
//             other kernel.
//   HELPERS   the other waves: look the items up and put them into rings in LDS, 16 bytes a lane, ahead of the relaxer.
// They never meet at a barrier before the end.  Item i of a lane goes to ring slot i mod slots; the last half word of the entry is
// i + slots, written last, which tells the relaxer that it is there (what the slot held before is less); the relaxer tells how
// many it has taken, plus slots, every four steps.  The R lanes of a machine have to stay in step: the delays of messages that
// share a channel are laid out for lanes that read the channel's time in the same step.  An LDS access of a wavefront need
// not be one moment for all its lanes, so what a lane reads of another wavefront's writing is never acted upon alone: an
// item is taken when the least of its lanes' tags says so, and a helper goes as far as the least of the lanes' counts.
//
// What bounds it is the chain of dependent steps (MoE graph: a candidate's longest path of operations and messages),
// each an LDS round trip and about 40 instructions of a lone wavefront.  MoE graph, 512 candidates, two workgroups of one
// candidate per CU: 609 us, which is the slowest candidate (601 us) and the second launch; 33 us of ingest and 3664 steps of
// 306 cycles at 2.27 GHz (494 us) on the average, 38 us and 4216 steps (563 us) at most.  In about one step of eight
// some machine waits for the helpers.  With one lane per machine 4377 steps (of 280), with a barrier every 17 steps 755 us,
// with the messages written to memory at ingest (262 KB a candidate) 860 us.  The kernel before took 17235 us.  Zero-bubble
// pipeline, 2048 candidates: 1030 -> 77 us (9 us of ingest, 302 steps of 312 cycles, then the accountants' last 16 us).
// A candidate that is left to the other kernel costs the ingest and the accountants' first streams: MoE graph, all channels'
// orders reversed 1199 us with the other kernel alone, 1236 us with this one in front of it.
#pragma once

#include "device_common.h"

namespace dagsched_dev {

struct TransferParams {
  int32_t N, E, P, Pseg, log_pseg, G, C;
  int32_t R;                            // lanes per machine = messages per item: 1, 2 or 4
  int32_t threads;                      // 512 where two workgroups fit a CU, else 1024
  int32_t teams;                        // candidates ingested side by side (a power of two, at most G)
  int32_t slots;                        // ring slots per lane: 16 or 32
  int32_t accountants;                  // four where the LDS has room: they are what short streams wait for (zero-bubble pipeline: 106 us with two)
  const uint32_t *first;                // [N] first item of operation v | how many << 16
  const uint2 *item;                    // [items][R] x = own operation (N: none) | receiver (N: none) << 16, y = edge
  const int32_t *dur, *comm;            // [N], [P * P] (0 where the pair has no channel)
  const int64_t *mem_delta, *weight, *mem_limit;
  int64_t sum_dur;
  const int32_t *placement, *rank, *edge_rank;   // [C][N], [C][N], [C][E]
  const uint32_t *in_degree;            // [N] a byte each
  uint16_t *stream;                     // [grid][G][row_items] items, machine after machine
  int64_t row_items;
  int32_t *fb_count, *fb_list;          // candidates left to the other kernel
  int32_t *ticket, *fb_todo;            // workgroups that are through; how many candidates are left, for the other kernel
  // LDS: arrival times at 0, then these; ingest works in the first `scratch` bytes of every team, all before o_cnt
  uint32_t acc_stride, o_free, free_stride, o_ring, o_cnt, cnt_stride, o_book, total;
  uint32_t team_stride, s_base, s_list, s_part;   // scratch of a team: placement bytes at 0, then these
  OutPtrs out_ptrs;
};

constexpr int kTransferThreads = 1024;

inline int64_t transfer_items(const int32_t *row_ptr, int n, int R) {
  int64_t items = 0;
  for (int v = 0; v < n; ++v) items += row_ptr[v + 1] > row_ptr[v] ? (row_ptr[v + 1] - row_ptr[v] + R - 1) / R : 1;
  return items;
}

// Shape for a problem, or false when it does not fit (the other kernel then does everything).
inline bool transfer_plan(TransferParams *p, int64_t n_cand, int n_cu, uint32_t lds_max) {
  const uint32_t N = (uint32_t)p->N, E = (uint32_t)p->E, P = (uint32_t)p->P;
  if ((uint64_t)N + E > 65000u) return false;            // item numbers and tags are 16-bit
  auto up = [](uint32_t x, uint32_t a) { return (x + a - 1) / a * a; };
  p->acc_stride = up(4 * (N + 1), 16);
  p->free_stride = up(4 * P * P, 16);
  p->cnt_stride = up(N + 1, 16);
  p->s_base = up(N, 16);
  p->s_list = p->s_base + up(2 * N, 16);
  p->s_part = p->s_list + up(2 * N, 16);
  p->team_stride = p->s_part + 64;
  // Two lanes per machine where operations send more than one message: the MoE graph (2.2 out-edges per operation) then
  // takes 3664 steps instead of 4377, a pipeline (1.25) as many as before with half the candidates in a wavefront.
  p->R = 2 * (uint64_t)E > 3 * (uint64_t)N && p->Pseg <= kWave / 2 ? 2 : 1;
  for (int G = kWave / (p->Pseg * p->R); G >= 1; G >>= 1) {
    for (int slots : {32, 16}) {
      uint32_t at = (uint32_t)G * p->acc_stride;
      p->o_free = at; at += (uint32_t)G * p->free_stride;
      p->o_ring = at; at += (uint32_t)slots * kWave * 16u;
      const uint32_t room = at > p->team_stride ? at : p->team_stride;
      at = room;
      p->o_cnt = at; at += (uint32_t)G * p->cnt_stride;
      p->o_book = at; at += 64 * 4 * (slots == 32 ? 10 : 8) + 16;
      p->total = at;
      p->G = G; p->slots = slots; p->accountants = slots == 32 ? 4 : 2;
      const int wgs = (int)(lds_max / at);
      if (wgs < 1 || (wgs < 2 && slots == 32 && (int)(lds_max / (at - 16 * kWave * 16u)) >= 2 && room > p->team_stride + 16 * kWave * 16u)) continue;   // (shallow rings if that fits a second workgroup)
      p->threads = wgs >= 2 ? 512 : 1024;
      // (small batches: rather more workgroups than full wavefronts, as long as CUs would stay empty)
      if (G > 1 && (n_cand + G - 1) / G < (int64_t)n_cu * (wgs >= 2 ? 2 : 1)) break;
      p->teams = 1;
      while (p->teams < G && (uint32_t)p->teams * 2u * p->team_stride <= room && p->threads / (p->teams * 2) >= kWave) p->teams *= 2;
      while (E > N && p->R < 4 && G * p->Pseg * p->R * 2 <= kWave) p->R *= 2;   // (lanes that would be idle)
      return true;
    }
  }
  return false;
}

// R: lanes per machine.  Ring entry of a lane: x = own operation | receiver << 16 (as LDS addresses of arrival times / 4),
// y = duration, z = delay (negative: no message), w = channel (likewise) | tag << 16.
template <int R>
__global__ __launch_bounds__(kTransferThreads) void transfer_kernel(TransferParams p) {
  extern __shared__ __align__(16) unsigned char lds[];
  lds_byte_t *const ldsb = (lds_byte_t *)lds;
  const int tid = threadIdx.x, lane = tid & 63, T = (int)blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = p.N, E = p.E, P = p.P, Pseg = p.Pseg, G = p.G;
  int32_t *const mcount = (int32_t *)(lds + p.o_book);       // [64] operations per lane
  int32_t *const off = mcount + 64;                          // [64] list position of the machine's first operation
  uint32_t *const item0 = (uint32_t *)(off + 64);            // [64] the lane's first item, and its number of items
  uint32_t *const items = item0 + 64;
  uint32_t *const taken = items + 64;                        // [64] tag of the item the relaxer takes next
  int32_t *const flagw = (int32_t *)(taken + 64);            // [64] (G used)
  uint32_t *const seenw = (uint32_t *)(flagw + 64);          // [accountants][64] transfers so far, by receiving machine
  int32_t *const misc = (int32_t *)(seenw + 64 * p.accountants);            // [0] 1: the relaxer is through
  constexpr uint32_t kNoMessage = 0x80000000u;
  constexpr int kBitOrder = 128;                             // internal: some channel's order does not follow the producers

  const int64_t n_groups = ((int64_t)p.C + G - 1) / G;
  for (int64_t group = blockIdx.x; group < n_groups; group += gridDim.x) {
    const int64_t c0 = group * G;
    const int ng = (int)min((int64_t)G, (int64_t)p.C - c0);
    uint16_t *const stream = p.stream + (int64_t)blockIdx.x * G * p.row_items;

    // ---------------------------------------------------------------- ingest
    const int tpc = T / p.teams, team = tid / tpc, tt = tid - team * tpc;
    unsigned char *const sc = lds + (uint32_t)team * p.team_stride;
    uint8_t *const machine = sc;                             // [N]
    uint16_t *const base = (uint16_t *)(sc + p.s_base);      // [N] by list position: items of the operation there, then its first item
    uint16_t *const list = (uint16_t *)(sc + p.s_list);      // [N] operations, machine after machine
    uint32_t *const part = (uint32_t *)(sc + p.s_part);      // [16] sums of the team's wavefronts
    if (tid < 64) { mcount[tid] = 0; flagw[tid] = 0; items[tid] = 0; item0[tid] = 0; }
    __syncthreads();
    for (int g0 = 0; g0 < G; g0 += p.teams) {
      const int gg = g0 + team;
      const bool live = gg < ng;
      const int64_t c = c0 + (live ? gg : 0);
      const int32_t *const pl = p.placement + c * N, *const rk = p.rank + c * N;
      int32_t *const mc = mcount + gg * Pseg, *const mo = off + gg * Pseg;
      uint32_t *const cntw = (uint32_t *)(lds + p.o_cnt + (uint32_t)gg * p.cnt_stride);
      constexpr int kB = 4;
      if (live) {
        for (int i = tt; i < (N + 1) / 2; i += tpc) ((uint32_t *)list)[i] = 0xFFFFFFFFu;
        for (int i = tt; i < (N + 4) / 4; i += tpc) cntw[i] = 4 * i < N ? p.in_degree[i] : 0u;   // every message is on its way
        // x in range (eq. (6)), operations per machine
        for (int v0 = tt; v0 < N; v0 += kB * tpc) {
          int32_t m[kB];
#pragma unroll
          for (int u = 0; u < kB; ++u) m[u] = pl[min(v0 + u * tpc, N - 1)];
#pragma unroll
          for (int u = 0; u < kB; ++u)
            if (v0 + u * tpc < N) {
              if ((uint32_t)m[u] >= (uint32_t)P) { atomicOr(&flagw[gg], kBitBadPlacement); m[u] = 0; }
              else atomicAdd(&mc[m[u]], 1);
              machine[v0 + u * tpc] = (uint8_t)m[u];
            }
        }
      }
      __syncthreads();
      if (wave == 0) {
        const int my = lane < G * Pseg ? mcount[lane] : 0, jj = lane & (Pseg - 1);
        int incl = my;
        for (int d = 1; d < Pseg; d <<= 1) {
          const int t = __shfl_up(incl, d, Pseg);
          if (jj >= d) incl += t;
        }
        off[lane] = incl - my;
      }
      __syncthreads();
      const bool well = live && !(flagw[gg] & kBitBadPlacement);
      if (well) {
        // ranks in range (eqs. (7)-(8))
        for (int v0 = tt; v0 < N; v0 += kB * tpc) {
          int32_t r[kB];
#pragma unroll
          for (int u = 0; u < kB; ++u) r[u] = rk[min(v0 + u * tpc, N - 1)];
#pragma unroll
          for (int u = 0; u < kB; ++u) {
            const int v = v0 + u * tpc;
            if (v >= N) break;
            const int a = machine[v];
            if ((uint32_t)r[u] >= (uint32_t)mc[a]) atomicOr(&flagw[gg], kBitBadRank);
            else list[mo[a] + r[u]] = (uint16_t)v;
          }
        }
      }
      __syncthreads();
      const bool ranked = well && !(flagw[gg] & kBitBadRank);
      if (ranked) {                                          // items by list position; a slot nobody wrote: bad ranks
        for (int k0 = tt; k0 < N; k0 += kB * tpc) {
          uint32_t v[kB], o[kB];
#pragma unroll
          for (int u = 0; u < kB; ++u) v[u] = list[min(k0 + u * tpc, N - 1)];
#pragma unroll
          for (int u = 0; u < kB; ++u) o[u] = p.first[min(v[u], (uint32_t)N - 1u)];
#pragma unroll
          for (int u = 0; u < kB; ++u)
            if (k0 + u * tpc < N) {
              if (v[u] == 0xFFFFu) atomicOr(&flagw[gg], kBitBadRank);
              base[k0 + u * tpc] = (uint16_t)(o[u] >> 16);
            }
        }
      }
      __syncthreads();
      // exclusive sums, a block of consecutive entries per thread
      const int ob = (N + tpc - 1) / tpc;
      uint32_t so = 0;
      const bool fine = ranked && !(flagw[gg] & kBitBadRank);
      if (fine) for (int i = tt * ob; i < min(N, (tt + 1) * ob); ++i) so += base[i];
      uint32_t io = so;
      for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t a = __shfl_up(io, d, kWave);
        if (lane >= d) io += a;
      }
      const int tw = tt >> 6;                                // (a team is at least a wavefront)
      if (live && lane == 63) part[tw] = io;
      __syncthreads();
      if (fine) {
        uint32_t bo = io - so;
        for (int w = 0; w < tw; ++w) bo += part[w];
        for (int i = tt * ob; i < min(N, (tt + 1) * ob); ++i) { const uint32_t x = base[i]; base[i] = (uint16_t)bo; bo += x; }
      }
      __syncthreads();
      if (fine) {
        if (tt < P) {                                        // the lanes' streams
          const int m = tt;
          uint32_t total = 0;
          for (int w = 0; w < tpc / kWave; ++w) total += part[w];
          const int lo = mo[m], hi = lo + mc[m];
          const uint32_t i0 = lo < N ? base[lo] : total, i1 = hi < N ? base[hi] : total;
          item0[gg * Pseg + m] = i0;
          items[gg * Pseg + m] = i1 - i0;
        }
        uint16_t *const row = stream + (int64_t)gg * p.row_items;
        for (int k0 = tt; k0 < N; k0 += kB * tpc) {
          uint32_t o[kB];
#pragma unroll
          for (int u = 0; u < kB; ++u) o[u] = p.first[list[min(k0 + u * tpc, N - 1)]];
#pragma unroll
          for (int u = 0; u < kB; ++u)
            if (k0 + u * tpc < N) {
              uint16_t *const at = row + base[k0 + u * tpc];
              at[0] = (uint16_t)o[u];
              for (uint32_t z = 1; z < (o[u] >> 16); ++z) at[z] = (uint16_t)(o[u] + z);
            }
        }
      }
      __syncthreads();
    }
    // nothing has arrived anywhere; entry N of every candidate (the operation of items without one) stays 0
    for (int i = tid; i < (int)(G * p.acc_stride / 4); i += T) ((uint32_t *)lds)[i] = 0;
    for (int i = tid; i < (int)(G * p.free_stride / 4); i += T) ((uint32_t *)(lds + p.o_free))[i] = 0;
    // (a tag below every one that is looked for)
    for (int i = tid; i < p.slots * kWave; i += T) ((u32x4_t *)(lds + p.o_ring))[i] = u32x4_t{0u, 0u, 0u, 0u};
    if (tid < 64) taken[tid] = (uint32_t)p.slots;
    if (tid == 0) misc[0] = 0;
    __syncthreads();

    // ---------------------------------------------------------------- relaxation
    const int ml = lane / R;
    const bool lane_on = ml < G * Pseg;
    const int ql = lane_on ? ml : 0, g = ql >> p.log_pseg, j = ql & (Pseg - 1);
    const bool ok = lane_on && g < ng && flagw[g] == 0 && j < P;
    const uint32_t n_items = ok ? items[ql] : 0u;
    __syncthreads();                                         // (everyone has read the flags before an accountant adds one)
    const int ring_mask = p.slots - 1;
    const uint32_t acc0 = (uint32_t)g * p.acc_stride >> 2;   // LDS address / 4 of this candidate's arrival times, and of its channels
    const uint32_t free0 = (p.o_free + (uint32_t)g * p.free_stride) >> 2;
    // least of a machine's lanes, in each of them (all lanes of the wavefront take part)
    auto least = [](uint32_t x) {
      if (R >= 2) x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true));   // lane ^ 1
      if (R >= 4) x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true));   // lane ^ 2
      return x;
    };
    uint32_t x_acc = 0;
    bool cyclic = false;
    if (wave == 0) {
      __builtin_amdgcn_s_setprio(3);
      lds_byte_t *const ring_lane = ldsb + p.o_ring + (uint32_t)lane * 16u;
      const uint32_t cnt_k = p.o_cnt + (uint32_t)g * p.cnt_stride - acc0;   // LDS address of a count = index of the arrival time + this
      const uint32_t none = (acc0 + (uint32_t)N) * 0x10001u;
      const uint64_t segmask = ((Pseg * R == kWave) ? ~0ull : ((1ull << (Pseg * R)) - 1ull)) << (g * Pseg * R);
      uint32_t t = (uint32_t)p.slots;                        // tag of the next item
      const uint32_t t_end = n_items + (uint32_t)p.slots;
      uint64_t have = 0;                                     // lanes that hold an item
      bool dead = false;
      u32x4_t w = {none, 0u, kNoMessage, free0}, nw = {0u, 0u, 0u, 0u};   // the item at work, and the content of the next one's ring slot
      // arrival time and open messages of the item's operation; when its channel is free
      uint32_t arr = 0, cnt = 0, ch0 = 0;
      lds_vu32_t *const taken_p = (lds_vu32_t *)(ldsb + (uint32_t)((unsigned char *)taken - lds) + (uint32_t)lane * 4u);
      const uint32_t max_turns = 8u * ((uint32_t)N + (uint32_t)E + 1024u);
      uint32_t done_turns = 0;
      for (; done_turns < max_turns; ++done_turns) {
        uint64_t moved = 0;
#pragma unroll
        for (int sub = 0; sub < 8; ++sub) {
          const uint32_t e = max(arr, x_acc) + w.y;          // eqs. (3), (7), (12)
          const uint64_t ran_m = __ballot(cnt == 0) & have;
          const bool ran = lane_bit(ran_m);
          const uint32_t d = max(e, ch0) + w.z;              // eqs. (11), (13)-(15)
          x_acc = ran ? e : x_acc;
          uint64_t there;                                    // machines whose next item is there in all their lanes
          if (R == 4) {                                      // (missing in any lane of the four: one scalar instruction; two moves cost 1 % of a step)
            asm("s_wqm_b64 %0, %1" : "=s"(there) : "s"(__ballot((nw.w >> 16) != (t & 0xFFFFu))) : "scc");
            there = ~there;
          } else {
            there = __ballot((least(nw.w) >> 16) == (t & 0xFFFFu));
          }
          const uint64_t take_m = (ran_m | ~have) & there;
          const bool take = lane_bit(take_m);
          have = (have & ~ran_m) | take_m;
          moved |= ran_m | take_m;
          // The message: the arrival time first, then the count (LDS keeps their order).  Under the lanes' mask and
          // without a branch: at a branch's end the compiler waits for every LDS access before it, a round trip per step.
          // (The channel's time by a maximum: lanes of one item may share the channel.)
          const uint32_t to = hi16_x4(w.x), to_cnt = (w.x >> 16) + cnt_k, chan_at = lo16_x4(w.w);
          uint64_t all_lanes;
          asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, %1\n\tds_max_u32 %2, %3\n\tds_max_u32 %4, %3\n\tds_sub_u32 %5, %6\n\ts_mov_b64 exec, %0"
                       : "=&s"(all_lanes) : "s"(ran_m & __ballot((int32_t)w.z >= 0)), "v"(chan_at), "v"(d), "v"(to), "v"(to_cnt & ~3u), "v"(1u << ((to_cnt & 3u) * 8u)) : "memory");
          w.x = take ? nw.x : w.x; w.y = take ? nw.y : w.y; w.z = take ? nw.z : w.z; w.w = take ? nw.w : w.w;
          const uint32_t own = w.x & 0xFFFFu;
          cnt = *(lds_cu8_t *)(uintptr_t)(own + cnt_k);
          arr = *(lds_vu32_t *)(uintptr_t)(own << 2);
          uint64_t carry;
          asm("v_addc_co_u32 %0, %1, %2, 0, %3" : "=v"(t), "=&s"(carry) : "v"(t), "s"(take_m));   // t + 1 where taken
          nw = *(lds_vu32x4_t *)(ring_lane + ((t & (uint32_t)ring_mask) << 10));
          ch0 = *(lds_vu32_t *)(uintptr_t)lo16_x4(w.w);      // (needed last: read before the entry it costs 8 us of 592)
          if (sub == 3 || sub == 7) *taken_p = t;
          __builtin_amdgcn_sched_barrier(0);                 // (all reads are on their way before the first is waited for)
        }
        const bool held = lane_bit(have);
        bool through = dead || (!held && t == t_end);
        const uint64_t open = __ballot(!through);
        if (open == 0) break;
        // every unfinished machine of a candidate holds an item and none of them moved in eight steps: a cycle
        const uint64_t stuck = (__ballot(held) | ~open) & ~moved;
        if (!through && (stuck & segmask) == segmask) { dead = cyclic = true; }
      }
      if (done_turns == max_turns && !(dead || (!lane_bit(have) && t == t_end))) flagw[g] = kBitInternal;   // never expected
      *(lds_vu32_t *)(ldsb + (uint32_t)((unsigned char *)misc - lds)) = 1u;
      __builtin_amdgcn_s_setprio(0);
    } else if (wave <= p.accountants) {
      // Accountants: 64 messages of one machine per turn.  What a turn looks up (item, message, receiver's machine and rank) is
      // three lookups one behind the other, each requested a turn ahead of the next, across the ends of the streams.
      uint32_t *const seen = seenw + (wave - 1) * 64;
      struct Turn { int g, m; uint32_t s, end; };            // candidate, machine (g == ng: none left), messages s .. of end
      auto begin = [&](int g_at, int m_at) {
        for (;; m_at += p.accountants) {
          while (m_at >= P) { m_at -= P; ++g_at; }
          if (g_at >= ng || !(__builtin_amdgcn_readfirstlane(flagw[g_at]) & (kBitBadPlacement | kBitBadRank | kBitOrder))) break;
        }
        return Turn{g_at, m_at, 0u, g_at < ng ? (uint32_t)__builtin_amdgcn_readfirstlane((int)items[g_at * Pseg + m_at]) * R : 0u};
      };
      auto next = [&](const Turn &x) { return x.g >= ng ? x : x.s + kWave < x.end ? Turn{x.g, x.m, x.s + kWave, x.end} : begin(x.g, x.m + p.accountants); };
      auto item_of = [&](const Turn &x) {
        return x.s + lane < x.end ? (uint32_t)stream[(int64_t)x.g * p.row_items + item0[x.g * Pseg + x.m] + (x.s + lane) / R] : 0u;
      };
      auto message_of = [&](const Turn &x, uint32_t item) { return x.s + lane < x.end ? p.item[item * R + lane % R] : make_uint2((uint32_t)N * 0x10001u, 0u); };
      int32_t to = -1, rank = 0;
      int64_t md = 0, wt = 0;
      auto look_up = [&](const Turn &x, const uint2 &msg) {
        const uint32_t own = lane % R == 0 ? msg.x & 0xFFFFu : (uint32_t)N, dst = msg.x >> 16;
        const int64_t c = c0 + min(x.g, ng - 1);
        to = dst < (uint32_t)N ? p.placement[c * N + dst] : -1;
        rank = dst < (uint32_t)N ? p.edge_rank[c * E + msg.y] : 0;
        md = own < (uint32_t)N ? p.mem_delta[own] : 0;
        wt = own < (uint32_t)N && p.weight ? p.weight[own] : 0;
      };
      Turn t0 = begin(0, wave - 1), t1 = next(t0), t2 = next(t1), t3 = next(t2);
      uint2 msg1 = message_of(t1, item_of(t1));
      uint32_t item2 = item_of(t2), item3 = item_of(t3);
      look_up(t0, message_of(t0, item_of(t0)));
      int64_t level = 0, peak = 0, base_mem = 0;
      bool strange = false;
      auto turn = [&]() {
        if (t0.s == 0) { level = peak = base_mem = 0; strange = false; seen[lane] = 0; }
        const int32_t to_now = to, rank_now = rank, m = t0.m;
        int64_t sum = md;
        base_mem += wt;
        const uint2 msg2 = message_of(t2, item2);
        const Turn t4 = next(t3);
        item2 = item3; item3 = item_of(t4);
        look_up(t1, msg1);
        msg1 = msg2;
        // lanes that send on the same channel find one another by ballots over the bits of the receiving machine
        const bool has = to_now >= 0 && to_now != m;
        uint64_t same = __ballot(has);
        for (int bit = 0; (1 << bit) < P; ++bit) {
          const uint64_t set = __ballot((to_now >> bit) & 1);
          same &= (to_now >> bit) & 1 ? set : ~set;
        }
        if (has) {
          const uint32_t want = seen[to_now] + (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
          strange = strange || want != (uint32_t)rank_now;
          if ((same >> lane) == 1ull) seen[to_now] = want + 1u;   // the last of them
        }
        // inclusive sums over the wavefront (eq. (19)), largest of them in lane 63
#define DAGSCHED_STEP64(x, ctrl, rows, expr)                                                                      \
  {                                                                                                               \
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, ctrl, rows, 0xF, false);       \
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), ctrl, rows, 0xF, false); \
    const int64_t other = (int64_t)(((uint64_t)hi << 32) | lo);                                                   \
    x = expr;                                                                                                     \
  }
#define DAGSCHED_WAVE64(x, expr)                                                                                          \
  DAGSCHED_STEP64(x, 0x111, 0xF, expr) DAGSCHED_STEP64(x, 0x112, 0xF, expr) DAGSCHED_STEP64(x, 0x114, 0xF, expr)          \
  DAGSCHED_STEP64(x, 0x118, 0xF, expr) DAGSCHED_STEP64(x, 0x142, 0xA, expr) DAGSCHED_STEP64(x, 0x143, 0xC, expr)
        auto last = [](int64_t x) {
          return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), 63) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, 63));
        };
        DAGSCHED_WAVE64(sum, sum + other)
        peak = max(peak, level + sum);
        level += last(sum);
        if (t0.s + kWave >= t0.end) {                        // the stream's last turn
          DAGSCHED_WAVE64(peak, max(peak, other))            // (no peak is below 0)
          DAGSCHED_WAVE64(base_mem, base_mem + other)
          const int64_t top = last(peak) + last(base_mem);
          const int bits = (__ballot(strange) ? kBitOrder : 0) | (p.mem_limit && top > p.mem_limit[m] ? kBitOverMemory : 0);
          if (lane == 0) {
            p.out_ptrs.peak_mem[(c0 + t0.g) * p.out_ptrs.peak_stride_c + m * p.out_ptrs.peak_stride_j] = top;
            if (bits) atomicOr(&flagw[t0.g], bits);
          }
          if (bits & kBitOrder) {
            // The other kernel's candidate: its counts get a bit that no message takes away (bit 7 where it is not set already,
            // which is enough of them), so that its machines come to a halt, which the relaxer takes for a cycle.  (A look at the
            // flag by the relaxer cost 1 % of every batch, by the helpers 2 %; this test at every turn instead of at a stream's
            // last one, 1 to 3 %.)
            lds_byte_t *const cnt_b = ldsb + p.o_cnt + (uint32_t)t0.g * p.cnt_stride;
            for (int i = lane; i < (N + 4) / 4; i += kWave)
              __hip_atomic_fetch_or((DAGSCHED_LDS uint32_t *)cnt_b + i, 0x80808080u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
#undef DAGSCHED_WAVE64
#undef DAGSCHED_STEP64
        t0 = t1; t1 = t2; t2 = t3; t3 = t4;
      };
      while (t0.g < ng) turn();
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");     // (the peaks are out before a flagged candidate's are overwritten)
    } else {
      // helpers: item fed + i of lane `lane`, i = h, h + nh, ...
      const int h = wave - 1 - p.accountants, nh = (T >> 6) - 1 - p.accountants, r = lane % R;
      const uint16_t *const row = stream + (int64_t)g * p.row_items + (ok ? item0[ql] : 0u);
      const int32_t *const pl = p.placement + (c0 + (ok ? g : 0)) * N;
      const uint32_t bias_x = acc0 * 0x10001u;
      lds_vu32_t *const taken_p = (lds_vu32_t *)(ldsb + (uint32_t)((unsigned char *)taken - lds) + (uint32_t)lane * 4u);
      lds_vu32_t *const done_p = (lds_vu32_t *)(ldsb + (uint32_t)((unsigned char *)misc - lds));
      uint32_t f = (uint32_t)h;                              // the lane's next item that is this wavefront's
      while (__ballot(f < n_items) != 0 && !*done_p) {       // (the relaxer always ends, and says so)
        const uint32_t upto = min(n_items, least(*taken_p));
        if (__ballot(f < upto) == 0) { __builtin_amdgcn_s_sleep(2); continue; }
        // (messages of one item on one channel: the second one starts when the first is through, which is what twice the
        // delay says.  Three items at a time: each is three lookups, one behind the other)
        constexpr int kI = 3;
        if (f < upto) {
          uint32_t it[kI], dur[kI], delay[kI];
          int32_t to[kI];
          uint2 q[kI];
#pragma unroll
          for (int u = 0; u < kI; ++u) it[u] = row[min(f + (uint32_t)(u * nh), upto - 1u)];
#pragma unroll
          for (int u = 0; u < kI; ++u) q[u] = p.item[it[u] * R + r];
#pragma unroll
          for (int u = 0; u < kI; ++u) {
            const uint32_t own = q[u].x & 0xFFFFu, dst = q[u].x >> 16;
            dur[u] = own < (uint32_t)N ? (uint32_t)p.dur[own] : 0u;
            to[u] = dst < (uint32_t)N ? pl[dst] : -1;
          }
#pragma unroll
          for (int u = 0; u < kI; ++u) delay[u] = to[u] >= 0 ? (uint32_t)p.comm[j * P + to[u]] : 0u;
#pragma unroll
          for (int u = 0; u < kI; ++u) {
            const uint32_t at = f + (uint32_t)(u * nh);
            uint32_t times = 1;
            if (R == 2) {                                    // (the move itself for all lanes: it reads lanes that take part in it)
              const int32_t t0 = __builtin_amdgcn_update_dpp(0, to[u], 0xA0, 0xF, 0xF, true);
              times += r > 0 && t0 == to[u] ? 1u : 0u;
            }
            if (R == 4) {
              const int32_t t0 = __builtin_amdgcn_update_dpp(0, to[u], 0x00, 0xF, 0xF, true), t1 = __builtin_amdgcn_update_dpp(0, to[u], 0x55, 0xF, 0xF, true),
                            t2 = __builtin_amdgcn_update_dpp(0, to[u], 0xAA, 0xF, 0xF, true);
              times += (r > 0 && t0 == to[u] ? 1u : 0u) + (r > 1 && t1 == to[u] ? 1u : 0u) + (r > 2 && t2 == to[u] ? 1u : 0u);
            }
            if (at >= upto) continue;
            const uint32_t chan = to[u] >= 0 ? (uint32_t)(j * P + to[u]) + free0 : free0;
            // (the tag last: it says that the rest is there; until then the one before it)
            const u32x4_t val = {q[u].x + bias_x, dur[u], to[u] >= 0 ? delay[u] * times : kNoMessage, chan | (at << 16)};
            lds_byte_t *const sp = ldsb + p.o_ring + ((at & (uint32_t)ring_mask) << 10) + (uint32_t)lane * 16u;
            *(lds_vu32x4_t *)sp = val;
            *(lds_vu32_t *)(sp + 12) = chan | ((at + (uint32_t)p.slots) << 16);
          }
#pragma unroll
          for (int u = 0; u < kI; ++u) f += f < upto ? (uint32_t)nh : 0u;
        }
      }
    }
    __syncthreads();

    // ---------------------------------------------------------------- reductions and outputs (wave 0)
    if (wave == 0) {
      int32_t z = (int32_t)x_acc;
      uint32_t cyc = cyclic ? 1u : 0u;
      for (int d = 1; d < Pseg * R; d <<= 1) { z = max(z, __shfl_xor(z, d, kWave)); cyc |= __shfl_xor(cyc, d, kWave); }
      if (lane_on && g < ng && j < P && lane % R == 0) {
        const int64_t c = c0 + g;
        const int bits = flagw[g] | (cyc ? kBitCyclic : 0);
        if ((bits & kBitOrder) && !(bits & (kBitBadPlacement | kBitBadRank))) {
          if (j == 0) { const int slot = atomicAdd(p.fb_count, 1); p.fb_list[slot] = (int32_t)c; }   // the other kernel writes this candidate
        } else {
          const int flag = flag_from_bits(bits);             // (the peaks are there already)
          if (flag) p.out_ptrs.peak_mem[c * p.out_ptrs.peak_stride_c + j * p.out_ptrs.peak_stride_j] = -1;
          if (j == 0) {
            p.out_ptrs.makespan[c] = flag ? -1 : z;
            p.out_ptrs.bubble[c] = flag ? -1 : (int64_t)P * z - p.sum_dur;
            p.out_ptrs.flags[c] = flag;
          }
        }
      }
    }
    __syncthreads();                                         // everything is set up again for the next candidates
  }
  // The last workgroup says how many candidates are left and clears the counters for the next call.  (Done here, where
  // workgroups end one after the other: as the other kernel's last act, all its
  // workgroups met at one counter: 94 instead of 77 us for the zero-bubble pipeline, 617 instead of 609 for the MoE graph.)
  if (tid == 0) {
    __threadfence();
    if (atomicAdd(p.ticket, 1) == (int32_t)gridDim.x - 1) {
      __threadfence();
      *p.fb_todo = atomicExch(p.fb_count, 0);
      atomicExch(p.ticket, 0);
    }
  }
}

}  // namespace dagsched_dev
