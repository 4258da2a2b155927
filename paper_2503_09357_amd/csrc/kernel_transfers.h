// Evaluation with channel contention (Sec. III, eqs. (11)-(15)) for candidates whose channel orders follow their
// producers: the fast path beside kernel_contended.h, which takes the rest.
//
// Every transfer of a channel (a, b) is produced by an operation of machine a, and machine a runs its operations one
// after the other.  Where the transfers of every channel are ranked in the order in which machine a produces them (first
// come, first served, and every order that does not put a transfer behind one that is produced later), a transfer can be
// completed the moment its producer has ended:
//   d_k = max(e_u, free(a, b)) + comm[a][b],  free(a, b) = d_k       (eqs. (11), (13)-(15))
// so nothing ever waits for a channel, and an edge inside a machine is implied by the chain (or contradicts it, a cycle).
// What is left is the evaluation without contention with the roles turned round: instead of polling its predecessors, an
// operation waits until the number of messages still on their way to it is 0, and whoever completes a transfer takes the
// maximum into the receiver's arrival time and one off its count (eq. (12)).
//
// One workgroup = G candidates, lane (g, j) = machine j of candidate g, arrival times and counts in LDS:
//   ingest    (all wavefronts) checks the candidate and writes machine j's stream of ITEMS to a workspace row: an operation
//             together with its first message, then its further messages.
//   RELAXER   wave 0: per step at most one item per lane.  An item is ready when its operation's count is 0 (at once when
//             it holds no operation).
//   HELPERS   waves 2..: copy the streams into rings in LDS, 16 bytes an item, ahead of the relaxer.
//   ACCOUNTANT wave 1: memory levels along the streams (eqs. (16)-(19)).
// They meet at one barrier per slots / 2 steps; the counts they hand over are kept twice, by the parity of the phase.
//
// What bounds it is the chain of dependent steps (MoE graph: a candidate's longest path of operations and messages),
// each an LDS round trip and about 40 instructions of a lone wavefront.  MoE graph, 512 candidates: %MEASURED%
#pragma once

#include "device_common.h"

namespace dagsched_dev {

struct TransferParams {
  int32_t N, E, P, Pseg, log_pseg, G, C;
  int32_t teams;                        // candidates ingested side by side (a power of two, at most G)
  int32_t slots;                        // ring slots per lane: 16 or 32
  const uint4 *out;                     // [N] out-edges of operation v: x = first edge, y = how many, z = first two receivers (16 bits each), w = next two
  const int32_t *col_idx;               // [E] receivers in successor-CSR order
  const int32_t *dur, *comm;            // [N], [P * P] (0 where the pair has no channel)
  const int64_t *mem_delta, *weight, *mem_limit;
  int64_t sum_dur;
  const int32_t *placement, *rank, *edge_rank;   // [C][N], [C][N], [C][E]
  uint4 *stream;                        // [grid][G][row_items] x = own operation (N: none) | receiver << 16, y = duration, z = delay,
                                        // w = channel | (1: there is a message) << 16
  int64_t row_items;
  int32_t *fb_count, *fb_list;          // candidates left to the other kernel
  // LDS: arrival times at 0, then these; ingest works in the first `scratch` bytes of every team, all before o_cnt
  uint32_t acc_stride, o_free, free_stride, o_ring, o_cnt, cnt_stride, o_book, total;
  uint32_t team_stride, s_base, s_order, s_chan, s_first, s_part;   // scratch of a team: placement bytes at 0, then these
  OutPtrs out_ptrs;
};

// Shape for a problem, or false when it does not fit (the other kernel then does everything).
inline bool transfer_plan(TransferParams *p, int threads, int64_t n_cand, int n_cu, uint32_t lds_max) {
  const uint32_t N = (uint32_t)p->N, E = (uint32_t)p->E, P = (uint32_t)p->P;
  if ((uint64_t)N + E > 65000u) return false;            // item numbers are 16-bit
  auto up = [](uint32_t x, uint32_t a) { return (x + a - 1) / a * a; };
  p->acc_stride = up(4 * (N + 1), 16);
  p->free_stride = up(4 * P * P, 16);
  p->cnt_stride = up(N + 1, 16);
  p->s_base = up(N, 16);
  p->s_order = p->s_base + up(2 * N, 16);
  p->s_chan = p->s_order + up(2 * E, 16);
  p->s_first = p->s_chan + up(4 * (P * P + 1), 16);
  p->s_part = p->s_first + up(4 * ((E + 31) / 32), 16);
  p->team_stride = p->s_part + 256;
  const int g_max = kWave / p->Pseg;
  for (int G = g_max; G >= 1; G >>= 1) {
    // (small batches: rather more workgroups than full wavefronts, as long as CUs would stay empty)
    if (G > 1 && (n_cand + G - 1) / G < n_cu) continue;
    for (int slots : {32, 16}) {
      uint32_t at = (uint32_t)G * p->acc_stride;
      p->o_free = at; at += (uint32_t)G * p->free_stride;
      p->o_ring = at; at += (uint32_t)slots * kWave * 16u;
      at = at > p->team_stride ? at : p->team_stride;
      p->teams = 1;
      while (p->teams < G && (uint32_t)p->teams * 2u * p->team_stride <= at && threads / (p->teams * 2) >= kWave) p->teams *= 2;
      p->o_cnt = at; at += (uint32_t)G * p->cnt_stride;
      p->o_book = at; at += 64 * 4 * 10 + 64 * 8 + 64;
      p->total = at;
      p->G = G; p->slots = slots;
      if (at <= lds_max) return true;
    }
  }
  return false;
}

constexpr int kTransferThreads = 1024;

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
  uint32_t *const taken = items + 64;                        // [2][64]
  uint32_t *const fed = taken + 128;                         // [2][64]
  int32_t *const flagw = (int32_t *)(fed + 128);             // [64] (G used)
  int32_t *const misc = flagw + 64;                          // [0..1] done by parity of the phase
  int64_t *const peakw = (int64_t *)(misc + 64);             // [64]
  uint8_t *const overb = (uint8_t *)(peakw + 64);            // [64]
  constexpr int kBitOrder = 128;                             // internal: some channel's order does not follow the producers

  const int64_t n_groups = ((int64_t)p.C + G - 1) / G;
  for (int64_t group = blockIdx.x; group < n_groups; group += gridDim.x) {
    const int64_t c0 = group * G;
    const int ng = (int)min((int64_t)G, (int64_t)p.C - c0);
    uint4 *const stream = p.stream + (int64_t)blockIdx.x * G * p.row_items;

    // ---------------------------------------------------------------- ingest
    const int tpc = T / p.teams, team = tid / tpc, tt = tid - team * tpc;
    unsigned char *const sc = lds + (uint32_t)team * p.team_stride;
    uint8_t *const machine = sc;                             // [N]
    uint16_t *const base = (uint16_t *)(sc + p.s_base);      // [N] by list position: items of the operation there, then its first item
    uint16_t *const order = (uint16_t *)(sc + p.s_order);    // [transfers] by channel and rank: the transfer's item
    int32_t *const chan = (int32_t *)(sc + p.s_chan);        // [P * P + 1] transfers per channel, then the channel's start
    uint32_t *const first = (uint32_t *)(sc + p.s_first);    // [E bits] first transfer of a channel
    uint32_t *const part = (uint32_t *)(sc + p.s_part);      // [2][32] sums of the team's wavefronts
    if (tid < 64) { mcount[tid] = 0; flagw[tid] = 0; overb[tid] = 0; peakw[tid] = 0; items[tid] = 0; item0[tid] = 0; }
    for (int i = tid; i < (int)(G * p.cnt_stride / 4); i += T) ((uint32_t *)(lds + p.o_cnt))[i] = 0;
    __syncthreads();
    for (int g0 = 0; g0 < G; g0 += p.teams) {
      const int gg = g0 + team;
      const bool live = gg < ng;
      const int64_t c = c0 + (live ? gg : 0);
      const int32_t *const pl = p.placement + c * N, *const rk = p.rank + c * N, *const er = p.edge_rank + c * E;
      int32_t *const mc = mcount + gg * Pseg, *const mo = off + gg * Pseg;
      uint32_t *const cntw = (uint32_t *)(lds + p.o_cnt + (uint32_t)gg * p.cnt_stride);
      constexpr int kB = 4;
      if (live) {
        for (int i = tt; i < (N + 1) / 2; i += tpc) ((uint32_t *)base)[i] = 0xFFFFFFFFu;
        for (int i = tt; i < (E + 1) / 2; i += tpc) ((uint32_t *)order)[i] = 0xFFFFFFFFu;
        for (int i = tt; i <= P * P; i += tpc) chan[i] = 0;
        for (int i = tt; i < (E + 31) / 32; i += tpc) first[i] = 0;
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
        // ranks in range (eqs. (7)-(8)); items per operation; transfers per channel; messages per receiver
        for (int v0 = tt; v0 < N; v0 += kB * tpc) {
          int32_t r[kB];
          uint4 o[kB];
#pragma unroll
          for (int u = 0; u < kB; ++u) { const int v = min(v0 + u * tpc, N - 1); r[u] = rk[v]; o[u] = p.out[v]; }
#pragma unroll
          for (int u = 0; u < kB; ++u) {
            const int v = v0 + u * tpc;
            if (v >= N) break;
            const int a = machine[v];
            int n = 0;
            for (uint32_t e = 0; e < o[u].y; ++e) {
              const uint32_t x = e < 4 ? ((e < 2 ? o[u].z : o[u].w) >> ((e & 1) * 16)) & 0xFFFFu : (uint32_t)p.col_idx[o[u].x + e];
              const int b = machine[x];
              if (a != b) {
                atomicAdd(&chan[a * P + b], 1);
                atomicAdd(&cntw[x >> 2], 1u << ((x & 3) * 8));
                ++n;
              } else if (rk[x] <= r[u]) {
                atomicOr(&flagw[gg], kBitCyclic);           // the chain contradicts an edge inside the machine (or a rank is bad)
              }
            }
            if ((uint32_t)r[u] >= (uint32_t)mc[a]) atomicOr(&flagw[gg], kBitBadRank);
            else base[mo[a] + r[u]] = (uint16_t)max(1, n);
          }
        }
      }
      __syncthreads();
      // exclusive sums of both, a block of consecutive entries per thread; a slot of a list that nobody wrote: bad ranks
      const int ob = (N + tpc - 1) / tpc, cb = (P * P + tpc - 1) / tpc;
      uint32_t so = 0, sch = 0;
      if (well) {
        bool hole = false;
        for (int i = tt * ob; i < min(N, (tt + 1) * ob); ++i) { hole |= base[i] == 0xFFFFu; so += base[i]; }
        if (hole) atomicOr(&flagw[gg], kBitBadRank);
        for (int i = tt * cb; i < min(P * P, (tt + 1) * cb); ++i) sch += (uint32_t)chan[i];
      }
      uint32_t io = so, ic = sch;
      for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t a = __shfl_up(io, d, kWave), b = __shfl_up(ic, d, kWave);
        if (lane >= d) { io += a; ic += b; }
      }
      const int tw = tt >> 6;                                // (a team is at least a wavefront)
      if (live && lane == 63) { part[tw] = io; part[16 + tw] = ic; }
      __syncthreads();
      const bool fine = well && !(flagw[gg] & kBitBadRank);
      uint32_t n_transfers = 0;
      if (fine) {
        uint32_t bo = io - so, bc = ic - sch;
        for (int w = 0; w < tpc / kWave; ++w) { bo += w < tw ? part[w] : 0; bc += w < tw ? part[16 + w] : 0; n_transfers += part[16 + w]; }
        for (int i = tt * ob; i < min(N, (tt + 1) * ob); ++i) { const uint32_t x = base[i]; base[i] = (uint16_t)bo; bo += x; }
        for (int i = tt * cb; i < min(P * P, (tt + 1) * cb); ++i) {
          const uint32_t x = (uint32_t)chan[i];
          chan[i] = (int32_t)bc;
          if (x) atomicOr(&first[bc >> 5], 1u << (bc & 31));
          bc += x;
        }
        if (tt == tpc - 1) chan[P * P] = (int32_t)n_transfers;
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
        // the items, and a total order per channel (eqs. (14)-(15))
        uint4 *const row = stream + (int64_t)gg * p.row_items;
        for (int v0 = tt; v0 < N; v0 += kB * tpc) {
          int32_t r[kB], d[kB];
          uint4 o[kB];
#pragma unroll
          for (int u = 0; u < kB; ++u) { const int v = min(v0 + u * tpc, N - 1); r[u] = rk[v]; o[u] = p.out[v]; d[u] = p.dur[v]; }
#pragma unroll
          for (int u = 0; u < kB; ++u) {
            const int v = v0 + u * tpc;
            if (v >= N) break;
            const int a = machine[v];
            const uint32_t i0 = base[mo[a] + r[u]];
            uint32_t n = 0;
            for (uint32_t e = 0; e < o[u].y; ++e) {
              const uint32_t x = e < 4 ? ((e < 2 ? o[u].z : o[u].w) >> ((e & 1) * 16)) & 0xFFFFu : (uint32_t)p.col_idx[o[u].x + e];
              const int b = machine[x];
              if (a == b) continue;
              const int ch = a * P + b;
              const int32_t q = er[o[u].x + e];
              const int s = chan[ch];
              if ((uint32_t)q >= (uint32_t)(chan[ch + 1] - s)) atomicOr(&flagw[gg], kBitBadRank);
              else order[s + q] = (uint16_t)(i0 + n);
              row[i0 + n] = make_uint4((n == 0 ? (uint32_t)v : (uint32_t)N) | (x << 16), n == 0 ? (uint32_t)d[u] : 0u, (uint32_t)p.comm[ch], (uint32_t)ch | 0x10000u);
              ++n;
            }
            if (n == 0) row[i0] = make_uint4((uint32_t)v | ((uint32_t)N << 16), (uint32_t)d[u], 0u, 0u);
          }
        }
      }
      __syncthreads();
      if (fine) {
        int bits = 0;
        for (uint32_t i = (uint32_t)tt; i < n_transfers; i += (uint32_t)tpc) {
          const uint32_t x = order[i], before = i ? order[i - 1] : 0u;
          if (x == 0xFFFFu) bits |= kBitBadRank;
          else if (!((first[i >> 5] >> (i & 31)) & 1u) && before >= x) bits |= kBitOrder;
        }
        if (bits) atomicOr(&flagw[gg], bits);
      }
      __syncthreads();
    }
    // nothing has arrived anywhere; entry N of every candidate (the operation of items without one) stays 0
    for (int i = tid; i < (int)(G * p.acc_stride / 4); i += T) ((uint32_t *)lds)[i] = 0;
    for (int i = tid; i < (int)(G * p.free_stride / 4); i += T) ((uint32_t *)(lds + p.o_free))[i] = 0;
    if (tid < 128) { taken[tid] = 0; fed[tid] = 0; }
    if (tid < 2) misc[tid] = 0;
    __syncthreads();

    // ---------------------------------------------------------------- relaxation
    const bool lane_on = lane < G * Pseg;
    const int ql = lane_on ? lane : 0, g = ql >> p.log_pseg, j = ql & (Pseg - 1);
    const bool ok = lane_on && g < ng && flagw[g] == 0 && j < P;
    const uint32_t n_items = ok ? items[ql] : 0u;
    const int ring_mask = p.slots - 1, trips = p.slots / 2;
    const uint32_t acc0 = (uint32_t)g * p.acc_stride >> 2;   // LDS address / 4 of this candidate's arrival times, and of its channels
    const uint32_t free0 = (p.o_free + (uint32_t)g * p.free_stride) >> 2;
    uint32_t x_acc = 0;
    bool cyclic = false;
    if (wave == 0) {
      __builtin_amdgcn_s_setprio(3);
      lds_byte_t *const ring_lane = ldsb + p.o_ring + (uint32_t)lane * 16u;
      const uint32_t cnt_k = p.o_cnt + (uint32_t)g * p.cnt_stride - acc0;   // LDS address of a count = index of the arrival time + this
      const uint32_t none = (acc0 + (uint32_t)N) * 0x10001u;
      const uint64_t segmask = ((Pseg == kWave) ? ~0ull : ((1ull << Pseg) - 1ull)) << (g * Pseg);
      uint32_t t = 0;
      uint64_t have = 0;                                     // lanes that hold an item
      bool dead = false;
      u32x4_t w = {none, 0u, 0u, free0}, nw = w;
      uint32_t arr = 0, cnt = 0, chf = 0;                    // arrival time and open messages of the item's operation; when its channel is free
      const int64_t max_phases = 4 * ((int64_t)N + E) + 64;
      for (int64_t phase = 0; ; ++phase) {
        const uint32_t avail = fed[((phase + 1) & 1) * 64 + lane];
        uint64_t moved = 0;
        if (have | __ballot(t < avail)) {
          nw = *(lds_vu32x4_t *)(ring_lane + ((t & (uint32_t)ring_mask) << 10));
          for (int i = 0; i < trips; i += 8) {
#pragma unroll
            for (int sub = 0; sub < 8; ++sub) {
              const uint32_t e = max(arr, x_acc) + w.y;      // eqs. (3), (7), (12)
              const uint64_t ran_m = __ballot(cnt == 0) & have;
              const bool ran = lane_bit(ran_m);
              const uint32_t d = max(e, chf) + w.z;          // eqs. (11), (13)-(15)
              x_acc = ran ? e : x_acc;
              if (lane_bit(ran_m & __ballot((w.w >> 16) != 0u))) {
                const uint32_t x = w.x >> 16;                // the arrival time first, then the count: LDS keeps their order
                *(lds_vu32_t *)(uintptr_t)lo16_x4(w.w) = d;
                (void)__hip_atomic_fetch_max((DAGSCHED_LDS uint32_t *)(uintptr_t)(x << 2), d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const uint32_t q = x + cnt_k;
                (void)__hip_atomic_fetch_sub((DAGSCHED_LDS uint32_t *)(uintptr_t)(q & ~3u), 1u << ((q & 3u) * 8u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              }
              const uint64_t take_m = (ran_m | ~have) & __ballot(t < avail);
              const bool take = lane_bit(take_m);
              have = (have & ~ran_m) | take_m;
              moved |= ran_m | take_m;
              w.x = take ? nw.x : w.x; w.w = take ? nw.w : w.w;
              const uint32_t own = w.x & 0xFFFFu;
              cnt = *(lds_cu8_t *)(uintptr_t)(own + cnt_k);
              arr = *(lds_vu32_t *)(uintptr_t)(own << 2);
              chf = *(lds_vu32_t *)(uintptr_t)lo16_x4(w.w);
              w.y = take ? nw.y : w.y; w.z = take ? nw.z : w.z;
              t += take ? 1u : 0u;
              nw = *(lds_vu32x4_t *)(ring_lane + ((t & (uint32_t)ring_mask) << 10));
            }
          }
        }
        taken[(phase & 1) * 64 + lane] = t;
        const bool held = lane_bit(have), through = dead || (!held && t == n_items);
        // every unfinished machine of a candidate holds an item and none of them moved in a whole phase: a cycle
        const uint64_t stuck = (__ballot(held) | __ballot(through)) & ~moved;
        if (!through && (stuck & segmask) == segmask) { dead = cyclic = true; }
        const int done = __ballot(!(dead || (!held && t == n_items))) == 0 ? 1 : phase >= max_phases ? 2 : 0;
        if (lane == 0) misc[phase & 1] = done;
        __syncthreads();
        if (done) {
          if (done == 2 && !(dead || (!held && t == n_items))) flagw[g] = kBitInternal;
          break;
        }
      }
      __builtin_amdgcn_s_setprio(0);
    } else if (wave == 1) {
      // accountant (eqs. (16)-(19)): walks the lane's stream, eight items per phase
      const uint4 *const row = stream + (int64_t)g * p.row_items + (ok ? item0[ql] : 0u);
      uint32_t k = 0;
      int64_t level = 0, peak = 0, base_mem = 0;
      auto walk = [&]() {
        uint32_t id[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) id[u] = k + u < n_items ? row[k + u].x & 0xFFFFu : (uint32_t)N;
        int64_t md[8], wt[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) { md[u] = id[u] < (uint32_t)N ? p.mem_delta[id[u]] : 0; wt[u] = id[u] < (uint32_t)N && p.weight ? p.weight[id[u]] : 0; }
#pragma unroll
        for (int u = 0; u < 8; ++u) { level += md[u]; peak = max(peak, level); base_mem += wt[u]; }
        k += 8;
      };
      for (int64_t phase = 0; ; ++phase) {
        if (__ballot(k < n_items)) walk();
        __syncthreads();
        if (misc[phase & 1]) break;
      }
      while (__ballot(k < n_items)) walk();
      if (ok && p.mem_limit && base_mem + peak > p.mem_limit[j]) overb[g] = 1;
      peakw[lane] = base_mem + peak;
    } else {
      // helpers: item fed + i of lane `lane`, i = h, h + nh, ...
      const int h = wave - 2, nh = (T >> 6) - 2;
      const uint4 *const row = stream + (int64_t)g * p.row_items + (ok ? item0[ql] : 0u);
      const uint32_t bias_x = acc0 * 0x10001u;
      uint32_t f = 0;
      for (int64_t phase = 0; ; ++phase) {
        const uint32_t tk = taken[((phase + 1) & 1) * 64 + lane];
        const uint32_t upto = min(n_items, tk + (uint32_t)p.slots);
        for (uint32_t i = f + (uint32_t)h; i < upto; i += (uint32_t)nh) {
          const uint4 q = row[i];
          const u32x4_t val = {q.x + bias_x, q.y, q.z, q.w + free0};
          *(lds_vu32x4_t *)(ldsb + p.o_ring + ((i & (uint32_t)ring_mask) << 10) + (uint32_t)lane * 16u) = val;
        }
        f = max(f, upto);
        if (h == 0) fed[(phase & 1) * 64 + lane] = f;
        __syncthreads();
        if (misc[phase & 1]) break;
      }
    }
    __syncthreads();

    // ---------------------------------------------------------------- reductions and outputs (wave 0)
    if (wave == 0) {
      int32_t z = (int32_t)x_acc;
      uint32_t cyc = cyclic ? 1u : 0u;
      for (int d = 1; d < Pseg; d <<= 1) { z = max(z, __shfl_xor(z, d, Pseg)); cyc |= __shfl_xor(cyc, d, Pseg); }
      if (lane_on && g < ng && j < P) {
        const int64_t c = c0 + g;
        const int bits = flagw[g] | (cyc ? kBitCyclic : 0) | (overb[g] ? kBitOverMemory : 0);
        if ((bits & kBitOrder) && !(bits & (kBitBadRank | kBitCyclic))) {
          if (j == 0) { const int slot = atomicAdd(p.fb_count, 1); p.fb_list[slot] = (int32_t)c; }   // the other kernel writes this candidate
        } else {
          const int flag = flag_from_bits(bits);
          p.out_ptrs.peak_mem[c * p.out_ptrs.peak_stride_c + j * p.out_ptrs.peak_stride_j] = flag ? -1 : peakw[ql];
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
}

}  // namespace dagsched_dev
