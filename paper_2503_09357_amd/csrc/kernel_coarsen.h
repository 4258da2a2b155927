// Graph coarsening before the planning (Sec. IV, Alg. 1): operations are merged greedily until at most a target
// number is left.  One persistent workgroup holds the whole procedure, because every merge changes which edges are
// redundant and which pairs qualify, so the merges are inherently one after the other; inside a step everything is
// data-parallel over the graph:
//
//   B as two bit matrices: succ[u] and pred[v], n rows of W = ceil(n / 64) words.
//   Topologically redundant edge (u, v):  some w with (u, w) and (w, v) in B  <=>  succ[u] AND pred[v] != 0.  The
//   reduced graph B' is kept as a third bit matrix with its degrees.  A merge into m can change the status only of
//   edges that leave m or a predecessor of m (an edge (u, v) looks at succ[u] and at the rows of u's successors),
//   so after a merge only those rows are worked out again, a wavefront per row.
//   GetCandidateEdge:     the lowest row with a single output in B' whose target has a single input there.
//   GetCandidateNonEdge:  depth = longest path in edges from a source, by peeling sources round by round.  Merging
//                         two operations of equal depth changes no depth (the new operation's predecessors are the
//                         union of theirs), so the depths are worked out once per run of non-edge merges.  Every
//                         operation u keeps its best partner v > u as a key (summed duration, u, v); sums only grow,
//                         so a merge of m and o can worsen only the keys that name m or o, and only those (and m's
//                         own) are looked for again.
//   MergeNodes:           a thread per operation moves o's bits to m in its own rows, then OR of the two rows in both
//                         matrices, sums of duration, memory adjustment and memory requirement; the merged operation
//                         keeps the smaller name.
//
// What bounds it is the chain of merges, each a few barriers with a little work between them; waiting out one memory
// access after the other is what makes them long.  So graphs of up to 512 operations (coarsen_lds_kernel) are held in LDS,
// a thread per operation and a wavefront per 64 of them, with rows short enough to be read whole: a row of B' is a
// ballot per 64 columns, an edge merge takes three barriers and a non-edge merge none.  Larger graphs (coarsen_kernel)
// work in the L2.
// The paper's scale, 200 operations to 40: 271 us (321 us for the whole call with its allocation and copies) against
// 7400 us for the kernel that worked in the L2 and searched all pairs for every merge; the MoE graph (11712 operations,
// 700 merges, in the L2) 0.2 s against 11 s.  What is left of the small one is instructions of a lone wavefront: about
// 1000 cycles per partner looked for, two per merge.
//
// Every loop either merges (at most n - 1 times in all) or ends, and no wavefront ever waits for another one
// except at barriers that all reach: the kernel always terminates.
#pragma once

#include "device_common.h"

namespace dagsched_dev {

constexpr int kCoarsenLdsNodes = 512;
// Work arrays in global memory: byte offsets from the start of the arena.
struct CoarsenLayout {
  size_t succ, pred, kept;               // [n][words] u64
  size_t dur, mem, req;                  // [n] i64: the groups' sums at their names
  size_t best;                           // [n] u64: key of the best non-edge partner
  size_t parent, indeg, only, depth, aux;   // [n] i32: parent[v] == v: v is alive; only: the single output in B', or -1
  size_t total;
};
inline CoarsenLayout coarsen_layout(int n) {
  CoarsenLayout l;
  const size_t words = ((size_t)n + 63) / 64, m = (size_t)n * words * 8;
  size_t at = 0;
  auto take = [&](size_t bytes) { const size_t o = at; at += bytes; return o; };
  l.succ = take(m); l.pred = take(m); l.kept = take(m);   // first: these are the ones to be cleared
  l.dur = take((size_t)n * 8); l.mem = take((size_t)n * 8); l.req = take((size_t)n * 8); l.best = take((size_t)n * 8);
  l.parent = take((size_t)n * 4); l.indeg = take((size_t)n * 4); l.only = take((size_t)n * 4); l.depth = take((size_t)n * 4);
  l.aux = take((size_t)n * 4);
  l.total = (at + 15) / 16 * 16;
  return l;
}

struct CoarsenParams {
  int32_t n, n_edges, words, target;     // words = ceil(n / 64)
  int64_t edge_dur_max, edge_mem_max, nonedge_dur_max, nonedge_mem_max;
  const int32_t *row_ptr, *col_idx;      // successor CSR of B
  const int32_t *dur;                    // [n]
  const int64_t *mem, *req;              // [n]; req may be NULL (all zero)
  unsigned char *arena;                  // work arrays of coarsen_kernel (matrices zero on entry)
  CoarsenLayout at;
  // results
  int32_t *node_map;                     // [n]
  int32_t *c_row_ptr, *c_col_idx;        // [n + 1], [n_edges]
  int32_t *c_dur;                        // [n]
  int64_t *c_mem, *c_req;                // [n]
  int32_t *counts;                       // [3] groups, edge merges, non-edge merges
};

constexpr uint64_t kNoCandidate = ~0ull;

// least of the wavefront's 64 values, in every lane
__device__ __forceinline__ uint64_t wave_min(uint64_t x) {
  // within rows of 16, then across: DPP moves, no LDS trip
#define DAGSCHED_MIN_STEP(ctrl, rows)                                                                                        \
  {                                                                                                                          \
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)(uint32_t)x, ctrl, rows, 0xF, false);                 \
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)(uint32_t)(x >> 32), ctrl, rows, 0xF, false);         \
    x = min(x, ((uint64_t)hi << 32) | lo);                                                                                   \
  }
  DAGSCHED_MIN_STEP(0x111, 0xF)          // from the lane 1, 2, 4, 8 before
  DAGSCHED_MIN_STEP(0x112, 0xF)
  DAGSCHED_MIN_STEP(0x114, 0xF)
  DAGSCHED_MIN_STEP(0x118, 0xF)
  DAGSCHED_MIN_STEP(0x142, 0xA)          // last lane of a row to the next row
  DAGSCHED_MIN_STEP(0x143, 0xC)          // lane 31 to the upper half
#undef DAGSCHED_MIN_STEP
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), 63) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, 63);
}

// f(v) for every set bit v of a row of W words, ascending, with all lanes of the wavefront taking part (the row is
// read 64 words at a time, a word per lane).
template <typename F>
__device__ __forceinline__ void for_each_bit(const uint64_t *row, int W, int lane, F f) {
  for (int base = 0; base < W; base += kWave) {
    const uint64_t word = (base + lane < W) ? row[base + lane] : 0ull;
    uint64_t nz = __ballot(word != 0);
    while (nz) {
      const int owner = __builtin_ctzll(nz);
      nz &= nz - 1;
      uint64_t bits = __shfl(word, owner, kWave);
      while (bits) {
        const int v = ((base + owner) << 6) + __builtin_ctzll(bits);
        bits &= bits - 1;
        f(v);
      }
    }
  }
}

// Work arrays in global memory (L2), any size; 1024 threads.
__global__ __launch_bounds__(1024) void coarsen_kernel(CoarsenParams p) {
  __shared__ uint64_t s_part[2][16];
  __shared__ int s_any;
  typedef uint64_t *U64;
  typedef int64_t *I64;
  typedef int32_t *I32;
  unsigned char *const base = p.arena;
  const U64 succ = (U64)(base + p.at.succ), pred = (U64)(base + p.at.pred), kept = (U64)(base + p.at.kept), best = (U64)(base + p.at.best);
  const I64 dur = (I64)(base + p.at.dur), mem = (I64)(base + p.at.mem), req = (I64)(base + p.at.req);
  const I32 parent = (I32)(base + p.at.parent), indeg = (I32)(base + p.at.indeg), only = (I32)(base + p.at.only),
            depth = (I32)(base + p.at.depth), aux = (I32)(base + p.at.aux);
  const int tid = threadIdx.x, nthreads = blockDim.x;
  const int lane = tid & 63, nwaves = nthreads >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = p.n, W = p.words;
  auto add = [](I32 q, int x) { __hip_atomic_fetch_add(q, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  auto set_bit = [](U64 q, uint64_t bit) { __hip_atomic_fetch_or(q, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  int turn = 0;
  // least value over the workgroup; one barrier, which also orders what was written before it
  auto group_min = [&](uint64_t x) {
    x = wave_min(x);
    turn ^= 1;
    if (lane == 0) s_part[turn][wave] = x;
    __syncthreads();
    uint64_t all = kNoCandidate;
    for (int w = 0; w < nwaves; ++w) all = min(all, s_part[turn][w]);
    return all;
  };

  for (int v = tid; v < n; v += nthreads) {
    parent[v] = v; indeg[v] = 0; only[v] = -1;
    dur[v] = p.dur[v]; mem[v] = p.mem[v]; req[v] = p.req ? p.req[v] : 0;
  }
  __syncthreads();
  for (int u = tid; u < n; u += nthreads)
    for (int k = p.row_ptr[u]; k < p.row_ptr[u + 1]; ++k) {
      const int v = p.col_idx[k];
      succ[(size_t)u * W + (v >> 6)] |= 1ull << (v & 63);     // (row u is this thread's)
      set_bit(&pred[(size_t)v * W + (u >> 6)], 1ull << (u & 63));
    }
  __syncthreads();

  // Row u of the reduced graph B' (one wavefront): an edge (u, v) stays unless some operation lies between u and v.
  // The in-degrees of B' follow the bits that changed against the row as it was.
  auto reduce_row = [&](int u) {
    const U64 su = succ + (size_t)u * W, ku = kept + (size_t)u * W;
    int kept_count = 0, last = -1;
    for (int b0 = 0; b0 < W; b0 += kWave) {
      const uint64_t word = (b0 + lane < W) ? su[b0 + lane] : 0ull;
      uint64_t keep = 0, nz = __ballot(word != 0);
      while (nz) {
        const int owner = __builtin_ctzll(nz);
        nz &= nz - 1;
        uint64_t bits = __shfl(word, owner, kWave);
        while (bits) {
          const int b = __builtin_ctzll(bits);
          bits &= bits - 1;
          const int v = ((b0 + owner) << 6) + b;
          const U64 pv = pred + (size_t)v * W;
          bool hit = false;
          for (int x = lane; x < W; x += kWave) hit = hit || (su[x] & pv[x]) != 0;
          if (__ballot(hit) == 0) {                        // no operation between u and v
            ++kept_count;
            last = v;
            if (lane == owner) keep |= 1ull << b;
          }
        }
      }
      if (b0 + lane < W) {
        uint64_t diff = ku[b0 + lane] ^ keep;
        while (diff) {
          const int b = __builtin_ctzll(diff);
          diff &= diff - 1;
          add(&indeg[((b0 + lane) << 6) + b], ((keep >> b) & 1ull) ? 1 : -1);
        }
        ku[b0 + lane] = keep;
      }
    }
    if (lane == 0) only[u] = kept_count == 1 ? last : -1;
  };

  for (int u = wave; u < n; u += nwaves) reduce_row(u);
  __syncthreads();

  // MergeNodes(a, b): the operation with the larger name vanishes into the one with the smaller name
  auto merge_nodes = [&](int a, int b) {
    const int m = min(a, b), o = max(a, b);
    const U64 sm = succ + (size_t)m * W, so = succ + (size_t)o * W, pm = pred + (size_t)m * W, po = pred + (size_t)o * W;
    const uint64_t bit_m = 1ull << (m & 63), bit_o = 1ull << (o & 63);
    const int wm = m >> 6, wo = o >> 6;
    // every neighbour of o now sees m instead (a neighbour's rows are its own thread's)
    for (int x = tid; x < n; x += nthreads) {
      const uint64_t bit = 1ull << (x & 63);
      if (x == m) continue;
      if (so[x >> 6] & bit) { const U64 px = pred + (size_t)x * W; px[wo] &= ~bit_o; px[wm] |= bit_m; }
      if (po[x >> 6] & bit) { const U64 sx = succ + (size_t)x * W; sx[wo] &= ~bit_o; sx[wm] |= bit_m; }
    }
    __syncthreads();
    for (int w = tid; w < W; w += nthreads) {
      uint64_t s = sm[w] | so[w], q = pm[w] | po[w];
      if (w == wm) { s &= ~bit_m; q &= ~bit_m; }
      if (w == wo) { s &= ~bit_o; q &= ~bit_o; }
      sm[w] = s; pm[w] = q;
      so[w] = 0; po[w] = 0;
    }
    if (tid == 0) {
      dur[m] += dur[o]; mem[m] += mem[o]; req[m] += req[o];
      parent[o] = m;
    }
    __syncthreads();
    // the reduced graph again, where it can have changed: the rows of m, of o (now empty) and of m's predecessors
    int item = 2;
    if (wave == 0) reduce_row(m);
    if (wave == 1 % nwaves) reduce_row(o);
    for_each_bit(pm, W, lane, [&](int x) {
      if (item++ % nwaves == wave) reduce_row(x);
    });
  };

  // the best partner of operation u among the later ones of its depth (one wavefront)
  auto find_partner = [&](int u) {
    uint64_t mine = kNoCandidate;
    if (parent[u] == u) {
      const int du = depth[u];
      const int64_t dur_u = dur[u], req_u = req[u];
      for (int v = (u & ~63) + lane; v < n; v += kWave) {
        if (v <= u || parent[v] != v || depth[v] != du) continue;
        const int64_t s = dur_u + dur[v];
        if (s <= p.nonedge_dur_max && req_u + req[v] <= p.nonedge_mem_max)
          mine = min(mine, ((uint64_t)s << 32) | ((uint64_t)(uint32_t)u << 16) | (uint32_t)v);
      }
      mine = wave_min(mine);
    }
    if (lane == 0) best[u] = mine;
  };

  int size = n, merges_edge = 0, merges_nonedge = 0;
  while (size > p.target) {                                 // the outer loop of Alg. 1
    bool merged = false;
    while (size > p.target) {                               // GetCandidateEdge / MergeNodes
      uint64_t mine = kNoCandidate;
      for (int u = tid; u < n; u += nthreads) {
        const int v = only[u];                              // (-1 for operations that are gone)
        if (v < 0 || indeg[v] != 1) continue;
        if (dur[u] + dur[v] <= p.edge_dur_max && req[u] + req[v] <= p.edge_mem_max)
          mine = min(mine, ((uint64_t)(uint32_t)u << 32) | (uint32_t)v);
      }
      const uint64_t found = group_min(mine);
      if (found == kNoCandidate) break;
      merge_nodes((int)(found >> 32), (int)(found & 0xFFFFFFFFu));
      __syncthreads();
      --size; ++merges_edge; merged = true;
    }
    if (size <= p.target) break;
    // depth = edges on the longest path from a source: sources are peeled round by round
    // (aux = predecessors not yet peeled; per round first the operations to peel are marked, aux = -1; what the marking
    // reads is at rest since the last barrier; then, behind a barrier, their successors are told; peeled: aux = -2)
    for (int v = wave; v < n; v += nwaves) {
      int c = 0;
      if (parent[v] == v) {
        const U64 pv = pred + (size_t)v * W;
        for (int x = lane; x < W; x += kWave) c += __popcll(pv[x]);
        for (int s = 1; s < kWave; s <<= 1) c += __shfl_xor(c, s, kWave);
      }
      if (lane == 0) { aux[v] = c; depth[v] = 0; }
    }
    __syncthreads();
    for (int round = 0; round < n; ++round) {
      if (tid == 0) s_any = 0;
      for (int v = tid; v < n; v += nthreads)
        if (parent[v] == v && aux[v] == 0 && depth[v] == round) aux[v] = -1;
      __syncthreads();
      for (int v = wave; v < n; v += nwaves) {
        if (parent[v] != v || aux[v] != -1) continue;      // wave-uniform
        for_each_bit(succ + (size_t)v * W, W, lane, [&](int x) {
          if (lane == 0) {
            __hip_atomic_fetch_max(&depth[x], round + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            add(&aux[x], -1);
            s_any = 1;
          }
        });
        if (lane == 0) aux[v] = -2;
      }
      __syncthreads();
      const int any = s_any;
      __syncthreads();
      if (!any) break;
    }
    for (int u = wave; u < n; u += nwaves) find_partner(u);
    __syncthreads();
    while (size > p.target) {                               // GetCandidateNonEdge / MergeNodes
      uint64_t mine = kNoCandidate;
      for (int u = tid; u < n; u += nthreads) mine = min(mine, best[u]);
      const uint64_t found = group_min(mine);
      if (found == kNoCandidate) break;
      const int m = (int)((found >> 16) & 0xFFFFu), o = (int)(found & 0xFFFFu);
      merge_nodes(m, o);
      // keys that name m or o (and m's own) are out of date: m's sums grew, o is gone
      for (int u0 = wave << 6; u0 < n; u0 += nwaves << 6) {
        const int u = u0 + lane;
        const uint64_t key = u < n ? best[u] : kNoCandidate;
        const int v = (int)(key & 0xFFFFu);
        uint64_t stale = __ballot(u < n && key != kNoCandidate && (v == m || v == o || u == o)) | __ballot(u == m);
        while (stale) {
          const int i = __builtin_ctzll(stale);
          stale &= stale - 1;
          find_partner(u0 + i);
        }
      }
      __syncthreads();
      --size; ++merges_nonedge; merged = true;
    }
    if (!merged) break;
  }

  // groups numbered in the order of their names; the coarse graph as a CSR with ascending columns
  __syncthreads();
  for (int v = wave; v < n; v += nwaves) {                  // edges per row
    int c = 0;
    if (parent[v] == v) {
      const U64 sv = succ + (size_t)v * W;
      for (int x = lane; x < W; x += kWave) c += __popcll(sv[x]);
      for (int s = 1; s < kWave; s <<= 1) c += __shfl_xor(c, s, kWave);
    }
    if (lane == 0) aux[v] = c;
  }
  __syncthreads();
  if (wave == 0) {                                          // 64 operations at a time: index and start of the row
    int k = 0, at = 0;
    for (int v0 = 0; v0 < n; v0 += kWave) {
      const int v = v0 + lane;
      const bool alive = v < n && parent[min(v, n - 1)] == v;
      const uint64_t mask = __ballot(alive);
      const int mine = alive ? aux[v] : 0;
      int incl = mine;
      for (int s = 1; s < kWave; s <<= 1) {
        const int o = __shfl_up(incl, s, kWave);
        if (lane >= s) incl += o;
      }
      if (alive) {
        const int i = k + __popcll(mask & ((1ull << lane) - 1ull));
        aux[v] = i;
        p.c_dur[i] = (int32_t)dur[v]; p.c_mem[i] = mem[v]; p.c_req[i] = req[v];
        p.c_row_ptr[i] = at + incl - mine;
        depth[v] = at + incl - mine;                        // (no longer needed as a depth)
      }
      k += __popcll(mask);
      at += __builtin_amdgcn_readlane(incl, 63);
    }
    if (lane == 0) { p.c_row_ptr[k] = at; p.counts[0] = k; p.counts[1] = merges_edge; p.counts[2] = merges_nonedge; }
  }
  __syncthreads();
  for (int v = tid; v < n; v += nthreads) {
    int r = v;
    while (parent[r] != r) r = parent[r];                   // names only ever point to smaller names: the walk ends
    p.node_map[v] = aux[r];
  }
  for (int v = wave; v < n; v += nwaves) {
    if (parent[v] != v) continue;
    int at = depth[v];
    for (int b0 = 0; b0 < W; ++b0) {
      const uint64_t word = succ[(size_t)v * W + b0];
      if ((word >> lane) & 1ull) p.c_col_idx[at + __popcll(word & ((1ull << lane) - 1ull))] = aux[(b0 << 6) + lane];
      at += __popcll(word);
    }
  }
}

// least of the wavefront's 64 values, in every lane
__device__ __forceinline__ uint32_t wave_min32(uint32_t x) {
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x111, 0xF, 0xF, false));
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x112, 0xF, 0xF, false));
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x114, 0xF, 0xF, false));
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x118, 0xF, 0xF, false));
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x142, 0xA, 0xF, false));
  x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x143, 0xC, 0xF, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// LDS of coarsen_lds_kernel<WM>: three matrices with rows of WM words and one of padding (rows apart by a power of two
// would share banks), then the attributes.
constexpr size_t coarsen_lds_bytes(int WM) { return (size_t)64 * WM * (3 * 8 * (WM + 1) + 2 * 8 + 6 * 4) + 2 * 8 * WM; }

// n <= 64 * WM; thread v stands for operation v, wavefront w for the operations 64 w .. 64 w + 63.  GetCandidateNonEdge
// looks at depths, durations and memory requirements only, none of which needs the matrices: a run of non-edge merges is
// the work of one wavefront with all of that in registers (no barrier, no LDS), and the matrices are built anew from the
// edges afterwards.
template <int WM>
__global__ __launch_bounds__(64 * WM) void coarsen_lds_kernel(CoarsenParams p) {
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ uint64_t s_part[2][WM];
  typedef DAGSCHED_LDS uint64_t *U64;
  typedef DAGSCHED_LDS int64_t *I64;
  typedef DAGSCHED_LDS int32_t *I32;
  constexpr int NT = 64 * WM, S = WM + 1;
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  const U64 succ = (U64)lds, pred = succ + NT * S, kept = pred + NT * S;
  const I64 mem = (I64)(kept + NT * S), req = mem + NT;
  const U64 open = (U64)(req + NT);                          // [2][WM] operations not yet peeled
  const I32 parent = (I32)(open + 2 * WM), indeg = parent + NT, depth = indeg + NT, dur = depth + NT, pmin = dur + NT,
            pwho = pmin + NT;
  // parent[v] == v: alive; indeg: inputs in B'; depth: -1 for operations that are gone; pmin, pwho: summed
  // duration with the best later partner of the same depth (kNone: there is none), and the partner
  const int tid = threadIdx.x, lane = tid & 63, n = p.n;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t below = (1ull << lane) - 1ull;
  int turn = 0;
  auto group_min = [&](uint64_t mine) {                      // least of the wavefronts' values; one barrier
    turn ^= 1;
    if (lane == 0) s_part[turn][wave] = mine;
    __syncthreads();
    uint64_t all = s_part[turn][0];
#pragma unroll
    for (int w = 1; w < WM; ++w) all = min(all, s_part[turn][w]);
    return all;
  };

  // every operation's parent becomes its group's name (chains of up to n - 1 names, halved nine times; names only ever
  // point to smaller names)
  auto shorten = [&]() {
    for (int i = 0; i < 9; ++i) {
      const int r = tid < n ? parent[parent[tid]] : -1;
      __syncthreads();
      parent[tid] = r;
      __syncthreads();
    }
  };
  int my_indeg = 0;                                          // inputs of operation tid in B'
  // B between the groups as they are; B' empty
  auto build = [&]() {
    for (int i = tid; i < 3 * NT * S; i += NT) succ[i] = 0;
    my_indeg = 0;
    shorten();
    if (tid < n) {
      const int u = parent[tid];
      for (int k = p.row_ptr[tid]; k < p.row_ptr[tid + 1]; ++k) {
        const int v = parent[p.col_idx[k]];
        if (v == u) continue;
        __hip_atomic_fetch_or(&succ[u * S + (v >> 6)], 1ull << (v & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_or(&pred[v * S + (u >> 6)], 1ull << (u & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    __syncthreads();
  };
  parent[tid] = tid < n ? tid : -1;
  dur[tid] = tid < n ? p.dur[tid] : 0; mem[tid] = 0; req[tid] = tid < n && p.req ? p.req[tid] : 0;
  __syncthreads();
  build();

  // Rows of the reduced graph B', four at a time: an edge (u, v) stays unless some operation lies between u and v.  Every
  // wavefront does the 64 columns of its own operations, whose rows of pred it holds in registers (column()), and keeps
  // their in-degrees in B'.  The row of an operation that was merged away (gone) becomes empty.  (A wavefront per row
  // instead took 1400 cycles a row: it is instructions that count here, and this way a row takes 30 of them.)
  uint64_t pr[WM];
  auto column = [&]() {
#pragma unroll
    for (int x = 0; x < WM; ++x) pr[x] = pred[tid * S + x];
  };
  auto reduce_rows = [&](const int (&u)[4], int count, int gone) {
    uint64_t su[4][WM], own[4], old[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int c = 0; c < WM; ++c) su[i][c] = succ[u[i] * S + c];
      own[i] = succ[u[i] * S + wave];
      old[i] = kept[u[i] * S + wave];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i >= count) break;
      uint64_t between = 0;
#pragma unroll
      for (int x = 0; x < WM; ++x) between |= su[i][x] & pr[x];
      const uint64_t keep = u[i] == gone ? 0ull : own[i] & __ballot(between == 0);
      my_indeg += (int)((keep >> lane) & 1ull) - (int)((old[i] >> lane) & 1ull);
      if (lane == 0) kept[u[i] * S + wave] = keep;
    }
  };

  // MergeNodes(m, o), m < o, of an edge merge: o vanishes into m.  Row o itself is left alone until everybody has read it.
  auto merge_nodes = [&](int m, int o) {
    const uint64_t bit_m = 1ull << (m & 63), bit_o = 1ull << (o & 63);
    const int wm = m >> 6, wo = o >> 6;
    const uint64_t so = succ[o * S + wave], po = pred[o * S + wave];
    // every neighbour of o now sees m instead (a neighbour's rows are its own thread's)
    if (tid != m) {
      if ((so >> lane) & 1ull) { pred[tid * S + wo] &= ~bit_o; pred[tid * S + wm] |= bit_m; }
      if ((po >> lane) & 1ull) { succ[tid * S + wo] &= ~bit_o; succ[tid * S + wm] |= bit_m; }
    }
    if (wave == 0 && lane < WM) {
      const uint64_t both = succ[m * S + lane] | succ[o * S + lane];
      succ[m * S + lane] = both & ~(lane == wm ? bit_m : 0) & ~(lane == wo ? bit_o : 0);
    }
    if (wave == 1 && lane < WM) {
      const uint64_t both = pred[m * S + lane] | pred[o * S + lane];
      pred[m * S + lane] = both & ~(lane == wm ? bit_m : 0) & ~(lane == wo ? bit_o : 0);
    }
    if (tid == 2 * kWave) { dur[m] += dur[o]; req[m] += req[o]; parent[o] = m; }
    __syncthreads();
    // the reduced graph again, where it can have changed: the rows of m, of o (now empty) and of m's predecessors
    uint64_t pm[WM];
#pragma unroll
    for (int c = 0; c < WM; ++c) {
      const uint64_t word = pred[m * S + c];
      pm[c] = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(word >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)word);
    }
    column();
    int rows[4] = {m, o, m, m}, count = 2;
#pragma unroll
    for (int c = 0; c < WM; ++c)
      for (uint64_t bits = pm[c]; bits; bits &= bits - 1) {
        const int x = (c << 6) + __builtin_ctzll(bits);
        rows[0] = count == 0 ? x : rows[0]; rows[1] = count == 1 ? x : rows[1]; rows[2] = count == 2 ? x : rows[2]; rows[3] = count == 3 ? x : rows[3];
        if (++count == 4) { reduce_rows(rows, 4, o); count = 0; }
      }
    if (count) reduce_rows(rows, count, o);
    indeg[tid] = my_indeg;
    __syncthreads();
    if (tid < WM) { succ[o * S + tid] = 0; pred[o * S + tid] = 0; }   // (read again behind the next barrier)
  };

  // Registers of a run of non-edge merges, the same in every wavefront: lane i, word c stands for operation 64 c + i
  int r_dur[WM], r_depth[WM], r_who[WM];
  int64_t r_req[WM];
  uint32_t r_sum[WM];
  auto of = [](const int (&r)[WM], int v) {                  // value of operation v (the same for all lanes)
    int x = __builtin_amdgcn_readlane(r[0], v & 63);
#pragma unroll
    for (int c = 1; c < WM; ++c) { const int y = __builtin_amdgcn_readlane(r[c], v & 63); x = (v >> 6) == c ? y : x; }
    return x;
  };
  auto of64 = [](const int64_t (&r)[WM], int v) {
    int64_t x = 0;
#pragma unroll
    for (int c = 0; c < WM; ++c) {
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)r[c], v & 63), hi = (uint32_t)__builtin_amdgcn_readlane((int)(r[c] >> 32), v & 63);
      x = (v >> 6) == c ? (int64_t)(((uint64_t)hi << 32) | lo) : x;
    }
    return x;
  };
  // the best partner of operation u among the later ones of its depth: least summed duration (kNone: there is none)
  auto find_partner = [&](int u, int &who) {
    const int du = of(r_depth, u), dur_u = of(r_dur, u);
    who = -1;
    if (du < 0) return kNone;
    const int64_t req_room = p.nonedge_mem_max - of64(r_req, u);   // (requirements are not negative)
    const int dur_room = (int)min(p.nonedge_dur_max - dur_u, (int64_t)INT32_MAX);
    uint32_t s[WM], least = kNone;
#pragma unroll
    for (int c = 0; c < WM; ++c) {
      s[c] = kNone;
      if (c < (u >> 6)) continue;                            // (the same for all lanes)
      s[c] = (c << 6) + lane > u && r_depth[c] == du && r_dur[c] <= dur_room && r_req[c] <= req_room ? (uint32_t)(dur_u + r_dur[c]) : kNone;
      least = min(least, s[c]);
    }
    least = wave_min32(least);
#pragma unroll
    for (int c = WM - 1; c >= 0; --c) {
      const uint64_t b = __ballot(s[c] == least);
      who = b ? (c << 6) + __builtin_ctzll(b) : who;
    }
    return least;
  };

  int size = n, merges_edge = 0, merges_nonedge = 0;
  bool stale_matrices = false;
  while (size > p.target) {                                 // the outer loop of Alg. 1
    bool merged = false;
    if (stale_matrices) { build(); stale_matrices = false; }
    column();
    for (int u = 0; u < n; u += 4) {
      const int rows[4] = {u, u + 1, u + 2, u + 3};          // (n is at most a multiple of 64: the rows beyond it are empty)
      reduce_rows(rows, 4, -1);
    }
    indeg[tid] = my_indeg;
    __syncthreads();
    while (size > p.target) {                               // GetCandidateEdge / MergeNodes
      int outs = 0, v = -1;                                  // outputs in B', and the last of them
#pragma unroll
      for (int c = 0; c < WM; ++c) {
        const uint64_t word = kept[tid * S + c];
        outs += __popcll(word);
        v = word ? (c << 6) + 63 - __builtin_clzll(word) : v;
      }
      bool fit = false;
      if (outs == 1) fit = indeg[v] == 1 && (int64_t)dur[tid] + dur[v] <= p.edge_dur_max && req[tid] + req[v] <= p.edge_mem_max;
      const uint64_t b = __ballot(fit);
      const int first = b ? __builtin_ctzll(b) : 0;
      const uint64_t mine = ((uint64_t)(uint32_t)((wave << 6) + first) << 32) | (uint32_t)__builtin_amdgcn_readlane(v, first);
      const uint64_t found = group_min(b ? mine : kNoCandidate);
      if (found == kNoCandidate) break;
      const int x = (int)(found >> 32), y = (int)(found & 0xFFFFFFFFu);
      merge_nodes(min(x, y), max(x, y));
      --size; ++merges_edge; merged = true;
    }
    if (size <= p.target) break;
    // depth = edges on the longest path from a source: sources are peeled round by round, one barrier each
    {
      column();
      const bool alive = parent[tid] == tid;
      const uint64_t mask = __ballot(alive);
      if (lane == 0) open[wave] = mask;
      int d = -1;
      __syncthreads();
      for (int round = 0; round <= n; ++round) {
        const U64 now = open + (round & 1) * WM, next = open + (~round & 1) * WM;
        uint64_t o[WM], any = 0, waits = 0;
#pragma unroll
        for (int x = 0; x < WM; ++x) o[x] = now[x];
#pragma unroll
        for (int x = 0; x < WM; ++x) { any |= o[x]; waits |= o[x] & pr[x]; }
        if (any == 0) break;
        const uint64_t own = now[wave];
        const bool go = ((own >> lane) & 1ull) && waits == 0;   // none of its predecessors is left
        d = go ? round : d;
        const uint64_t gone = __ballot(go);
        if (lane == 0) next[wave] = own & ~gone;
        __syncthreads();
      }
      depth[tid] = d;
      __syncthreads();
    }
    // GetCandidateNonEdge / MergeNodes: first every operation's best partner, shared out among the wavefronts
#pragma unroll
    for (int c = 0; c < WM; ++c) { const int v = (c << 6) + lane; r_dur[c] = dur[v]; r_depth[c] = depth[v]; r_req[c] = req[v]; }
    for (int u = wave; u < NT; u += WM) {
      int who;
      const uint32_t least = find_partner(u, who);
      if (lane == 0) { pmin[u] = (int)least; pwho[u] = who; }
    }
    __syncthreads();
    if (wave == 0) {
      int count = 0;
#pragma unroll
      for (int c = 0; c < WM; ++c) { const int v = (c << 6) + lane; r_sum[c] = (uint32_t)pmin[v]; r_who[c] = pwho[v]; }
      while (size - count > p.target) {
        uint32_t least = r_sum[0];
#pragma unroll
        for (int c = 1; c < WM; ++c) least = min(least, r_sum[c]);
        least = wave_min32(least);
        if (least == kNone) break;
        int m = 0;
#pragma unroll
        for (int c = WM - 1; c >= 0; --c) { const uint64_t b = __ballot(r_sum[c] == least); m = b ? (c << 6) + __builtin_ctzll(b) : m; }
        const int o = of(r_who, m);
        const int64_t req_m = of64(r_req, m) + of64(r_req, o);
        if (lane == 0) parent[o] = m;
        // keys that name m or o (and m's own) are out of date: m's sums grew, o is gone
        // (o needs no partner any more)
        uint64_t again[WM];
#pragma unroll
        for (int c = 0; c < WM; ++c) {
          const int v = (c << 6) + lane;
          r_dur[c] = v == m ? (int)least : r_dur[c];
          r_req[c] = v == m ? req_m : r_req[c];
          r_depth[c] = v == o ? -1 : r_depth[c];
          r_sum[c] = v == o ? kNone : r_sum[c];
          again[c] = __ballot(v == m || (r_sum[c] != kNone && (r_who[c] == m || r_who[c] == o)));
        }
#pragma unroll
        for (int c = 0; c < WM; ++c)
          for (uint64_t bits = again[c]; bits; bits &= bits - 1) {
            const int i = __builtin_ctzll(bits);
            int who;
            const uint32_t sum = find_partner((c << 6) + i, who);
            r_sum[c] = lane == i ? sum : r_sum[c];
            r_who[c] = lane == i ? who : r_who[c];
          }
        ++count;
      }
#pragma unroll
      for (int c = 0; c < WM; ++c) { const int v = (c << 6) + lane; dur[v] = r_dur[c]; req[v] = r_req[c]; }
      if (lane == 0) s_part[0][0] = (uint64_t)count;
    }
    __syncthreads();
    const int count = (int)s_part[0][0];
    __syncthreads();
    size -= count; merges_nonedge += count;
    merged = merged || count > 0;
    stale_matrices = count > 0;
    if (!merged) break;
  }

  // groups numbered in the order of their names; the coarse graph as a CSR with ascending columns
  if (stale_matrices) build(); else shorten();
  if (tid < n) __hip_atomic_fetch_add(&mem[parent[tid]], p.mem[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  const bool alive = parent[tid] == tid;
  const uint64_t mask = __ballot(alive);
  int degree = 0;
#pragma unroll
  for (int c = 0; c < WM; ++c) degree += alive ? __popcll(succ[tid * S + c]) : 0;
  int incl = degree;
  for (int s = 1; s < kWave; s <<= 1) {
    const int o = __shfl_up(incl, s, kWave);
    if (lane >= s) incl += o;
  }
  turn ^= 1;
  if (lane == 63) s_part[turn][wave] = ((uint64_t)__popcll(mask) << 32) | (uint32_t)incl;
  __syncthreads();
  uint64_t before = 0, all = 0;                              // groups << 32 | edges
#pragma unroll
  for (int w = 0; w < WM; ++w) { const uint64_t x = s_part[turn][w]; before += w < wave ? x : 0; all += x; }
  const int index = (int)(before >> 32) + __popcll(mask & below), at = (int)(uint32_t)before + incl - degree;
  if (alive) {
    depth[tid] = index;                                      // (no longer needed as a depth)
    p.c_dur[index] = dur[tid]; p.c_mem[index] = mem[tid]; p.c_req[index] = req[tid];
    p.c_row_ptr[index] = at;
  }
  if (tid == 0) { p.c_row_ptr[all >> 32] = (int32_t)(uint32_t)all; p.counts[0] = (int32_t)(all >> 32); p.counts[1] = merges_edge; p.counts[2] = merges_nonedge; }
  __syncthreads();
  if (tid < n) {
    p.node_map[tid] = depth[parent[tid]];
  }
  if (alive) {
    int k = at;
#pragma unroll
    for (int c = 0; c < WM; ++c)
      for (uint64_t bits = succ[tid * S + c]; bits; bits &= bits - 1) p.c_col_idx[k++] = depth[(c << 6) + __builtin_ctzll(bits)];
  }
}

}  // namespace dagsched_dev
