// Host side: operations that share an end-time cell.
//
// A kernel that keeps one end-time cell per operation needs N of them per candidate, although only few end times are
// still waited for at any moment.  Which ones depends on the candidate, but B alone already says a lot: once an
// operation x runs, everything that precedes x in B has run.  So x may take over the cell of u as soon as every
// operation that reads u's end time is x itself or a predecessor of x in B (by any path), whatever the candidate:
// along a chain one cell goes from hand to hand.  (1F1B pipeline, 64 operations: 8 cells; zero-bubble pipeline, 768: 32;
// bidirectional pipeline, 6144: 64.  Where many operations run side by side the bounded search below finds little:
// the layered graph, 50000 operations, keeps some 45000.)
//
// A reader may look at a cell long before the end time it waits for is there, when the cell still holds an earlier
// user's.  So the users of a cell are numbered 1, 2, 3, ... (0: nobody yet), and a cell holds number << T | end time.
// A reader that waits for user n adds delay - (n << T): once user n has ended that is its end time plus the delay,
// before that it is negative, i.e. as an unsigned number above every time.  One addition is the whole test.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace dagsched_host {

struct SharedCells {
  int n_cells = 0;                       // cells 1 .. n_cells; cell 0 stays 0 ("ended at time 0"), for absent predecessors
  int max_user = 0;                      // the largest user number
  std::vector<int32_t> cell, user;       // [N] cell 0 for operations that nobody reads
};

// reach_ptr / reach_idx: predecessor lists whose paths may be relied on (all of B, or B without edges that other paths
// imply); read_ptr / read_idx: the predecessors whose end times are read.  A bounded search: ancestors are known over
// the last kWindow operations in topological order, and the cells looked at are bounded too; what is not found only
// costs another cell.
inline SharedCells share_cells(int N, const std::vector<int32_t> &reach_ptr, const std::vector<int32_t> &reach_idx,
                               const std::vector<int32_t> &read_ptr, const std::vector<int32_t> &read_idx, int max_user) {
  constexpr int kWindow = 512, kWords = kWindow / 64, kLooked = 64;
  SharedCells out;
  out.cell.assign((size_t)N, 0);
  out.user.assign((size_t)N, 0);
  // topological order: the ids themselves where they are one, else sources first
  std::vector<int32_t> pos((size_t)N), order((size_t)N);
  bool by_id = true;
  for (int v = 0; v < N && by_id; ++v)
    for (int32_t k = reach_ptr[v]; k < reach_ptr[v + 1]; ++k) by_id = by_id && reach_idx[k] < v;
  if (by_id) {
    for (int v = 0; v < N; ++v) order[v] = pos[v] = v;
  } else {
    std::vector<int32_t> sp((size_t)N + 1, 0), si(reach_idx.size()), left((size_t)N);
    for (int32_t u : reach_idx) ++sp[u + 1];
    for (int v = 0; v < N; ++v) sp[v + 1] += sp[v];
    std::vector<int32_t> fill(sp.begin(), sp.end() - 1);
    for (int v = 0; v < N; ++v)
      for (int32_t k = reach_ptr[v]; k < reach_ptr[v + 1]; ++k) si[fill[reach_idx[k]]++] = v;
    std::vector<int32_t> stack;            // depth first: what follows one another in B stays close together
    for (int v = N - 1; v >= 0; --v)
      if ((left[v] = reach_ptr[v + 1] - reach_ptr[v]) == 0) stack.push_back(v);
    int at = 0;
    while (!stack.empty()) {
      const int32_t u = stack.back();
      stack.pop_back();
      order[at] = u; pos[u] = at++;
      for (int32_t k = sp[u + 1] - 1; k >= sp[u]; --k)
        if (--left[si[k]] == 0) stack.push_back(si[k]);
    }
    if (at != N) return out;               // (B is acyclic: never)
  }
  // readers of every operation, by position in the order
  std::vector<int32_t> rp((size_t)N + 1, 0), ri(read_idx.size());
  for (int32_t u : read_idx) ++rp[u + 1];
  for (int v = 0; v < N; ++v) rp[v + 1] += rp[v];
  {
    std::vector<int32_t> fill(rp.begin(), rp.end() - 1);
    for (int v = 0; v < N; ++v)
      for (int32_t k = read_ptr[v]; k < read_ptr[v + 1]; ++k) ri[fill[read_idx[k]]++] = pos[v];
  }
  std::vector<uint64_t> ring((size_t)kWindow * kWords, 0);   // row of position i: bit q mod kWindow = the operation at q precedes it
  // the operations that hold a cell which nobody has taken over, newest first
  std::vector<int32_t> older((size_t)N, -1), newer((size_t)N, -1);
  int32_t newest = -1;
  auto drop = [&](int32_t u) {
    (newer[u] >= 0 ? older[newer[u]] : newest) = older[u];
    if (older[u] >= 0) newer[older[u]] = newer[u];
  };
  for (int i = 0; i < N; ++i) {
    const int x = order[i];
    uint64_t *const row = ring.data() + (size_t)(i % kWindow) * kWords;
    std::fill(row, row + kWords, 0);
    for (int32_t k = reach_ptr[x]; k < reach_ptr[x + 1]; ++k) {
      const int q = pos[reach_idx[k]];
      if (q <= i - kWindow) continue;
      const uint64_t *const from = ring.data() + (size_t)(q % kWindow) * kWords;
      // bits (q + 1 .. i) mod kWindow of that row are operations from before this window
      uint64_t known[kWords];
      std::copy(from, from + kWords, known);
      for (int b = (q + 1) % kWindow, n = i - q; n > 0;) {
        const int lo = b % 64, take = std::min(64 - lo, n);
        known[b / 64] &= ~((take == 64 ? ~0ull : (1ull << take) - 1ull) << lo);
        b = (b + take) % kWindow; n -= take;
      }
      for (int w = 0; w < kWords; ++w) row[w] |= known[w];
      row[(q % kWindow) / 64] |= 1ull << (q % 64);
    }
    if (rp[x + 1] == rp[x]) continue;                        // nobody reads it
    int32_t cell = 0, user = 1;
    for (int32_t u = newest, looked = 0; u >= 0 && looked < kLooked; ++looked) {
      const int32_t then = older[u];
      bool free = true;
      for (int32_t k = rp[u]; free && k < rp[u + 1]; ++k) {
        const int q = ri[k];
        free = q == i || (q < i && q > i - kWindow && ((row[(q % kWindow) / 64] >> (q % 64)) & 1ull));
      }
      if (free && out.user[u] < max_user) { cell = out.cell[u]; user = out.user[u] + 1; drop(u); break; }
      u = then;
    }
    if (!cell) cell = ++out.n_cells;
    out.cell[x] = cell; out.user[x] = user;
    out.max_user = std::max(out.max_user, user);
    older[x] = newest; newer[x] = -1;
    if (newest >= 0) newer[newest] = x;
    newest = x;
  }
  return out;
}

}  // namespace dagsched_host
