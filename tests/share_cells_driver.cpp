// share_cells behind a C entry, for tests/test_share_cells.py
#include <cstdint>

#include "share_cells.h"

extern "C" int share_cells(int n, const int32_t *reach_ptr, const int32_t *reach_idx, const int32_t *read_ptr, const int32_t *read_idx,
                           int max_user, int32_t *cell, int32_t *user) {
  using V = std::vector<int32_t>;
  const dagsched_host::SharedCells s = dagsched_host::share_cells(n, V(reach_ptr, reach_ptr + n + 1), V(reach_idx, reach_idx + reach_ptr[n]),
                                                                  V(read_ptr, read_ptr + n + 1), V(read_idx, read_idx + read_ptr[n]), max_user);
  for (int i = 0; i < n; ++i) { cell[i] = s.cell[i]; user[i] = s.user[i]; }
  return s.n_cells;
}
