// Panel sizes of the matrix engine when its workspace has to be smaller.  Host code only, without
// HIP: compiled by the library and by its CPU test.
#pragma once
#include <stdint.h>

namespace spdz {

inline int64_t up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// The next smaller panel of pm rows and pn columns, whole tiles of tm x tn: halves the longer side
// that has more than one tile, so every sequence of calls ends at one tile.  False there (unchanged).
inline bool smaller_panel(int64_t &pm, int64_t &pn, int64_t tm, int64_t tn) {
  if (pm <= tm && pn <= tn) return false;
  if (pm > tm && (pm >= pn || pn <= tn)) pm = up((pm + 1) / 2, tm);
  else pn = up((pn + 1) / 2, tn);
  return true;
}

}  // namespace spdz
