// Order of a plan's tiles where every workgroup takes one.  Plain host C++.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <numeric>
#include <vector>

namespace pdfmi {

constexpr size_t kXcds = 8;

// The tile at each place of the list, of which each XCD takes a contiguous run
// (one more tile for the first of them if 8 does not divide their number):
// costliest first, the tiles of one cost dealt out evenly over the XCDs and, to
// each, neighbours.  In the order of the requests an XCD can get only the
// costly ones, and dealt out one by one the tiles of a member are on every XCD.
inline std::vector<size_t> deal_tiles(const std::vector<int64_t>& cost) {
  const size_t n = cost.size(), per = n / kXcds, rest = n % kXcds;
  std::vector<size_t> order(n), at(n);
  std::iota(order.begin(), order.end(), (size_t)0);
  std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return cost[a] > cost[b]; });
  for (size_t b = 0, e = 0; b < n; b = e) {
    while (e < n && cost[order[e]] == cost[order[b]]) ++e;
    size_t next = b;
    for (size_t x = 0; x < kXcds; ++x)  // its places among [b, e), were they dealt out one by one
      for (size_t i = b + (x + kXcds - b % kXcds) % kXcds; i < e; i += kXcds)
        at[x * per + std::min(x, rest) + i / kXcds] = order[next++];
  }
  return at;
}

}  // namespace pdfmi
