// How the requests of a batched plan are cut into tiles, and the order of the
// tiles where every workgroup takes one.  Plain host C++.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <numeric>
#include <utility>
#include <vector>

namespace pdfmi {

constexpr int kBatchThreads = 1024, kBatchSmall = 768, kBatchHalf = 512;  // threads of a workgroup
constexpr size_t kXcds = 8;

// A request: points, columns.
struct TileReq {
  int64_t n;
  int R;
};

// How a plan is cut: points per tile, threads per workgroup.
struct BatchTiling {
  int points, block;
};

// The requests of a plan are cut into tiles of at most `asked` points.  A plan
// of few tiles takes smaller ones, down to one pass of a workgroup, where it
// then ends sooner.  The time is estimated in half passes: a tile takes its
// passes and about one for the staging of the grid, or half of one for the
// tables alone.  The compute units share the tiles, so the time is at least
// their mean and, for every k, k + 1 of the tiles that the first k rounds leave;
// the costliest come first where grids are in LDS, else the compute units end
// half a tile apart on the average.  Grids in global memory are read column by
// column, so a pass there counts by its columns against the plan's mean: 12
// requests of 580000 points in all, 1 to 11 columns, FP64: 65 us in the tiles of
// 4096 points that were taken without this, 43 in those of 1024 (60 such plans,
// 4096 asked: 1.14 times the time of the best size on the average, so 1.01).
inline BatchTiling batch_tiling(bool lds, int asked, const std::vector<TileReq>& reqs, int n_cu) {
  int64_t half = 0;
  double points = 0.0, evals = 0.0;
  for (const TileReq& r : reqs) {
    half += (r.n + kBatchHalf - 1) / kBatchHalf;
    points += (double)r.n;
    evals += (double)r.n * r.R;
  }
  if (!lds && asked >= kBatchHalf && half <= 2 * (int64_t)n_cu) return {kBatchHalf, kBatchHalf};
  BatchTiling best{asked, kBatchThreads};
  int64_t tiles = 0;
  for (const TileReq& r : reqs) tiles += (r.n + asked - 1) / asked;
  if (tiles >= (lds ? 2 : 4) * (int64_t)n_cu) return best;
  const int setup = lds ? 2 : 1;
  std::vector<std::pair<double, int64_t>> kinds;  // cost of a tile, number of such tiles
  auto time_of = [&](int size) {
    kinds.clear();
    tiles = 0;
    for (const TileReq& r : reqs) {
      auto add = [&](int64_t p, int64_t count) {
        const double passes = (double)((p + kBatchThreads - 1) / kBatchThreads);
        if (count > 0) kinds.push_back({2.0 * passes * (lds ? 1.0 : r.R * points / evals) + setup, count});
        tiles += count;
      };
      add(size, r.n / size);
      add(r.n % size, r.n % size > 0);
    }
    std::sort(kinds.begin(), kinds.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
    double work = 0.0, least = 0.0;
    int64_t before = 0;  // tiles at least as costly
    for (const auto& k : kinds) {
      before += k.second;
      work += k.first * (double)k.second;
      least = std::max(least, (double)((before - 1) / n_cu + 1) * k.first);
    }
    work /= n_cu;
    return std::max(least, tiles <= n_cu || lds ? work : work + 0.5 * kinds[0].first);
  };
  double least = time_of(asked);
  for (int t = asked; t > kBatchThreads;) {
    t = std::max(kBatchThreads, (t / 2 + 63) / 64 * 64);
    const double c = time_of(t);
    if (c < least) {
      least = c;
      best.points = t;
    }
  }
  return best;
}

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
