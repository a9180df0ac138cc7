"""Tiles of batched plans (csrc/tiles.h), on the CPU.  Their order where every
workgroup takes one: every tile is there once, every XCD's run starts with its costliest
tiles and has as many of each cost as the others, give or take one, and tiles
of one cost are neighbours in it -- over all numbers of tiles that such a plan
can have and few or many different costs.  Their size: a plan is not longer for
one costly tile than the compute units' share of all of it, over requests of
uneven points and columns; requests of one number of columns are cut alike
whatever that number is."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <map>
#include "tiles.h"
using namespace pdfmi;
int main() {
  long bad[4] = {};
  unsigned seed = 1;
  for (size_t n = 0; n <= 600; ++n)
    for (unsigned costs : {1u, 2u, 11u, 1000u}) {
      std::vector<int64_t> cost(n);
      for (int64_t& c : cost) c = (int64_t)((seed = seed * 1664525u + 1013904223u) >> 8) % costs;
      const std::vector<size_t> at = deal_tiles(cost);
      std::vector<int> seen(n);
      for (size_t t : at) ++seen[t];
      bad[0] += at.size() != n || std::count(seen.begin(), seen.end(), 1) != (long)n;
      std::map<int64_t, std::vector<int>> share;
      for (size_t x = 0, i = 0; x < 8; ++x) {
        const size_t end = i + n / 8 + (x < n % 8);
        std::map<int64_t, std::vector<size_t>> got;
        for (size_t j = i; j < end; ++j) {
          bad[1] += j > i && cost[at[j]] > cost[at[j - 1]];
          got[cost[at[j]]].push_back(at[j]);
        }
        for (auto& g : got) {
          share[g.first].resize(8);
          share[g.first][x] = (int)g.second.size();
          for (size_t k = 1; k < g.second.size(); ++k) {  // no other tile of this cost between two of them
            bad[2] += g.second[k] < g.second[k - 1];
            for (size_t m = g.second[k - 1] + 1; m < g.second[k]; ++m) bad[2] += cost[m] == g.first;
          }
        }
        i = end;
      }
      for (auto& s : share)
        bad[3] += *std::max_element(s.second.begin(), s.second.end()) > 1 + *std::min_element(s.second.begin(), s.second.end());
    }
  std::printf("%ld %ld %ld %ld\n", bad[0], bad[1], bad[2], bad[3]);
  return 0;
}
"""

SIZES = r"""
#include <cmath>
#include <cstdio>
#include "tiles.h"
using namespace pdfmi;
int main() {
  const int n_cu = 256;
  long plans = 0, long_tiles = 0, differ = 0, above = 0;
  unsigned seed = 7;
  auto rnd = [&](int n) { return (int)((seed = seed * 1664525u + 1013904223u) >> 8) % n; };
  for (int p = 0; p < 3000; ++p) {
    std::vector<TileReq> uneven, ones, many;
    const int n_req = 1 + rnd(200);
    for (int i = 0; i < n_req; ++i) {
      const int64_t n = (int64_t)std::exp(6.9 + rnd(1000) * 0.005);
      uneven.push_back({n, 1 + rnd(11)});
      ones.push_back({n, 1});
      many.push_back({n, 13});
    }
    const int asked = 1024 << rnd(5);
    for (bool lds : {false, true}) {
      const BatchTiling a = batch_tiling(lds, asked, ones, n_cu), b = batch_tiling(lds, asked, many, n_cu);
      differ += a.points != b.points || a.block != b.block;
    }
    const BatchTiling t = batch_tiling(false, asked, uneven, n_cu);
    above += t.points > asked;
    if (t.block == kBatchHalf) continue;
    double work = 0.0, longest = 0.0;
    for (const TileReq& r : uneven) {
      work += (double)r.n * r.R / n_cu;
      longest = std::max(longest, (double)std::min<int64_t>(r.n, t.points) * r.R);
    }
    ++plans;
    long_tiles += t.points > kBatchThreads && longest > 2.0 * work;
  }
  std::printf("%ld %ld %ld %ld\n", plans, long_tiles, differ, above);
  return 0;
}
"""


def run(tmp_path, source):
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2009_06635_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    return [int(v) for v in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]


def test_tiles_of_a_cost_are_dealt_evenly_and_in_runs(tmp_path):
    assert run(tmp_path, SOURCE) == [0] * 4


def test_no_plan_waits_for_one_costly_tile(tmp_path):
    plans, long_tiles, differ, above = run(tmp_path, SIZES)
    assert plans > 1000 and long_tiles == differ == above == 0
