"""Order of the tiles of a plan with one tile per workgroup (csrc/tiles.h), on
the CPU: every tile is there once, every XCD's run starts with its costliest
tiles and has as many of each cost as the others, give or take one, and tiles
of one cost are neighbours in it -- over all numbers of tiles that such a plan
can have and few or many different costs."""
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


def test_tiles_of_a_cost_are_dealt_evenly_and_in_runs(tmp_path):
    src, exe = tmp_path / "order.cpp", tmp_path / "order"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2009_06635_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split() == ["0"] * 4
