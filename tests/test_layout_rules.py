"""Rules of the compacted copies (csrc/layouts.h), on the CPU: a copy that a
launch may stage in LDS has rows in which every group of columns is aligned to
its own size and lies inside its row, over all column counts, both precisions
and every row count around the LDS limit; a request that comes often reaches
its copy whatever other requests came before it or come between."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "layouts.h"
using namespace pdfmi;
int main() {
  long checked = 0, staged_packed = 0, bad = 0;
  for (int f32 = 0; f32 < 2; ++f32)
    for (int n = 1; n <= 40; ++n)
      for (long room = 20000; room <= 100000; room += 1111)
        for (long rows = 16; rows < 9000; rows += 1 + rows / 97) {
          const int es = f32 ? 4 : 8, g = layout_group(n, f32);
          const int stride = layout_stride(n, f32, rows, room);
          if (stride < n) ++bad;
          const bool fits = rows * stride * es <= room;  // what the launch looks at
          if (!fits || !layout_stageable(n, f32, stride)) continue;
          ++checked;
          staged_packed += stride % (16 / es) != 0;
          for (int j = 0; j < n; j += g)  // row r starts at r * stride: aligned for every r if stride is
            if (stride % g || j + g > stride) ++bad;
        }
  std::printf("%ld %ld %ld\n", checked, staged_packed, bad);
  return 0;
}
"""

WANTED = r"""
#include <cstdio>
#include "layouts.h"
using namespace pdfmi;
LayoutKey key(int a, int b, bool f32) {
  LayoutKey k;
  k.f32 = f32;
  k.n = 2;
  k.col[0] = (signed char)a;
  k.col[1] = (signed char)b;
  return k;
}
// calls until the hot request (n points a call) has its copy, `others` different small ones between two of its calls
int calls(int before, int others, int64_t n) {
  LayoutsWanted w;
  for (int i = 0; i < before; ++i) w.add(key(i % 60, i / 60, i & 1), 1);
  for (int c = 1, o = 0; c < 10000; ++c) {
    if (w.add(key(61, 61, false), n)) return c;
    for (int i = 0; i < others; ++i, ++o) w.add(key(o % 60, o / 60 % 60, o & 1), 1);
  }
  return -1;
}
int main() {
  LayoutsWanted w;
  const bool first = w.add(key(1, 2, false), kLayoutPoints), f32 = w.add(key(1, 2, true), kLayoutPoints - 1);
  w.again(key(1, 2, false));
  const bool fresh = w.add(key(1, 2, false), 1);
  w.remove(key(1, 2, true));
  const bool removed = w.add(key(1, 2, true), 1);
  std::printf("%d %d %d %d %d %d %d %d\n", calls(0, 0, 1 << 20), calls(1000, 0, 1 << 20), calls(1000, 200, 1 << 20),
              calls(8, 1, 1 << 15), first, f32, fresh, removed);
  return 0;
}
"""


def run(tmp_path, source):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2009_06635_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return [int(v) for v in out.split()]


def test_requests_reach_their_copy(tmp_path):
    assert run(tmp_path, WANTED) == [2, 2, 2, 64, 1, 0, 0, 0]


def test_staged_rows_hold_whole_groups(tmp_path):
    checked, packed, bad = run(tmp_path, SOURCE)
    assert checked > 100_000 and packed > 100   # rows shorter than 16 bytes are among them
    assert bad == 0
