"""Rules of the compacted copies (csrc/layouts.h), on the CPU: a copy that a
launch may stage in LDS has rows in which every group of columns is aligned to
its own size and lies inside its row, over all column counts, both precisions
and every row count around the LDS limit."""
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


def test_staged_rows_hold_whole_groups(tmp_path):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2009_06635_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    checked, packed, bad = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert checked > 100_000 and packed > 100   # rows shorter than 16 bytes are among them
    assert bad == 0
