// Shape of the compacted copies of a member's values (one request's columns
// in request order).  Plain host C++.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace pdfmi {

// Columns that one lane reads together from a copy of n columns: 16 bytes,
// fewer where there are fewer columns.
inline int layout_group(int n, bool f32) { return f32 ? (n >= 4 ? 4 : (n >= 2 ? 2 : 1)) : (n >= 2 ? 2 : 1); }

// Values per row of a copy of n columns and `rows` rows: whole 16-byte groups
// where such rows fit the lds_left bytes that a launch can give to the values,
// else 13 to 16 columns padded to full lines, fewer packed.
inline int layout_stride(int n, bool f32, int64_t rows, int64_t lds_left) {
  const int g = f32 ? 4 : 2, es = f32 ? 4 : 8;
  const int whole = (n + g - 1) / g * g;
  if (rows * whole * es <= lds_left) return whole;
  return n > 12 ? (n + 15) & ~15 : n;
}

// May such a copy be staged in LDS?  A lane reads a group with one aligned
// load, and a row's last group may run past its columns: rows have to be whole
// groups.  (Packed rows can be short enough for LDS where whole ones are not.)
inline bool layout_stageable(int n, bool f32, int stride) { return stride % layout_group(n, f32) == 0; }

}  // namespace pdfmi
