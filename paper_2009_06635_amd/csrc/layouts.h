// Shape of the compacted copies of a member's values (one request's columns
// in request order), and which requests get one.  Plain host C++.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <vector>

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

// A request: stored columns in request order (-1: absent) and precision.
struct LayoutKey {
  bool f32 = false;
  int n = 0;
  signed char col[64] = {};
  bool operator==(const LayoutKey& o) const { return f32 == o.f32 && n == o.n && memcmp(col, o.col, (size_t)n) == 0; }
};

constexpr size_t kMaxLayouts = 8;                    // copies of a member
constexpr int64_t kLayoutPoints = (int64_t)1 << 21;  // points of a request after which it gets one
constexpr int64_t kLayoutBytes = (int64_t)16 << 20;  // largest copy
constexpr size_t kMaxWanted = 64;                    // requests without a copy that are counted

inline bool layout_small(bool f32, int64_t rows, int stride) {
  return rows * stride * (f32 ? 4 : 8) <= kLayoutBytes;
}

// The points asked for by requests that have no copy.  A request that is new
// when the list is full takes the place of the one with the fewest points, so
// requests that come often are counted whatever else has been asked before.
class LayoutsWanted {
 public:
  // n more points of the request; true once it has asked for kLayoutPoints.
  bool add(const LayoutKey& key, int64_t n) {
    Entry* e = find(key);
    if (!e && list_.size() < kMaxWanted) {
      list_.push_back(Entry());
      e = &list_.back();
    }
    if (!e) {
      e = &list_[0];
      for (Entry& c : list_)
        if (c.points < e->points) e = &c;
    }
    if (!(e->key == key)) *e = Entry{key, 0};
    e->points += n;
    return e->points >= kLayoutPoints;
  }
  // Its copy could not be made: counted afresh.
  void again(const LayoutKey& key) {
    if (Entry* e = find(key)) e->points = 0;
  }
  // It has its copy.
  void remove(const LayoutKey& key) {
    if (Entry* e = find(key)) {
      *e = list_.back();
      list_.pop_back();
    }
  }

 private:
  struct Entry {
    LayoutKey key;
    int64_t points = 0;
  };
  Entry* find(const LayoutKey& key) {
    for (Entry& e : list_)
      if (e.key == key) return &e;
    return nullptr;
  }
  std::vector<Entry> list_;
};

}  // namespace pdfmi
