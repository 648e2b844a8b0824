// Host-side rules that decide how calls are launched, free of HIP so that they
// can be compiled and checked on their own.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace ckv {

// Bytes [lo, hi) of device memory; empty when lo >= hi.
struct ByteRange {
  uintptr_t lo = 0, hi = 0;
  bool empty() const { return lo >= hi; }
};

inline ByteRange byte_range(const void* p, int64_t bytes) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(p);
  return p && bytes > 0 ? ByteRange{a, a + (uintptr_t)bytes} : ByteRange{};
}

// A union of ranges, kept disjoint and ascending (ranges that touch are joined,
// so the layers of one allocation stay one range).
class RangeSet {
 public:
  bool hits(const ByteRange& x) const {
    if (x.empty()) return false;
    const auto it = std::upper_bound(v_.begin(), v_.end(), x.lo,
                                     [](uintptr_t a, const ByteRange& r) { return a < r.hi; });
    return it != v_.end() && it->lo < x.hi;
  }
  void add(ByteRange x) {
    if (x.empty()) return;
    auto b = std::lower_bound(v_.begin(), v_.end(), x.lo,
                              [](const ByteRange& r, uintptr_t a) { return r.hi < a; });
    auto e = b;
    for (; e != v_.end() && e->lo <= x.hi; ++e) {
      x.lo = std::min(x.lo, e->lo);
      x.hi = std::max(x.hi, e->hi);
    }
    if (b == e) {
      v_.insert(b, x);
    } else {
      *b = x;
      v_.erase(b + 1, e);
    }
  }
  size_t size() const { return v_.size(); }

 private:
  std::vector<ByteRange> v_;
};

// The problems of one launch run beside each other, so they may share what
// they read but not what any of them writes.
class RunMemory {
 public:
  template <int NR, int NW>
  bool independent(const ByteRange (&reads)[NR], const ByteRange (&writes)[NW]) const {
    for (const ByteRange& w : writes)
      if (w_.hits(w) || r_.hits(w)) return false;
    for (const ByteRange& r : reads)
      if (w_.hits(r)) return false;
    return true;
  }
  template <int NR, int NW>
  void add(const ByteRange (&reads)[NR], const ByteRange (&writes)[NW]) {
    for (const ByteRange& r : reads) r_.add(r);
    for (const ByteRange& w : writes) w_.add(w);
  }

 private:
  RangeSet r_, w_;
};

// Workgroups of the joint test (8 waves each) for so many window rows: about
// one row per wave, at most as many as the device holds at once and one per
// compute unit of a whole device.
constexpr int kJointWaves = 8;
constexpr int kJointBlocksMax = 256;
constexpr int kJointRowsLds = 64;       // rows whose state a workgroup keeps in LDS at most
constexpr int joint_blocks(int rows, int resident) {
  return std::max(1, std::min({(rows - 1) / kJointWaves + 1, resident, kJointBlocksMax}));
}
// Whether the rows' state has to live in global memory: where the workgroups
// that the device holds of the LDS form would own more rows than fit (above
// 16384 rows on 256 compute units, above 2048 on a partition of 32).
constexpr bool joint_state_global(int rows, int resident) {
  return (rows - 1) / joint_blocks(rows, resident) + 1 > kJointRowsLds;
}

// Fix-up of the joint test: a listed (candidate, row) pair is recomputed from
// segments of its row, one workgroup and one partial sum each, and the pairs
// whose partial sums fit the workspace go together (at least one).
constexpr int kJointFixItems = 30720;   // (pair, segment) items aimed at
constexpr int kFixSegMax = 1024;        // tokens of a segment at most

// tokens per segment for n listed pairs over S tokens: short segments while
// the items are few
constexpr int joint_segment(int n, int S) {
  int seg = 256;
  while (seg < kFixSegMax && (int64_t)n * ((S - 1) / seg + 1) > 32 * 256) seg *= 2;
  return seg;
}
constexpr int joint_segments(int seg, int S) { return (S - 1) / seg + 1; }
// pairs recomputed together
constexpr int joint_pairs(int segments) { return std::max(1, kJointFixItems / segments); }
// items of the workspace: those, or the segments of one pair where a paged
// cache is longer than all of them (31.4 million tokens)
constexpr int joint_fix_items(int S) { return std::max(kJointFixItems, joint_segments(kFixSegMax, S)); }

}  // namespace ckv
