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

// Candidates of a checkpoint's accepted pages that are read before their number
// is known: candidate arrays hold max_cand entries, or one per page where they
// come from the classification.  Thread `tid` of `threads` reads candidate tid
// of these and then, from first_candidate_left on, every threads-th of the rest.
constexpr int candidates_ahead(int max_cand, int n_pages) { return std::min(max_cand, n_pages); }
constexpr int first_candidate_left(int tid, int ahead, int threads) { return tid < ahead ? tid + threads : tid; }

// Units that one workgroup of a launch takes (pages, or splits of a row block).
// Problem i has n[i] units in each of u[i] places, the device holds `resident`
// workgroups at once, and a workgroup costs its units and `start` units to
// begin.  The launch lasts as many rounds as its workgroups fill the device,
// so the share is the smallest one that fits into the number of rounds for
// which rounds * (share + start) is least: shares between those only add a
// nearly empty last round (three problems of 1024 pages in 32 places: 193
// pages a workgroup made 576 workgroups, three rounds of 256, and took 1.5
// times as long as three launches).
class Shares {
 public:
  void add(int n, int u) {
    if (n <= 0 || u <= 0) return;
    if (!g_.empty() && g_.back().n == n) g_.back().u += u;
    else g_.push_back({n, u});
    most_ = std::max(most_, n);
    total_ += (int64_t)n * u;
  }
  int64_t workgroups(int share) const {
    int64_t b = 0;
    for (const Group& g : g_) b += ((g.n - 1) / share + 1) * g.u;
    return b;
  }
  int best(int resident, int limit, float start) const {
    limit = std::max(1, std::min(limit, most_));
    if (g_.empty()) return limit;
    const int64_t min_rounds = (workgroups(limit) - 1) / resident + 1;
    int best = limit;
    float least = -1.f;
    for (int64_t r = std::max<int64_t>(1, min_rounds); r < min_rounds + 8; ++r) {
      int share = (int)std::min<int64_t>(limit, std::max<int64_t>(1, (total_ - 1) / (r * resident) + 1));
      while (share < limit && workgroups(share) > r * resident) ++share;
      const float cost = r * (share + start);
      if (least < 0.f || cost < least) {
        least = cost;
        best = share;
      }
      if (share == 1) break;
    }
    return best;
  }

 private:
  struct Group { int n; int64_t u; };
  std::vector<Group> g_;
  int most_ = 0;
  int64_t total_ = 0;
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
