// Checks of the launch rules in csrc/ckv_plan.h against brute force (host only).
#include "ckv_plan.h"

#include <climits>
#include <cstdio>
#include <cstdlib>
#include <random>

using namespace ckv;

#define CHECK(x)                                                  \
  do {                                                            \
    if (!(x)) {                                                   \
      std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x);         \
      std::exit(1);                                               \
    }                                                             \
  } while (0)

static ByteRange range(int lo, int hi) { return ByteRange{(uintptr_t)lo, (uintptr_t)hi}; }

// RangeSet against a bitmap: empty, touching, nested and joining ranges
static void range_set() {
  std::mt19937 rng(1);
  for (int trial = 0; trial < 2000; ++trial) {
    RangeSet s;
    std::vector<bool> bit(64, false);
    for (int k = 0; k < 12; ++k) {
      const int a = 1 + rng() % 60, b = 1 + rng() % 60;   // empty when a >= b
      bool want = false;
      for (int i = a; i < b; ++i) want = want || bit[i];
      CHECK(s.hits(range(a, b)) == want);
      s.add(range(a, b));
      for (int i = a; i < b; ++i) bit[i] = true;
      size_t runs = 0;
      for (int i = 1; i < 64; ++i) runs += bit[i] && !bit[i - 1];
      CHECK(s.size() == runs);
    }
  }
  CHECK(byte_range(nullptr, 8).empty() && byte_range(&rng, 0).empty());
}

// A run's members against every pair of them
static void run_memory() {
  std::mt19937 rng(2);
  for (int trial = 0; trial < 5000; ++trial) {
    struct Problem { ByteRange r[2], w[2]; };
    std::vector<Problem> run;
    RunMemory mem;
    auto overlap = [](const ByteRange& x, const ByteRange& y) {
      return !x.empty() && !y.empty() && x.lo < y.hi && y.lo < x.hi;
    };
    for (int k = 0; k < 6; ++k) {
      Problem p;
      for (ByteRange* x : {p.r, p.w})
        for (int i = 0; i < 2; ++i) {
          const int lo = 1 + rng() % 200;
          x[i] = range(lo, lo + rng() % 9);
        }
      bool ok = true;
      for (const Problem& q : run)
        for (int i = 0; i < 2; ++i)
          for (int j = 0; j < 2; ++j)
            ok = ok && !overlap(p.w[i], q.w[j]) && !overlap(p.w[i], q.r[j]) && !overlap(p.r[i], q.w[j]);
      CHECK(mem.independent(p.r, p.w) == ok);
      if (!ok) continue;
      mem.add(p.r, p.w);
      run.push_back(p);
    }
  }
}

// The joint test's fix-up: the partial sums of the pairs that go together fit
// the workspace, and the segments cover the row
static void joint_fixup() {
  std::vector<int> lengths = {1, 255, 256, 257, 32768, 131072, (1 << 24) - 1, 30720 * 1024 - 1, 30720 * 1024,
                              30720 * 1024 + 1, 100000000, INT_MAX - 1024};
  std::mt19937 rng(3);
  for (int k = 0; k < 2000; ++k) lengths.push_back(1 + rng() % (INT_MAX - 1024));
  for (int S : lengths)
    for (int n : {1, 2, 31, 64, 1000, 32768, 2097152}) {
      const int seg = joint_segment(n, S), parts = joint_segments(seg, S);
      CHECK(seg >= 256 && seg <= kFixSegMax);
      CHECK((int64_t)(parts - 1) * seg < S && (int64_t)parts * seg >= S);
      CHECK((int64_t)std::min(n, joint_pairs(parts)) * parts <= joint_fix_items(S));
    }
}

// The joint test's workgroups on devices of any size: every row is owned, no
// more workgroups than the device holds, and the LDS form only where its rows fit
static void joint_workgroups() {
  for (int resident : {1, 2, 16, 32, 38, 64, 128, 255, 256, 304, 512, 4096})
    for (int rows = 1; rows <= 1 << 20; rows += 1 + rows / 64) {
      const int nb = joint_blocks(rows, resident), per = (rows + nb - 1) / nb;
      CHECK(nb >= 1 && nb <= resident && nb <= kJointBlocksMax);
      CHECK((int64_t)nb * per >= rows);
      CHECK(joint_state_global(rows, resident) == (per > kJointRowsLds));
      // a whole device keeps 64 rows a workgroup in LDS
      if (resident >= kJointBlocksMax) CHECK(joint_state_global(rows, resident) == (rows > 64 * 256));
    }
  // 64 heads of 128 rows on 32 compute units
  CHECK(joint_state_global(64 * 128, 32) && !joint_state_global(32 * 64, 32));
}

// Shares against every share: within the limit, and no share that needs up to 7
// rounds more than the fewest possible gives a cheaper launch
static void shares() {
  std::mt19937 rng(4);
  for (int trial = 0; trial < 3000; ++trial) {
    Shares s;
    struct Problem { int n, u; };
    std::vector<Problem> ps;
    for (int k = 1 + rng() % 8; k > 0; --k) {
      Problem p{(int)(rng() % (trial % 2 ? 40 : 300)), (int)(1 + rng() % 64)};
      if (k % 3 == 0 && !ps.empty()) p = ps.back();
      ps.push_back(p);
      s.add(p.n, p.u);
    }
    auto blocks = [&](int share) {
      int64_t b = 0;
      for (const Problem& p : ps) b += (int64_t)((p.n + share - 1) / share) * p.u;
      return b;
    };
    const int resident = trial % 3 ? 256 : 512, limit = 1 + rng() % 256;
    const float start = (rng() % 9) * 0.5f;
    const int best = s.best(resident, limit, start);
    CHECK(best >= 1 && best <= limit);
    int most = 1;
    for (const Problem& p : ps) most = std::max(most, p.n);
    if (blocks(1) == 0) continue;
    auto rounds = [&](int share) { return (blocks(share) + resident - 1) / resident; };
    const int top = std::min(limit, most);
    const float cost = rounds(best) * (best + start);
    for (int share = 1; share <= top; ++share) {
      CHECK(s.workgroups(share) == blocks(share));
      if (rounds(share) < rounds(top) + 8) CHECK(cost <= rounds(share) * (share + start) * 1.0001f);
    }
  }
  // three problems of 1024 pages in 32 places: whole rounds
  Shares s;
  for (int i = 0; i < 3; ++i) s.add(1024, 32);
  CHECK(s.workgroups(s.best(256, 256, 3.f)) % 256 == 0);
  CHECK(Shares().best(256, 64, 3.f) == 1);
}

// Candidates of a checkpoint: every one below the count is taken once, and
// nothing past the shortest array that callers pass is read before the count
static void candidates() {
  for (int threads : {1, 4, 256})
    for (int max_cand : {1, 2, 3, 7, 255, 256, 257, 600})
      for (int n_pages : {0, 1, 2, 5, 113, 256, 300, 1000})
        for (int nc = 0; nc <= max_cand; nc += 1 + max_cand / 9) {
          const int ahead = candidates_ahead(max_cand, n_pages);
          std::vector<int> taken(max_cand, 0);
          for (int tid = 0; tid < threads; ++tid) {
            if (tid < ahead) CHECK(tid < max_cand && tid < n_pages);
            if (tid < std::min(nc, ahead)) ++taken[tid];
            for (int i = first_candidate_left(tid, ahead, threads); i < nc; i += threads) ++taken[i];
          }
          for (int i = 0; i < max_cand; ++i) CHECK(taken[i] == (i < nc ? 1 : 0));
        }
}

int main() {
  range_set();
  run_memory();
  shares();
  candidates();
  joint_workgroups();
  joint_fixup();
  std::printf("plan checks passed\n");
  return 0;
}
