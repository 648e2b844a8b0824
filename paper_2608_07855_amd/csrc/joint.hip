// Greedy joint retirement test (CommitKV, Sec. 3.3, Eq. (11), Algorithm 1).
//
// For a page set X deleted at once, Eq. (6) gives, per window row,
//   o - o^{\X} = (sum_{E in X} r_E) / (1 - sum_{E in X} A_E),
//   r_E = sum_{i in E} a_i v_i - A_E o,
// so the union effect follows from per-page residuals r_E (computed once per
// candidate by the page kernel in residual mode) and the running sums
// D = sum_{E in A} r_E, A_A = sum_{E in A} A_E over the accepted set A.
//
// The greedy loop is evaluated in speculative rounds.  A round tests the next
// kJointWindow candidates under two guesses at once, from one read of their
// residuals: every candidate alone against the accepted set ("independent",
// right as long as the ones before it are rejected), and every candidate on
// top of all earlier ones of the round ("chain", right as long as those are
// accepted; the sums are added in the order in which single acceptances would
// add them).  The decision takes the chain up to its first failure, which it
// rejects, or, when the first candidate fails, the rejections up to the first
// candidate that passes, which it accepts.  Candidates come in the order of
// their own effects, so a call is mostly one run of acceptances and then
// rejections, and nearly every round decides many: the case of 206 candidates
// and 42-54 acceptances (32768 tokens, 2048 window rows) takes 9-14 rounds
// where testing against the accepted set alone took one per acceptance.
//
// All rounds run in one launch of at most as many workgroups as the device
// holds at once.  Workgroup b owns the window rows [b * rpb, (b + 1) * rpb)
// for the whole call and keeps their state (D, A_A, visible counts) to
// itself, in LDS (or its own part of global memory when a workgroup owns
// more than kRowsOwnedMax rows), so a round reads only the candidates'
// residual rows and publishes one maximum per candidate and guess.  The
// workgroups that arrive last reduce the maxima, the very last one decides
// and publishes the decision in one 64-bit word that the others poll: one
// grid-wide wait per round.  Everything that crosses workgroups moves through agent-scope
// atomics, so no fence (which would write back and invalidate the XCD's
// whole L2) is needed.  The candidate count is read on the device, so the
// call needs no host round trip; each round decides at least one candidate,
// so the loop ends within max_cand rounds.  A wait is bounded: if the
// workgroups cannot all run at once (a device shared with other work), every
// block leaves and *n_accepted = -1.
//
// A union that holds nearly all of a row's attention mass makes Eq. (6)
// ill-conditioned: o - o^{\X} = D / (1 - A_X) divides float32 cancellation
// by a small 1 - A_X.  A (candidate, row) pair whose union mass exceeds
// kJointFixA is left out of the closed form and recomputed by definition --
// the row's output over the tokens outside the union, o', in float32 from
// the keys and values -- and the ratio ||o - o'|| / ||o|| joins the
// candidate's maximum.  The union of candidate t is t and the accepted
// candidates before t, which the final decisions determine, so pairs of
// decided candidates are listed and recomputed together after the last
// round (they only enter union_R: a candidate whose other rows already
// exceed tau is rejected whatever they give).  A candidate that only such
// pairs can decide is resolved at once.  Pairs of candidates a round tested
// but did not decide are dropped.
#include "ckv_device.h"
#include "ckv_kernels.h"
#include "ckv_plan.h"

#include <algorithm>
#include <atomic>
#include <climits>

namespace ckv {

// Control words (cleared by the residual pass before this kernel starts),
// each on a 128-byte line of its own: pollers of the decision word and the
// arrival counts do not meet.  Arrivals are counted in groups of kJointGroup
// workgroups, then over the groups.
constexpr int kLine = 32;   // ints
enum { kWord = 0, kError = kLine, kFixN = 2 * kLine, kTop = 3 * kLine, kGroup0 = 4 * kLine };
constexpr int kJointGroup = 16;
static_assert(kGroup0 + 16 * kLine == kJointCtrlWords, "control words");
// payload of a decision: mode (1: chain) | n << 1 | extra << 7 | flags
constexpr unsigned kDecChain = 1u, kDecExtra = 1u << 7, kDecResolve = 1u << 8, kDecDefer = 1u << 9,
                   kDecFlush = 1u << 10;
constexpr int kVisSlice = 8192;        // tokens per visible-count item
constexpr int kJW = kJointWaves, kJT = 64 * kJW;   // waves and threads of a workgroup
constexpr int kCandBatch = 16;         // candidates reduced together
static_assert(kJointWindow == 2 * kCandBatch, "a round's maxima fill one wave: window x 2 guesses");

template <class T>
__device__ __forceinline__ T ld_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void st_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void store_pair(int* p, int2 v) {
  st_agent(p, v.x);
  st_agent(p + 1, v.y);
}
__device__ __forceinline__ int2 load_pair(const int* p) { return make_int2(ld_agent(p), ld_agent(p + 1)); }

// v[0..31] per lane -> the sum over the wave's 64 lanes of value lane / 2
// (each exchange step keeps half of the values).  The order of the additions
// is that of a butterfly over lane offsets 32, 16, 8, 4, 2, 1.
__device__ __forceinline__ float reduce_scatter32(float (&v)[32], int lane) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 16]), false, false);
    v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 8]), false, false);
    v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int off = 8, n = 4; off >= 2; off >>= 1, n >>= 1) {
    const bool up = (lane & off) != 0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const float mine = up ? v[i + n] : v[i], other = up ? v[i] : v[i + n];
      v[i] = mine + __shfl_xor(other, off, 64);
    }
  }
  return v[0] + __shfl_xor(v[0], 1, 64);
}

// The state of the workgroup's rows: in LDS, or in its rows' part of global
// memory.  A row belongs to one wave, and every lane writes what it reads
// back (A, C, onorm, nvis, the fix bits: all lanes the same value).
struct RowState {
  float* D;                   // [nr][D]
  float* A;
  int* C;
  float* onorm;
  int* nvis;
  unsigned long long* fix;    // [nr][2]: pairs left to the fix-up, bit 2 * candidate (+ 32: chain) per batch
};

// Folds the candidates [f0, f0 + nf) accepted last round into the rows'
// state, then tests the candidates from `cursor` on under both guesses.
// Memory-bound: a round reads rows x window x D floats (32 MB at 2048 rows,
// d = 128), so a wave issues all loads of a row's window before the first use.
template <int D>
__device__ void joint_tests(const JointArgs& j, const RowState& st, int rb0, int nr, int cursor, int n_eff, int f0,
                            int nf, unsigned* sMax, int* sAny) {
  constexpr int KD = D / 64, NB = kJointWindow / kCandBatch;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kind = lane >> 5, cq = (lane >> 1) & 15;
  unsigned wmax[NB];
  int wany[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) { wmax[b] = 0u; wany[b] = 0; }
  for (int r = wave; r < nr; r += kJW) {
    const int row = rb0 + r;
    // this row's candidates sit together: 32-bit offsets from the row's base
    const size_t rbase = (size_t)CKV_IDX(row, j.total_rows, j.geo.dbg, 11) * j.max_cand;
    const float* rrow = j.resid + rbase * D;
    const float* arow = j.resA + rbase;
    const int* crow = j.resC + rbase;
    float tv[kJointWindow][KD];
#pragma unroll
    for (int c = 0; c < kJointWindow; ++c) {
      const int t = min(cursor + c, n_eff - 1);
#pragma unroll
      for (int k = 0; k < KD; ++k) tv[c][k] = rrow[t * D + lane + 64 * k];
    }
    const int tl = min(cursor + (lane & 31), n_eff - 1);
    const float aw = arow[tl];
    const int cw = crow[tl];
    float dv[KD];
#pragma unroll
    for (int k = 0; k < KD; ++k) dv[k] = st.D[r * D + lane + 64 * k];
    float Ac = st.A[r];
    int Cc = st.C[r];
    if (nf > 0) {
      for (int f = 0; f < nf; f += 8) {
        float fv[8][KD], fa[8];
        int fc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int t = f0 + min(f + q, nf - 1);
#pragma unroll
          for (int k = 0; k < KD; ++k) fv[q][k] = rrow[t * D + lane + 64 * k];
          fa[q] = arow[t];
          fc[q] = crow[t];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (f + q < nf) {
#pragma unroll
            for (int k = 0; k < KD; ++k) dv[k] += fv[q][k];
            Ac += fa[q];
            Cc += fc[q];
          }
      }
#pragma unroll
      for (int k = 0; k < KD; ++k) st.D[r * D + lane + 64 * k] = dv[k];
      st.A[r] = Ac;
      st.C[r] = Cc;
    }
    const float on = st.onorm[r];
    const int nv = st.nvis[r];
    // chain sums of the masses and counts: lane c holds them through candidate c
    float run = Ac, preA = 0.f;
    int crun = Cc, preC = 0;
#pragma unroll
    for (int c = 0; c < kJointWindow; ++c) {
      run += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(aw), c));
      crun += __builtin_amdgcn_readlane(cw, c);
      preA = lane == c ? run : preA;
      preC = lane == c ? crun : preC;
    }
    float pv[KD];
#pragma unroll
    for (int k = 0; k < KD; ++k) pv[k] = dv[k];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float n2[2 * kCandBatch];   // squared norms: independent, then chain
#pragma unroll
      for (int q = 0; q < kCandBatch; ++q) {
        float x2 = 0.f, y2 = 0.f;
#pragma unroll
        for (int k = 0; k < KD; ++k) {
          const float x = dv[k] + tv[kCandBatch * b + q][k];
          x2 = __builtin_fmaf(x, x, x2);
          pv[k] += tv[kCandBatch * b + q][k];
          y2 = __builtin_fmaf(pv[k], pv[k], y2);
        }
        n2[q] = x2;
        n2[kCandBatch + q] = y2;
      }
      const float s = reduce_scatter32(n2, lane);
      const int c = kCandBatch * b + cq;
      // (every lane takes both exchanges: a lane reads nothing from a lane that sits one out)
      const float A_i = Ac + __shfl(aw, c, 64), A_c = __shfl(preA, c, 64);
      const int C_i = Cc + __shfl(cw, c, 64), C_c = __shfl(preC, c, 64);
      const float Au = kind ? A_c : A_i;
      const int Cu = kind ? C_c : C_i;
      float ratio = 0.f;
      bool fix = false;
      if (cursor + c < n_eff && Cu > 0) {
        if (Cu >= nv) ratio = INFINITY;
        else if (Au > kJointFixA) fix = true;   // recomputed by definition
        else if (on > 0.f) ratio = sqrtf(s) / ((1.f - Au) * on);
        else ratio = s > 0.f ? INFINITY : 0.f;
      }
      st.fix[2 * r + b] = __ballot(fix && !(lane & 1));
      if (ratio > 0.f) wmax[b] = max(wmax[b], __float_as_uint(ratio));
      wany[b] |= fix ? 1 : 0;
    }
  }
  if (!(lane & 1)) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int w = 32 * kind + kCandBatch * b + cq;
      if (wmax[b]) atomicMax(&sMax[w], wmax[b]);
      if (wany[b]) sAny[w] = 1;
    }
  }
}

// Maxima over n <= 16 rows of 64 words (one per candidate and guess; bit 31:
// some row left the pair to the fix-up) into LDS: every load of the block at once.
__device__ void joint_reduce(const unsigned* words, int n, unsigned* sRed, int* sRedAny) {
  const int tid = threadIdx.x, w = tid & 31, b = tid >> 5;
  static_assert(kJT / 32 == kJointGroup, "one word pair per thread");
  if (tid < 64) {
    sRed[tid] = 0u;
    sRedAny[tid] = 0;
  }
  const unsigned long long v = b < n ? ld_agent(reinterpret_cast<const unsigned long long*>(words) + b * 32 + w) : 0ull;
  __syncthreads();
  const unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
  if (lo & 0x7fffffffu) atomicMax(&sRed[2 * w], lo & 0x7fffffffu);
  if (hi & 0x7fffffffu) atomicMax(&sRed[2 * w + 1], hi & 0x7fffffffu);
  if (lo >> 31) sRedAny[2 * w] = 1;
  if (hi >> 31) sRedAny[2 * w + 1] = 1;
  __syncthreads();
}

// Page ap was accepted with candidate t.  A page that is listed twice keeps the
// earlier candidate: it is gone for every candidate after that one.
__device__ __forceinline__ void mark_accepted(const JointArgs& j, int ap, int t) {
  __hip_atomic_fetch_min(&j.acc_t[ap], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The decision of a round from its maxima (the workgroup that arrives last),
// published in `word` under the wait's number.  What it stores besides is read
// behind a later arrival of this workgroup only, so the word goes first and the
// others do not wait for those stores; the loads leave before everything.
__device__ void joint_decide(const JointArgs& j, int cursor, int n_eff, const unsigned* sRed, const int* sRedAny,
                             unsigned long long* word, int epoch) {
  const int tid = threadIdx.x;
  if (tid >= 64) return;
  const int c = tid & 31, t = cursor + c;
  const float r = __uint_as_float(sRed[tid]);
  const bool any = sRedAny[tid] != 0, valid = t < n_eff;
  const int ap = valid ? j.cand[t] : -1, n_listed = ld_agent(&j.ctrl[kFixN]);
  const unsigned long long bp = __ballot(valid && (j.accept_all || (r <= j.tau && !any)));
  const unsigned long long bf = __ballot(valid && !j.accept_all && r > j.tau);
  const unsigned long long ba = __ballot(any);
  auto ones = [](unsigned x) { return x == 0xffffffffu ? 32 : __ffs(~x) - 1; };   // trailing ones
  const unsigned pass_c = (unsigned)(bp >> 32), fail_c = (unsigned)(bf >> 32);
  const unsigned pass_i = (unsigned)bp, fail_i = (unsigned)bf;
  const int m = ones(pass_c);
  const bool chain = m > 0;
  const int n = chain ? m : ones(fail_i);
  const bool extra = n < 32 && (((chain ? fail_c : pass_i) >> n) & 1u);
  const bool resolve = n == 0 && !extra;
  const int dec = n + (extra ? 1 : 0);
  const unsigned decided = dec >= 32 ? 0xffffffffu : (1u << dec) - 1u;
  const bool defer = j.want_union && ((unsigned)(chain ? ba >> 32 : ba) & decided) != 0u;
  unsigned p = (chain ? kDecChain : 0u) | (unsigned)n << 1 | (extra ? kDecExtra : 0u) |
               (resolve ? kDecResolve : 0u) | (defer ? kDecDefer : 0u);
  // empty the list first unless it has room for a whole round's pairs
  if ((defer || resolve) && n_listed > kJointWindow * j.total_rows) p |= kDecFlush;
  if (tid == 0) st_agent(word, (unsigned long long)epoch << 32 | p);
  const bool mine = (tid >> 5) == (chain ? 1 : 0);   // the lanes that hold the chosen guess
  if (mine && (c < dec || (resolve && c == 0))) st_agent(&j.ur[t], r);
  if (mine && c < dec && (chain ? c < n : c == n)) {
    st_agent(&j.accepted[t], (uint8_t)1);
    if (ap >= 0 && ap < j.n_pages) mark_accepted(j, ap, t);
  }
}

struct JointSync {
  unsigned* sRed;
  int* sRedAny;
  int* s_flag;
  unsigned long long* s_word;
  int epoch;    // grid-wide waits so far
};

// Grid-wide wait.  With `tests`, the workgroups' maxima (j.bmax) are reduced
// on the way -- by the last workgroup of each group over its group, then by
// the last group over the groups -- and that workgroup's decision travels
// back in the word the others poll: one round trip per round (about 6 us;
// two barriers of 256 arrivals at one counter with a reduction of all
// workgroups' words between them took 17).  Every wave waits for its own
// stores before its workgroup arrives.  False (in every thread) if the bound
// ran out here or elsewhere.
__device__ bool joint_sync(const JointArgs& j, JointSync& sy, bool tests, int cursor, int n_eff, unsigned* payload) {
  const int tid = threadIdx.x;
  const int grp = blockIdx.x / kJointGroup, n_grp = (gridDim.x + kJointGroup - 1) / kJointGroup;
  const int gs = min(kJointGroup, (int)gridDim.x - grp * kJointGroup);
  unsigned long long* word = reinterpret_cast<unsigned long long*>(j.ctrl + kWord);
  ++sy.epoch;
  auto arrive = [&](int* count, int target) {
    wait_own_stores();
    __syncthreads();
    if (tid == 0)
      *sy.s_flag = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == target - 1;
    __syncthreads();
    return *sy.s_flag != 0;
  };
  if (arrive(&j.ctrl[kGroup0 + kLine * grp], sy.epoch * gs)) {
    if (tests) {
      joint_reduce(j.bmax + (size_t)grp * kJointGroup * 64, gs, sy.sRed, sy.sRedAny);
      if (tid < 64) st_agent(&j.gmax[grp * 64 + tid], sy.sRed[tid] | (sy.sRedAny[tid] ? 0x80000000u : 0u));
    }
    if (arrive(&j.ctrl[kTop], sy.epoch * n_grp)) {
      if (tests) {
        joint_reduce(j.gmax, n_grp, sy.sRed, sy.sRedAny);
        joint_decide(j, cursor, n_eff, sy.sRed, sy.sRedAny, word, sy.epoch);
      } else if (tid == 0) {
        st_agent(word, (unsigned long long)sy.epoch << 32);
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    const long long t0 = wall_clock64();
    unsigned long long w = 0;
    int ok = j.barrier_ticks > 0;   // a zero bound gives up at once: the failure path, forced
    while (ok) {
      w = ld_agent(word);
      if ((w >> 32) == (unsigned long long)sy.epoch) break;
      if (ld_agent(&j.ctrl[kError]) != 0 || wall_clock64() - t0 >= j.barrier_ticks) ok = 0;
      __builtin_amdgcn_s_sleep(1);
    }
    if (!ok) st_agent(&j.ctrl[kError], 1);
    *sy.s_word = w;
    *sy.s_flag = ok;
  }
  __syncthreads();
  const bool ok = *sy.s_flag != 0;
  if (payload) *payload = (unsigned)*sy.s_word;
  __syncthreads();
  return ok;
}

// Lists the fix-up pairs of the candidates in the masks (bits as in
// RowState::fix) for this wave's rows.
__device__ void joint_append(const JointArgs& j, const RowState& st, int rb0, int nr, int cursor,
                             unsigned long long mask0, unsigned long long mask1) {
  const int lane = threadIdx.x & 63;
  for (int r = threadIdx.x >> 6; r < nr; r += kJW) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const unsigned long long m = st.fix[2 * r + b] & (b ? mask1 : mask0);
      if ((m >> lane) & 1ull) {
        const int slot = __hip_atomic_fetch_add(&j.ctrl[kFixN], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (slot < j.fix_cap) store_pair(j.fix_list + 2 * slot, make_int2(cursor + kCandBatch * b + ((lane >> 1) & 15), rb0 + r));
      }
    }
  }
}

// Fix-up of listed pairs e0 .. e0 + np - 1, one item per pair and `seg`
// tokens of its row: sums w_i and w_i v_i over the tokens that are visible
// and outside the union (the candidate's page and the pages accepted before
// it), with w_i = 2^(x_i - lse) <= 1, and writes the (D + 1) sums to fpart.
// Thread layout: D / 8 threads per token (16 bytes of its key and value
// each); the loads of UNR token rounds are in flight together, and the
// union's tokens of the segment are marked in LDS once per item.
template <int D, bool PG>
__device__ void joint_fix_partial(const JointArgs& j, int e0, int np, int seg, int parts, float* sacc,
                                  uint8_t* sMask) {
  constexpr int TPR = D / 8, RPR = kJT / TPR, UNR = 4;
  const AttnGeom& a = j.geo;
  const int tid = threadIdx.x, c = tid % TPR, r = tid / TPR;
  for (int item = blockIdx.x; item < np * parts; item += gridDim.x) {
    // consecutive items share the segment, so pairs of one head meet in the caches
    const int e = e0 + item % np, part = item / np;
    const int2 ent = load_pair(j.fix_list + 2 * e);
    const int rg = (int)CKV_IDX(ent.y, j.total_rows, j.geo.dbg, 12);
    const int t_c = (int)CKV_IDX(ent.x, j.max_cand, j.geo.dbg, 13);
    const int cp = j.cand[t_c];   // the candidate's page
    const int h = rg / a.W, p = rg % a.W, g = h / a.group;
    const int qp = a.qpos[p];
    const float ref = j.lse[rg] * kLog2e;
    const int a0 = part * seg, a1 = min(a.S, a0 + seg);
    const uint16_t* kh = a.k + (int64_t)g * a.kv_head_stride;
    const uint16_t* vh = a.v + (int64_t)g * a.kv_head_stride;
    const u32x4 qc = ldg_u4(a.q + (int64_t)h * a.q_head_stride + (int64_t)p * a.q_row_stride + 8 * c);
    u32x4 kc[UNR], vc[UNR];
    int pv[UNR];
    auto load_round = [&](int b0) {
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int tt = min(b0 + u * RPR + r, a1 - 1);
        const int64_t row = PG ? (int64_t)min((uint32_t)a.slot[tt], a.pool_last) : tt;
        kc[u] = ldg_u4(kh + row * a.kv_tok_stride + 8 * c);
        vc[u] = ldg_u4(vh + row * a.kv_tok_stride + 8 * c);
        pv[u] = ldg_i32(a.pos + tt);
      }
    };
    load_round(a0);
    for (int i = tid; i < seg; i += kJT) sMask[i] = 0;
    // pages are sorted and disjoint: the first one that reaches into the
    // segment lies in [lo, hi], and at most `seg` more follow it
    int lo = 0, hi = j.n_pages;
    while (hi - lo > 1024) {
      const int mid = (lo + hi) >> 1;
      if (j.pstart[mid] + j.plen[mid] <= a0) lo = mid + 1;
      else hi = mid;
    }
    __syncthreads();
    for (int q = lo + tid; q < min(j.n_pages, hi + seg + 1); q += kJT) {
      const int s0 = j.pstart[q], s1 = s0 + j.plen[q];
      if (s0 < a1 && s1 > a0 && (q == cp || ld_agent(&j.acc_t[q]) < t_c))
        for (int i = max(s0, a0); i < min(s1, a1); ++i) sMask[i - a0] = 1;
    }
    __syncthreads();
    float qv[8], acc[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      qv[m] = bf16_bits_to_float(chunk_elem(qc, m));
      acc[m] = 0.f;
    }
    float lacc = 0.f;
    for (int b0 = a0; b0 < a1; b0 += UNR * RPR) {
      if (b0 != a0) load_round(b0);
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int t = b0 + u * RPR + r;
        float x = 0.f;
#pragma unroll
        for (int m = 0; m < 8; ++m) x = __builtin_fmaf(qv[m], bf16_bits_to_float(chunk_elem(kc[u], m)), x);
#pragma unroll
        for (int off = TPR / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
        const bool keep = t < a1 && pv[u] <= qp && !sMask[min(t, a1 - 1) - a0];
        const float w = keep ? __builtin_amdgcn_exp2f(__builtin_fmaf(x, a.sl2, -ref)) : 0.f;
#pragma unroll
        for (int m = 0; m < 8; ++m) acc[m] = __builtin_fmaf(w, bf16_bits_to_float(chunk_elem(vc[u], m)), acc[m]);
        if (c == 0) lacc += w;
      }
    }
#pragma unroll
    for (int m = 0; m < 8; ++m) sacc[r * (D + 1) + 8 * c + m] = acc[m];
    if (c == 0) sacc[r * (D + 1) + D] = lacc;
    __syncthreads();
    // the item's sums: token rows added in order
    float* out = j.fpart + ((size_t)(e - e0) * parts + part) * (D + 1);
    for (int i = tid; i <= D; i += kJT) {
      float v = 0.f;
#pragma unroll 8
      for (int k = 0; k < RPR; ++k) v += sacc[k * (D + 1) + i];
      st_agent(out + i, v);
    }
    __syncthreads();
  }
}

// One workgroup per listed pair: each wave adds its share of the parts in
// order, the waves' sums are added in order, o' = sum w v / sum w, and
// ||o - o'|| / ||o|| is raised into the candidate's union effect.
template <int D>
__device__ void joint_fix_final(const JointArgs& j, int e0, int np, int parts, float* sacc) {
  constexpr int KD = D / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int per = (parts + kJW - 1) / kJW;
  for (int e = e0 + blockIdx.x; e < e0 + np; e += gridDim.x) {
    const int2 ent = load_pair(j.fix_list + 2 * e);
    const float* fp = j.fpart + (size_t)(e - e0) * parts * (D + 1);
    float num[KD], den = 0.f;
#pragma unroll
    for (int m = 0; m < KD; ++m) num[m] = 0.f;
    const int p1 = min(parts, (wave + 1) * per);
#pragma unroll 8
    for (int part = wave * per; part < p1; ++part) {
#pragma unroll
      for (int m = 0; m < KD; ++m) num[m] += ld_agent(fp + (size_t)part * (D + 1) + lane + 64 * m);
      den += ld_agent(fp + (size_t)part * (D + 1) + D);
    }
#pragma unroll
    for (int m = 0; m < KD; ++m) sacc[wave * (D + 1) + lane + 64 * m] = num[m];
    if (lane == 0) sacc[wave * (D + 1) + D] = den;
    __syncthreads();
    if (wave == 0) {
      float dd = 0.f, oo = 0.f, ds = 0.f;
#pragma unroll
      for (int k = 0; k < kJW; ++k) ds += sacc[k * (D + 1) + D];
#pragma unroll
      for (int m = 0; m < KD; ++m) {
        float ns = 0.f;
#pragma unroll
        for (int k = 0; k < kJW; ++k) ns += sacc[k * (D + 1) + lane + 64 * m];
        const float ov = j.o[(size_t)ent.y * D + lane + 64 * m];
        const float od = ds > 0.f ? ns / ds : 0.f;
        dd += (ov - od) * (ov - od);
        oo += ov * ov;
      }
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) {
        dd += __shfl_xor(dd, off, 64);
        oo += __shfl_xor(oo, off, 64);
      }
      if (lane == 0) {
        float ratio;
        if (!(ds > 0.f)) ratio = INFINITY;
        else if (oo > 0.f) ratio = sqrtf(dd) / sqrtf(oo);
        else ratio = dd > 0.f ? INFINITY : 0.f;
        __hip_atomic_fetch_max(reinterpret_cast<unsigned*>(&j.ur[ent.x]), __float_as_uint(ratio), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    __syncthreads();
  }
}

// Recomputes every listed pair and empties the list (in every workgroup; the
// first barrier publishes the workgroups' appends).
template <int D>
__device__ bool joint_flush(const JointArgs& j, JointSync& sy, float* sacc, uint8_t* sMask) {
  if (!joint_sync(j, sy, false, 0, 0, nullptr)) return false;
  const int n = min(ld_agent(&j.ctrl[kFixN]), j.fix_cap);
  if (n == 0) return true;   // the same in every block
  const int seg = joint_segment(n, j.geo.S), parts = joint_segments(seg, j.geo.S);
  const int npc = joint_pairs(parts);
  for (int e0 = 0; e0 < n; e0 += npc) {
    const int np = min(npc, n - e0);
    if (j.geo.slot) joint_fix_partial<D, true>(j, e0, np, seg, parts, sacc, sMask);
    else joint_fix_partial<D, false>(j, e0, np, seg, parts, sacc, sMask);
    if (!joint_sync(j, sy, false, 0, 0, nullptr)) return false;
    if (e0 + npc >= n && blockIdx.x == 0 && threadIdx.x == 0) st_agent(&j.ctrl[kFixN], 0);   // read by all above
    joint_fix_final<D>(j, e0, np, parts, sacc);
    if (!joint_sync(j, sy, false, 0, 0, nullptr)) return false;
  }
  return true;
}

// LDS: the rows' state is kept in LDS (nr <= kJointRowsLds)
template <int D, bool LDS>
__global__ __launch_bounds__(kJT) void joint_rounds(JointArgs j) {
  constexpr int KD = D / 64, NR = LDS ? kJointRowsLds : 1;
  __shared__ float sD[LDS ? NR * D : 1];
  __shared__ float sA[NR], sOn[NR];
  __shared__ int sC[NR], sNv[NR];
  __shared__ unsigned long long sFix[2 * NR];
  __shared__ unsigned sMax[64], sRed[64];
  __shared__ int sAny[64], sRedAny[64];
  __shared__ unsigned long long s_word;
  __shared__ int s_flag, s_part[kJW];
  __shared__ float sacc[(kJT / (D / 8)) * (D + 1)];   // fix-up: token rows x (D + 1) sums
  __shared__ uint8_t sMask[kFixSegMax];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const size_t gid = (size_t)blockIdx.x * kJT + tid, gsz = (size_t)gridDim.x * kJT;
  const int n_eff = min(min(*j.n_cand, j.max_cand), j.test_cap);
  // outputs; every word that another workgroup may write later goes through
  // agent-scope stores, so the first barrier needs no fence either
  for (size_t i = gid; i < (size_t)j.max_cand; i += gsz) {
    st_agent(&j.accepted[i], (uint8_t)0);
    st_agent(&j.ur[i], __builtin_nanf(""));
  }
  if (gid == 0) st_agent(j.n_accepted, 0);
  if (n_eff <= 0) return;              // nothing to test: the same in every block
  for (size_t i = gid; i < (size_t)j.n_pages; i += gsz) st_agent(&j.acc_t[i], INT_MAX);
  // n_vis of window row p (shared by every query head): #{i : pos[i] <= qpos[p]},
  // one partial count per (row, token slice)
  for (int it = blockIdx.x; it < j.W * j.n_vis_slices; it += gridDim.x) {
    const int p = it / j.n_vis_slices, sl = it % j.n_vis_slices;
    const int qp = j.qpos[p];
    const int t0 = sl * kVisSlice, t1 = min(j.S, t0 + kVisSlice);
    int c = 0;
    for (int i = t0 + tid; i < t1; i += kJT) c += j.pos[i] <= qp ? 1 : 0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
    if (lane == 0) s_part[wave] = c;
    __syncthreads();
    if (tid == 0) {
      int s = 0;
      for (int w = 0; w < kJW; ++w) s += s_part[w];
      st_agent(&j.nvis_part[it], s);
    }
    __syncthreads();
  }
  // this workgroup's rows: state and ||o_p||
  const int rpb = (j.total_rows + gridDim.x - 1) / gridDim.x;
  const int rb0 = blockIdx.x * rpb;
  const int nr = max(0, min(rpb, j.total_rows - rb0));
  RowState st;
  if constexpr (LDS) st = RowState{sD, sA, sC, sOn, sNv, sFix};
  else st = RowState{j.st_D + (size_t)rb0 * D, j.st_A + rb0, j.st_C + rb0, j.st_on + rb0, j.st_nv + rb0, j.st_fix + 2 * (size_t)rb0};
  for (int r = wave; r < nr; r += kJW) {
    const int row = rb0 + r;
    float n2 = 0.f;
#pragma unroll
    for (int k = 0; k < KD; ++k) {
      const float v = j.o[(size_t)row * D + lane + 64 * k];
      n2 = __builtin_fmaf(v, v, n2);
      st.D[r * D + lane + 64 * k] = 0.f;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) n2 += __shfl_xor(n2, off, 64);
    st.onorm[r] = sqrtf(n2);
    st.A[r] = 0.f;
    st.C[r] = 0;
    if (lane == 0 && (!(n2 <= 3.4e38f) || !(j.lse[row] < INFINITY))) latch_nonfinite(j.nonfinite);
  }
  JointSync sy{sRed, sRedAny, &s_flag, &s_word, 0};
  auto give_up = [&] {
    if (tid == 0) st_agent(j.n_accepted, -1);
  };
  if (!joint_sync(j, sy, false, 0, 0, nullptr)) return give_up();
  for (int r = wave; r < nr; r += kJW) {
    const int row = rb0 + r;
    int c = 0;
    for (int q = lane; q < j.n_vis_slices; q += 64) c += ld_agent(&j.nvis_part[(row % j.W) * j.n_vis_slices + q]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
    st.nvis[r] = c;
  }
  int cursor = 0, n_acc = 0, f0 = 0, nf = 0;
  bool listed = false;
  // every round decides at least one candidate: n_eff rounds suffice
  while (cursor < n_eff) {
    if (tid < 64) {
      sMax[tid] = 0u;
      sAny[tid] = 0;
    }
    __syncthreads();
    joint_tests<D>(j, st, rb0, nr, cursor, n_eff, f0, nf, sMax, sAny);
    __syncthreads();
    // this workgroup's maxima go to its own words (no contended atomics)
    if (tid < 64) st_agent(&j.bmax[(size_t)blockIdx.x * 64 + tid], sMax[tid] | (sAny[tid] ? 0x80000000u : 0u));
    unsigned dec;
    if (!joint_sync(j, sy, true, cursor, n_eff, &dec)) return give_up();
    const bool chain = dec & kDecChain;
    const int n = (dec >> 1) & 63, extra = (dec & kDecExtra) ? 1 : 0;
    f0 = chain ? cursor : cursor + n;    // the candidates accepted in this round
    nf = chain ? n : extra;
    if ((dec & kDecFlush) && !joint_flush<D>(j, sy, sacc, sMask)) return give_up();
    if (dec & (kDecDefer | kDecResolve)) {
      // candidates [0, nd) of the chosen guess, as bits of RowState::fix
      const int nd = (dec & kDecResolve) ? 1 : n + extra;
      auto bits = [&](int m) {
        const unsigned long long b = m <= 0 ? 0ull : 0x55555555ull >> (32 - 2 * min(m, 16));
        return chain ? b << 32 : b;
      };
      joint_append(j, st, rb0, nr, cursor, bits(nd), bits(nd - 16));
      listed = true;
    }
    if (dec & kDecResolve) {
      // the candidate at the cursor: its union effect is complete after a flush
      if (!joint_flush<D>(j, sy, sacc, sMask)) return give_up();
      listed = false;
      const bool pass = ld_agent(&j.ur[cursor]) <= j.tau;
      f0 = cursor;
      nf = pass ? 1 : 0;
      if (pass && gid == 0) {
        st_agent(&j.accepted[cursor], (uint8_t)1);
        const int ap = j.cand[cursor];
        if (ap >= 0 && ap < j.n_pages) mark_accepted(j, ap, cursor);
      }
      cursor += 1;
    } else {
      cursor += n + extra;
    }
    n_acc += nf;
  }
  if (listed && !joint_flush<D>(j, sy, sacc, sMask)) return give_up();
  if (gid == 0 && ld_agent(&j.ctrl[kError]) == 0) st_agent(j.n_accepted, n_acc);
}

int joint_vis_slices(int S) { return (S + kVisSlice - 1) / kVisSlice; }

namespace {
typedef void (*JointKernel)(JointArgs);
JointKernel joint_kernel(int D, bool lds) {
  if (D == 128) return lds ? joint_rounds<128, true> : joint_rounds<128, false>;
  return lds ? joint_rounds<64, true> : joint_rounds<64, false>;
}

// workgroups of one form that fit on the current device at once (queried once
// per device)
hipError_t joint_resident(int D, bool lds, int* out) {
  static std::atomic<int> resident[64][4];
  int dev = 0, per_cu = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::atomic<int>& res = resident[dev][(D == 128 ? 2 : 0) + (lds ? 1 : 0)];
  if ((*out = res.load(std::memory_order_relaxed)) > 0) return hipSuccess;
  if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, joint_kernel(D, lds), kJT, 0)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  *out = std::max(1, per_cu * cus);
  res.store(*out, std::memory_order_relaxed);
  return hipSuccess;
}
}  // namespace

hipError_t joint_needs_global_state(int D, int total_rows, bool* global) {
  int res = 0;
  const hipError_t e = joint_resident(D, true, &res);
  if (e == hipSuccess) *global = joint_state_global(total_rows, res);
  return e;
}

hipError_t launch_joint(const JointArgs& j, hipStream_t s) {
  const bool lds = j.st_D == nullptr;
  int res = 0;
  const hipError_t e = joint_resident(j.D, lds, &res);
  if (e != hipSuccess) return e;
  if (lds && joint_state_global(j.total_rows, res)) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(joint_kernel(j.D, lds), dim3(joint_blocks(j.total_rows, res)), dim3(kJT), 0, s, j);
  return hipGetLastError();
}

}  // namespace ckv
