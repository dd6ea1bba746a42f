// Workgroup selection of the C best keys (Algorithm 1 keeps the largest bins
// of each recursion): a key is a value and a unique index, and a key is
// better than another when its value is larger, or equal with a smaller
// index.  Every lane holds up to V keys (bit e of a 64-bit `live` mask marks
// key e as taking part).
//
// Bound, filter, rank: the C-th best of the best keys of small groups of lanes
// is a key that at least C keys reach, so it bounds the C-th best key overall
// from below.  Keys that reach it are appended to LDS, and each appended key's
// rank among them is its place in the answer.  A handful of keys usually
// pass; when more than CAP do (the best keys crowd into a few lanes), the
// caller runs its exhaustive selection over the narrowed `live` instead.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cq {

// Order-preserving 64-bit key of a double (larger value, larger key), the
// form in which a running threshold is raised with atomicMax.
__device__ inline unsigned long long ord_key(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return (b >> 63) ? ~b : (b | (1ull << 63));
}

__device__ inline double ord_val(unsigned long long k) {
  const unsigned long long b = (k >> 63) ? (k & ~(1ull << 63)) : ~k;
  return __longlong_as_double((long long)b);
}

template <typename T, typename I>
struct SelKey {
  T v;
  I i;
};

template <typename T, typename I>
__device__ inline bool sel_better(const SelKey<T, I>& a, const SelKey<T, I>& b) {
  return a.v > b.v || (a.v == b.v && a.i < b.i);
}

// Number of keys among S[0..n) (LDS) better than k, shared by L neighbouring
// lanes that hold the same k (every lane gets the count): each compares with
// every L-th key, then the partial counts are summed.
template <int L, typename K>
__device__ __forceinline__ int rank_shared(const K* S, int n, const K& k) {
  int r = 0;
#pragma unroll 4
  for (int t = (int)(threadIdx.x & (L - 1)); t < n; t += L) {
    const K a = S[t];
    r += (int)((a.v > k.v) | ((a.v == k.v) & (a.i < k.i)));
  }
#pragma unroll
  for (int o = 1; o < L; o <<= 1) r += __shfl_xor(r, o, 64);
  return r;
}

// The first C of S[0..n) (LDS, distinct keys) to out, best first; every thread
// of the workgroup calls it.  Sixteen lanes rank a key, so that the usual few
// dozen keys occupy every wave (one lane a key: 2.9 us of a tile, 1.6 so).
template <int NTHR, typename K>
__device__ __forceinline__ void rank_all(const K* S, int n, int C, K* out) {
  for (int t = (int)threadIdx.x / 16; t < n; t += NTHR / 16) {
    const K k = S[t];
    const int r = rank_shared<16>(S, n, k);
    if ((threadIdx.x & 15) == 0 && r < C) out[r] = k;
  }
}

// Number of keys among S[0..n) (LDS) better than k.  Eight keys are loaded
// before any is compared, and the comparison is branch-free, so the LDS reads
// overlap instead of each waiting for the one before.
template <typename K>
__device__ __forceinline__ int rank_of(const K* S, int n, const K& k) {
  int r = 0, t = 0;
  for (; t + 8 <= n; t += 8) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const K a = S[t + u];
      r += (int)((a.v > k.v) | ((a.v == k.v) & (a.i < k.i)));
    }
  }
  for (; t < n; ++t) {
    const K a = S[t];
    r += (int)((a.v > k.v) | ((a.v == k.v) & (a.i < k.i)));
  }
  return r;
}

// The place in `best` (NTHR keys of LDS, NTHR threads) of a bound for the C-th
// best key, or -1 when fewer than C lanes have one.  mine: the lane's best key
// (has: it has one, else the worst key); owner: LDS, -1 on entry; other(k, x):
// key k of lane ^ x.  Ranks are counted among the best keys of kBoundGroups
// groups of lanes, and among all lanes' only when fewer than C groups have a
// key: every key is compared with all others through LDS, and ranking 512
// lanes took 20 us of a selecting tile's 32.  The lanes of a group share its
// ranking: by one lane each it took 5.3 us of a tile's 16.3 (FP64, 512
// threads), shared 2.4 of 12.3.  The coarser bound lets few more keys pass:
// with C of G groups holding a key at or above it, -G ln(1 - C / G) of evenly
// spread keys are, 18 for C = 16 and 89 for C = 64 of 128 groups.
constexpr int kBoundGroups = 128;

template <typename T, int NTHR, typename K, typename Other>
__device__ __forceinline__ int bound_owner(K* best, int& owner, const K& mine, bool has, int C, Other other) {
  constexpr int G = NTHR / kBoundGroups;
  static_assert(G >= 1 && (G & (G - 1)) == 0 && G <= 64, "lanes per group");
  const int tid = threadIdx.x;
  K k = mine;
#pragma unroll
  for (int x = 1; x < G; x <<= 1) {
    const K o = other(k, x);
    const bool b = (o.v > k.v) | ((o.v == k.v) & (o.i < k.i));
    k.v = b ? o.v : k.v;
    k.i = b ? o.i : k.i;
  }
  // every lane of a group holds its best key (the worst key has the index that
  // no key has)
  const bool ghas = (k.i + 1) != 0, lead = (tid & (G - 1)) == 0;
  if (lead) best[tid / G] = k;
  if (__syncthreads_count(ghas & lead) >= C) {
    // distinct keys, distinct ranks
    const int r = rank_shared<G>(best, kBoundGroups, k);
    if (ghas & lead & (r == C - 1)) owner = tid / G;
  } else {
    best[tid] = mine;
    __syncthreads();
    if (has && rank_of(best, NTHR, mine) == C - 1) owner = tid;
  }
  __syncthreads();
  return owner;
}

template <typename T, typename I, int NTHR, int CAP>
struct SelShared {
  SelKey<T, I> lane_best[NTHR];
  SelKey<T, I> cand[CAP];
  int count;
  int owner;
};

// Every thread of the workgroup (NTHR threads) calls it with the same C,
// 1 <= C <= NTHR.  at(e) returns key e of the calling lane (called only for
// live e).  none: a key no live key is worse than (it never counts as better
// than one).  Returns found = min(C, live keys) with out[0..found) best
// first, or -1 when more than CAP keys pass the bound; `live` is narrowed to
// the keys that pass, which always include the C best.
template <typename T, typename I, int V, int NTHR, int CAP, typename At>
__device__ __forceinline__ int sel_bound_top(SelShared<T, I, NTHR, CAP>& sh, uint64_t& live, At at,
                                             int C, SelKey<T, I> none, SelKey<T, I>* out) {
  using K = SelKey<T, I>;
  static_assert(V >= 1 && V <= 64, "one live bit per key");
  const int tid = threadIdx.x;
  K best = none;
  bool has = false;
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const K k = at(e);
    const bool b = (bool)((live >> e) & 1) & (!has | (k.v > best.v) | ((k.v == best.v) & (k.i < best.i)));
    best.v = b ? k.v : best.v;  // field by field: a select of the whole struct goes through memory
    best.i = b ? k.i : best.i;
    has |= b;
  }
  if (tid == 0) {
    sh.count = 0;
    sh.owner = -1;
  }
  const int lanes = __syncthreads_count(has);
  int own = -1;
  if (lanes >= C)
    own = bound_owner<T, NTHR>(sh.lane_best, sh.owner, best, has, C, [](const K& k, int x) {
      return K{__shfl_xor(k.v, x), (I)__shfl_xor((long long)k.i, x)};
    });
  if (own >= 0) {
    const K t0 = sh.lane_best[own];
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const K k = at(e);
      const bool drop = (t0.v > k.v) | ((t0.v == k.v) & (t0.i < k.i));
      live &= ~((uint64_t)drop << e);
    }
  }
  const int mine = __popcll(live);
  int off = mine ? atomicAdd(&sh.count, mine) : 0;
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const bool l = (live >> e) & 1;
    if (l & (off < CAP)) sh.cand[off] = at(e);
    off += l ? 1 : 0;
  }
  __syncthreads();
  const int n = sh.count;
  if (n > CAP) return -1;
  rank_all<NTHR>(sh.cand, n, C, out);
  __syncthreads();
  return n < C ? n : C;
}

}  // namespace cq
