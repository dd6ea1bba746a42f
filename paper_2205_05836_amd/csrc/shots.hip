// Finite-shot emulation of subcircuit runs and the chi-square loss of Eq. 3.
//
// A QPU run reports the distribution of `shots` measured bit strings
// (Section 2).  Each row of a probability table is sampled independently and
// every decision is taken in integers, so any implementation of the same
// definition reproduces the counts exactly:
//   * probabilities are quantised to q = floor(clamp(p, 0, 1) * 2^52) and the
//     row's inclusive prefix sums C are exact 64-bit integers;
//   * shot s of row r draws x = word0 + 2^32 word1 of Philox4x32-10 (Salmon,
//     Moraes, Dror and Shaw, SC 2011) with key (seed lo, seed hi) and counter
//     (s lo, s hi, r lo, r hi), takes t = floor(x * T / 2^64) with T = C_last
//     and lands on the first index i with C_i > t.
// Frequencies are count / shots in FP64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "internal.hpp"
#include "kernels.hpp"

namespace cq {

namespace {

constexpr int kBlock = 2048;  // row entries per block
constexpr int kThreads = 256;
constexpr int kPer = kBlock / kThreads;
constexpr int kPad = kPer + 1;          // LDS words per thread run (one pad word)
constexpr int kScanThreads = 1024;      // row scans of block sums and counts
constexpr int kMaxShotsPerThread = 64;  // a shot group: 256 threads of 1..64 shots each
constexpr int kLdsBins = 4096;          // rows with at most this many blocks search and count in LDS
constexpr int kFewShots = 64;           // blocks with at most this many shots resolve in registers
constexpr int kSparseShots = 16;        // shots per block on average up to which only the runs with shots are read again
// fewest blocks of a table for that: a wave a block and the run sums cost small
// tables more than the second read (416 blocks of 7 shots: 28 us with a
// workgroup a block, 31.7 with a wave; 2048 blocks 41.1 and 41.0; 4096 blocks
// 67.8 and 63.3)
constexpr int64_t kSparseBlocks = 2048;
constexpr int kRun = 64;                // entries of a run, one a lane
constexpr int kRuns = kBlock / kRun;
// rows of one block that a workgroup takes whole: with at most so many shots
// (one row: 27 us either way at 6000, 40 against 28 at 15000), or so many rows
// that the chip is full anyway (600 rows of 20000 shots: 93 us whole, 80
// spread; 1100 rows of 10000: 77 and 85), else the shots of a row are spread
// over workgroups
constexpr int64_t kRowShots = 6144;
constexpr int64_t kRowRows = 1024;
constexpr int64_t kPartShots = 4096;  // fewest shots of a workgroup where rows are spread

__device__ inline uint64_t quant52(double p) {
  const double c = p > 0.0 ? (p < 1.0 ? p : 1.0) : 0.0;
  return (uint64_t)(c * 0x1p52);
}

typedef double d2_t __attribute__((ext_vector_type(2)));

// v of the lane that DPP control CTRL names (a row holds 16 lanes)
template <int CTRL>
__device__ inline unsigned long long dpp_u64(unsigned long long v) {
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xf, 0xf, true);
  return (unsigned long long)(uint32_t)lo | ((unsigned long long)(uint32_t)hi << 32);
}

// Pass 1: the quantised sum of every run of 64 entries and of every block of
// a row (one read of the table, which bounds it), and the block's shot
// counters cleared.  A thread sums eight neighbours, so a run is eight lanes:
// three cross-lane additions (pairs, quads, halves of a row) that stay in the
// vector ALU.  With runs spread over a wave's 64 lanes (one coalesced load
// each) the ten exchanges through LDS made the pass 1.17 ms at 144 x 2^22
// (4.8 GB) against 0.79; without run sums it takes 0.75.  Rows off the
// 16-byte alignment, whose loads would be 64 bytes apart and half as wide, go
// through LDS (49 us at 3189 x 13059 without run sums, 78 that way).  RUNS
// only where a resolution form reads them.
template <bool RUNS>
__global__ void __launch_bounds__(kThreads) shots_bsum_kernel(const double* __restrict__ P, int64_t cols,
                                                              int64_t nblk, uint64_t* __restrict__ bend,
                                                              uint64_t* __restrict__ runs,
                                                              uint32_t* __restrict__ bcnt,
                                                              uint32_t* __restrict__ bfill) {
  static_assert(kPer == 8 && kRun == 64 && kThreads == 256, "eight lanes sum a run");
  const int64_t row = blockIdx.y, blk = blockIdx.x;
  const double* p = P + row * cols + blk * kBlock;
  const int n = (int)(cols - blk * kBlock < kBlock ? cols - blk * kBlock : kBlock);
  const int64_t k = row * nblk + blk;
  unsigned long long t = 0;
  if constexpr (RUNS) {
    __shared__ double stage[kThreads * kPad];
    const int e0 = threadIdx.x * kPer;
    double x[kPer];
    if (n == kBlock && (reinterpret_cast<uintptr_t>(p) & 15) == 0) {
#pragma unroll
      for (int q = 0; q < kPer / 2; ++q) {
        const d2_t y = reinterpret_cast<const d2_t*>(p + e0)[q];
        x[2 * q] = y[0];
        x[2 * q + 1] = y[1];
      }
    } else {
      // (unconditional loads, so that all eight are in flight)
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int e = threadIdx.x + q * kThreads;
        x[q] = __builtin_nontemporal_load(p + (e < n ? e : n - 1));
      }
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int e = threadIdx.x + q * kThreads;
        stage[(e / kPer) * kPad + e % kPer] = e < n ? x[q] : 0.0;
      }
      __syncthreads();
#pragma unroll
      for (int e = 0; e < kPer; ++e) x[e] = stage[threadIdx.x * kPad + e];
    }
#pragma unroll
    for (int e = 0; e < kPer; ++e) t += quant52(x[e]);
    t += dpp_u64<0xb1>(t);   // quad_perm [1, 0, 3, 2]
    t += dpp_u64<0x4e>(t);   // quad_perm [2, 3, 0, 1]
    t += dpp_u64<0x141>(t);  // row_half_mirror: the other quad of eight
    if ((threadIdx.x & 7) == 0) runs[k * kRuns + (threadIdx.x >> 3)] = t;
  } else {
    double x[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int e = threadIdx.x + q * kThreads;
      x[q] = __builtin_nontemporal_load(p + (e < n ? e : n - 1));
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) t += (int)threadIdx.x + q * kThreads < n ? quant52(x[q]) : 0ull;
    t += dpp_u64<0xb1>(t);
    t += dpp_u64<0x4e>(t);
    t += dpp_u64<0x141>(t);
  }
  t += dpp_u64<0x140>(t);  // row_mirror: the other half of a row
  t += (unsigned long long)__shfl_xor((long long)t, 16);
  t += (unsigned long long)__shfl_xor((long long)t, 32);
  __shared__ unsigned long long part[kThreads / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    bend[k] = (part[0] + part[1]) + (part[2] + part[3]);
    bcnt[k] = 0;
    bfill[k] = 0;
  }
}

// Prefix over one row of `n` values (one workgroup per row, thread t owns a
// contiguous run): inclusive in place when `out` is null, else exclusive
// into `out`.
template <typename T>
__device__ inline void row_scan(T* __restrict__ v, T* __restrict__ out, int64_t n) {
  const int64_t per = (n + kScanThreads - 1) / kScanThreads;
  const int64_t b0 = (int64_t)threadIdx.x * per;
  const int64_t b1 = b0 + per < n ? b0 + per : n;
  __shared__ unsigned long long part[kScanThreads];
  unsigned long long s = 0;
#pragma unroll 8
  for (int64_t b = b0; b < b1; ++b) s += v[b];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int h = 1; h < kScanThreads; h <<= 1) {
    const unsigned long long add = threadIdx.x >= h ? part[threadIdx.x - h] : 0ull;
    __syncthreads();
    part[threadIdx.x] += add;
    __syncthreads();
  }
  unsigned long long run = threadIdx.x ? part[threadIdx.x - 1] : 0ull;
#pragma unroll 8
  for (int64_t b = b0; b < b1; ++b) {
    const T x = v[b];
    if (out) out[b] = (T)run;
    run += x;
    if (!out) v[b] = (T)run;
  }
}

// Pass 2: block sums -> inclusive block ends (C at each block's last entry).
__global__ void __launch_bounds__(kScanThreads) shots_bend_kernel(uint64_t* __restrict__ bend, int64_t nblk) {
  row_scan<uint64_t>(bend + (int64_t)blockIdx.x * nblk, nullptr, nblk);
}

// Philox4x32-10: ten rounds of two 32 x 32 -> 64-bit products of counter
// words 0 and 2 with the round multipliers; the high halves are xor-ed into
// the other words with the key, which advances by the Weyl constants.
__device__ inline void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
    c[1] = (uint32_t)p1;
    c[3] = (uint32_t)p0;
    c[0] = n0;
    c[2] = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

// Target t of shot s of row `row` (total mass T > 0) and its block: the
// first whose inclusive end exceeds t.
__device__ inline void shot_target(const uint64_t* __restrict__ E, int64_t nblk, uint64_t T, uint64_t seed,
                                   int64_t row, int64_t s, uint64_t& t, uint32_t& blk) {
  uint32_t w[4] = {(uint32_t)s, (uint32_t)((uint64_t)s >> 32), (uint32_t)row, (uint32_t)((uint64_t)row >> 32)};
  philox4x32_10(w, (uint32_t)seed, (uint32_t)(seed >> 32));
  const uint64_t x = (uint64_t)w[0] | ((uint64_t)w[1] << 32);
  t = __umul64hi(x, T);
  uint32_t lo = 0, hi = (uint32_t)nblk - 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (E[mid] > t) hi = mid;
    else lo = mid + 1;
  }
  blk = lo;
}

// Pass 3: shots per block.  grid (shot groups, rows); a group takes
// 256 * per consecutive shots of one row and, for rows of at most
// kLdsBins blocks, searches the block ends and counts its shots in LDS
// before one global add per block hit.
__global__ void __launch_bounds__(kThreads) shots_count_kernel(const uint64_t* __restrict__ bend, int64_t nblk,
                                                               int64_t shots, uint64_t seed, int per,
                                                               uint32_t* __restrict__ bcnt) {
  __shared__ uint32_t hist[kLdsBins];
  __shared__ uint64_t Es[kLdsBins];
  const int64_t row = blockIdx.y, s0 = (int64_t)blockIdx.x * per * kThreads;
  const uint64_t* E = bend + row * nblk;
  uint32_t* cnt = bcnt + row * nblk;
  const uint64_t T = E[nblk - 1];
  if (T == 0) return;
  if (nblk > kLdsBins) {
#pragma unroll 4
    for (int j = 0; j < per; ++j) {
      const int64_t s = s0 + j * kThreads + threadIdx.x;
      if (s < shots) {
        uint64_t t;
        uint32_t blk;
        shot_target(E, nblk, T, seed, row, s, t, blk);
        atomicAdd(&cnt[blk], 1u);
      }
    }
    return;
  }
  for (int b = threadIdx.x; b < nblk; b += kThreads) {
    hist[b] = 0;
    Es[b] = E[b];
  }
  __syncthreads();
#pragma unroll 4
  for (int j = 0; j < per; ++j) {
    const int64_t s = s0 + j * kThreads + threadIdx.x;
    if (s < shots) {
      uint64_t t;
      uint32_t blk;
      shot_target(Es, nblk, T, seed, row, s, t, blk);
      atomicAdd(&hist[blk], 1u);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nblk; b += kThreads)
    if (hist[b]) atomicAdd(&cnt[b], hist[b]);
}

// Pass 4: exclusive prefix of each row's block counts (bucket offsets).
__global__ void __launch_bounds__(kScanThreads) shots_bptr_kernel(uint32_t* __restrict__ bcnt,
                                                                  uint32_t* __restrict__ bptr, int64_t nblk) {
  const int64_t off = (int64_t)blockIdx.x * nblk;
  row_scan<uint32_t>(bcnt + off, bptr + off, nblk);
}

// Pass 5: every shot's target, relative to its block's first entry, into
// the block's bucket; row r's buckets fill slots [r shots, (r + 1) shots).
// Same groups as pass 3.  For rows counted in LDS the group counts its shots
// per block again, reserves one run of each bucket it hits with one global
// add, and then recomputes every shot and takes the next position of its
// run from LDS, so a group's shots of one bucket land next to each other
// (plain stores, so that L2 merges each run before it goes to HBM).
__global__ void __launch_bounds__(kThreads) shots_scatter_kernel(const uint64_t* __restrict__ bend, int64_t nblk,
                                                                 int64_t shots, uint64_t seed, int per,
                                                                 const uint32_t* __restrict__ bptr,
                                                                 uint32_t* __restrict__ bfill,
                                                                 uint64_t* __restrict__ slots) {
  __shared__ uint32_t hist[kLdsBins];  // group counts, then the next position in each bucket
  __shared__ uint64_t Es[kLdsBins];
  const int64_t row = blockIdx.y, s0 = (int64_t)blockIdx.x * per * kThreads;
  const uint64_t* E = bend + row * nblk;
  const uint32_t* ptr = bptr + row * nblk;
  uint32_t* fill = bfill + row * nblk;
  uint64_t* S = slots + row * shots;
  const uint64_t T = E[nblk - 1];
  if (T == 0) return;
  if (nblk > kLdsBins) {
#pragma unroll 4
    for (int j = 0; j < per; ++j) {
      const int64_t s = s0 + j * kThreads + threadIdx.x;
      if (s < shots) {
        uint64_t t;
        uint32_t blk;
        shot_target(E, nblk, T, seed, row, s, t, blk);
        const uint32_t pos = ptr[blk] + atomicAdd(&fill[blk], 1u);
        S[pos] = t - (blk ? E[blk - 1] : 0);
      }
    }
    return;
  }
  for (int b = threadIdx.x; b < nblk; b += kThreads) {
    hist[b] = 0;
    Es[b] = E[b];
  }
  __syncthreads();
#pragma unroll 4
  for (int j = 0; j < per; ++j) {
    const int64_t s = s0 + j * kThreads + threadIdx.x;
    if (s < shots) {
      uint64_t t;
      uint32_t blk;
      shot_target(Es, nblk, T, seed, row, s, t, blk);
      atomicAdd(&hist[blk], 1u);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nblk; b += kThreads)
    if (hist[b]) hist[b] = ptr[b] + atomicAdd(&fill[b], hist[b]);
  __syncthreads();
#pragma unroll 4
  for (int j = 0; j < per; ++j) {
    const int64_t s = s0 + j * kThreads + threadIdx.x;
    if (s < shots) {
      uint64_t t;
      uint32_t blk;
      shot_target(Es, nblk, T, seed, row, s, t, blk);
      const uint32_t pos = atomicAdd(&hist[blk], 1u);
      S[pos] = t - (blk ? Es[blk - 1] : 0);
    }
  }
}

// count / shots, 0 written as 0
__device__ inline double freq_of(uint32_t c, double ds) { return c ? (double)c / ds : 0.0; }

__device__ inline uint64_t lane_u64(uint64_t v, int lane) {  // lane uniform
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane) |
         ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32);
}

// Pass 6, tables with few shots a block (up to kSparseShots on average): a
// wave per block, blocks with at most kFewShots shots.  It writes the block's
// zeros first, then finds each shot -- the run sums tell the run, the run's 64
// entries (one a lane) the entry -- and stores count / shots over the zero.
// So 512 bytes a shot are read again instead of the block's 16 KB, and the
// chain of dependent loads of a block hides behind its zeros and the other
// waves.  Bound by writing the frequencies: 144 x 2^22 with 8192 shots a row
// takes 1.0 ms for 4.8 GB (1.74 ms when every block was read again).
__global__ void __launch_bounds__(kThreads) shots_resolve_sparse_kernel(const double* __restrict__ P, int64_t cols,
                                                                        int64_t nblk, int64_t total, int64_t shots,
                                                                        const uint64_t* __restrict__ runs,
                                                                        const uint32_t* __restrict__ bcnt,
                                                                        const uint32_t* __restrict__ bptr,
                                                                        const uint64_t* __restrict__ slots,
                                                                        double* __restrict__ F) {
  constexpr int kAtOnce = 4;  // shots whose loads are in flight together
  const int lane = threadIdx.x & 63;
  const int64_t k = (int64_t)blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (k >= total) return;
  const int64_t row = k / nblk, c0 = (k - row * nblk) * kBlock;
  const int n = (int)(cols - c0 < kBlock ? cols - c0 : kBlock);
  const int m = (int)__builtin_amdgcn_readfirstlane((int)bcnt[k]);
  if ((uint32_t)m > (uint32_t)kFewShots) return;
  // the loads that need nothing but m, then the zeros
  const uint64_t own = m && lane < kRuns ? runs[k * kRuns + lane] : 0ull;
  const uint64_t target = lane < m ? slots[row * shots + bptr[k] + lane] : 0ull;
  double* f = F + row * cols + c0;
  if (n == kBlock && (reinterpret_cast<uintptr_t>(f) & 15) == 0) {
#pragma unroll
    for (int q = 0; q < kBlock / 128; ++q)
      __builtin_nontemporal_store(d2_t{0.0, 0.0}, reinterpret_cast<d2_t*>(f) + lane + 64 * q);
  } else {
    for (int e = lane; e < n; e += 64) __builtin_nontemporal_store(0.0, f + e);
  }
  if (m == 0) return;
  unsigned long long incl = own;
#pragma unroll
  for (int d = 1; d < kRuns; d <<= 1) {
    const unsigned long long y = __shfl_up(incl, d);
    if (lane >= d) incl += y;
  }
  const unsigned long long excl = incl - own;
  const double* p = P + row * cols + c0;
  int hit = 0;  // lane j: shot j's entry
  for (int q0 = 0; q0 < m; q0 += kAtOnce) {
    double x[kAtOnce];
    uint64_t t[kAtOnce];
    int run[kAtOnce];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      // past the last shot its target is taken again, and not kept
      t[q] = lane_u64(target, q0 + q < m ? q0 + q : m - 1);
      // the first run whose inclusive end exceeds the target (there is one
      // unless the row's sum overflowed 64 bits: then any run, in bounds)
      const int r = __ffsll((unsigned long long)__ballot(lane < kRuns && incl > t[q])) - 1;
      run[q] = r < 0 ? 0 : r;
      t[q] -= lane_u64(excl, run[q]);
      const int e = run[q] * kRun + lane;
      x[q] = e < n ? p[e] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      unsigned long long c = quant52(x[q]);
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(c, d);
        if (lane >= d) c += y;
      }
      const int e = __ffsll((unsigned long long)__ballot(c > t[q])) - 1;
      if (lane == q0 + q) hit = run[q] * kRun + (e < 0 ? 0 : e);
    }
  }
  int c = 0;
  for (int j = 0; j < m; ++j) c += __builtin_amdgcn_readlane(hit, j) == hit ? 1 : 0;
  // the zeros are written before any count goes over them
  __builtin_amdgcn_s_waitcnt((0) | (7 << 4) | (15 << 8));  // vmcnt(0)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  if (lane < m && hit < n) f[hit] = (double)c / (double)shots;
}

// Pass 6, tables with more shots a block: blocks with at most kFewShots shots
// in a workgroup each.  Thread t holds entries t kPer .. t kPer + kPer - 1 in
// registers, the block scan gives its run's offset, and every thread tests the
// block's targets against its run (the first entry whose inclusive prefix
// exceeds the target), counting in registers.  No LDS staging of the entries,
// so many more blocks stay resident than in the LDS form below.  A block
// without shots writes zeros without reading its entries.  All forms give the
// same counts.
__global__ void __launch_bounds__(kThreads) shots_resolve_few_kernel(const double* __restrict__ P, int64_t cols,
                                                                     int64_t nblk, int64_t shots,
                                                                     const uint32_t* __restrict__ bcnt,
                                                                     const uint32_t* __restrict__ bptr,
                                                                     const uint64_t* __restrict__ slots,
                                                                     double* __restrict__ F) {
  __shared__ unsigned long long wtot[kThreads / 64];
  __shared__ uint64_t tg[kFewShots];
  const int64_t row = blockIdx.y, blk = blockIdx.x;
  const int64_t c0 = blk * kBlock;
  const int n = (int)(cols - c0 < kBlock ? cols - c0 : kBlock);
  const int64_t k = row * nblk + blk;
  const uint32_t m = bcnt[k];
  if (m > (uint32_t)kFewShots) return;
  double* f = F + row * cols + c0;
  const int e0 = threadIdx.x * kPer;
  const bool vec = e0 + kPer <= n && ((reinterpret_cast<uintptr_t>(f) | reinterpret_cast<uintptr_t>(P + row * cols + c0)) & 15) == 0;
  if (m == 0) {
    if (vec) {
#pragma unroll
      for (int q = 0; q < kPer / 2; ++q) reinterpret_cast<d2_t*>(f + e0)[q] = d2_t{0.0, 0.0};
    } else {
      for (int e = e0; e < e0 + kPer && e < n; ++e) __builtin_nontemporal_store(0.0, f + e);
    }
    return;
  }
  const double* p = P + row * cols + c0 + e0;
  unsigned long long v[kPer];
  if (vec) {
#pragma unroll
    for (int q = 0; q < kPer / 2; ++q) {
      const d2_t x = reinterpret_cast<const d2_t*>(p)[q];
      v[2 * q] = quant52(x[0]);
      v[2 * q + 1] = quant52(x[1]);
    }
  } else {
#pragma unroll
    for (int e = 0; e < kPer; ++e) v[e] = e0 + e < n ? quant52(p[e]) : 0ull;
  }
  unsigned long long s = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    s += v[e];
    v[e] = s;
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  unsigned long long x = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned long long y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  if (lane == 63) wtot[wid] = x;
  if (threadIdx.x < m) tg[threadIdx.x] = slots[row * shots + bptr[k] + threadIdx.x];
  __syncthreads();
  unsigned long long before = x - s;
  for (int w = 0; w < wid; ++w) before += wtot[w];
  uint32_t c[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) c[e] = 0;
  for (uint32_t j = 0; j < m; ++j) {
    const uint64_t t = tg[j];
    // this run holds the target when before <= t < before + s
    if (t >= before && t - before < s) {
      const uint64_t r = t - before;
      bool found = false;
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        const bool here = !found && v[e] > r;
        c[e] += here ? 1u : 0u;
        found = found || here;
      }
    }
  }
  const double ds = (double)shots;
  if (vec) {
#pragma unroll
    for (int q = 0; q < kPer / 2; ++q) {
      const d2_t y = {freq_of(c[2 * q], ds), freq_of(c[2 * q + 1], ds)};
      reinterpret_cast<d2_t*>(f + e0)[q] = y;
    }
  } else {
#pragma unroll
    for (int e = 0; e < kPer; ++e)
      if (e0 + e < n) __builtin_nontemporal_store(freq_of(c[e], ds), f + e0 + e);
  }
}

// Pass 6, blocks with many shots: the inclusive prefix of the block's
// quantised entries in LDS, its bucket's shots resolved there by binary
// search (the first entry whose prefix exceeds the shot's target), and
// count / shots written out; a block without shots writes zeros without
// reading its entries.  LDS layout: thread t's run of kPer entries at
// [t kPad, t kPad + kPer).
struct ResolveLds {
  unsigned long long C[kThreads * kPad];
  uint32_t cnt[kBlock];
  unsigned long long wtot[kThreads / 64];
};

// The inclusive prefix of n quantised entries into L.C, counts cleared.
__device__ __forceinline__ void block_prefix_lds(ResolveLds& L, const double* __restrict__ p, int n) {
  double x[kPer];  // unconditional loads, so that all eight are in flight
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int e = threadIdx.x + q * kThreads;
    x[q] = __builtin_nontemporal_load(p + (e < n ? e : n - 1));
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int e = threadIdx.x + q * kThreads;
    L.C[(e / kPer) * kPad + e % kPer] = e < n ? quant52(x[q]) : 0ull;
    L.cnt[e] = 0;
  }
  __syncthreads();
  unsigned long long* mine = L.C + threadIdx.x * kPad;
  unsigned long long v[kPer];
  unsigned long long s = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    s += mine[e];
    v[e] = s;
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  unsigned long long end = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned long long y = __shfl_up(end, d);
    if (lane >= d) end += y;
  }
  if (lane == 63) L.wtot[wid] = end;
  __syncthreads();
  unsigned long long before = end - s;
  for (int w = 0; w < wid; ++w) before += L.wtot[w];
#pragma unroll
  for (int e = 0; e < kPer; ++e) mine[e] = v[e] + before;
  __syncthreads();
}

// Counts target t in the entry it lands on.
__device__ __forceinline__ void count_target_lds(ResolveLds& L, uint64_t t, int n) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (L.C[(mid / kPer) * kPad + mid % kPer] > t) hi = mid;
    else lo = mid + 1;
  }
  atomicAdd(&L.cnt[lo], 1u);
}

__device__ __forceinline__ void write_counts_lds(const ResolveLds& L, double* __restrict__ f, int n, int64_t shots) {
  const double ds = (double)shots;
  for (int e = threadIdx.x; e < n; e += kThreads) __builtin_nontemporal_store(freq_of(L.cnt[e], ds), f + e);
}

__device__ __forceinline__ void resolve_block_lds(ResolveLds& L, const double* __restrict__ P, int64_t cols,
                                                  int64_t nblk, int64_t shots, int64_t k, uint32_t m,
                                                  const uint32_t* __restrict__ bptr,
                                                  const uint64_t* __restrict__ slots, double* __restrict__ F) {
  const int64_t row = k / nblk, blk = k - row * nblk;
  const int64_t c0 = blk * kBlock;
  const int n = (int)(cols - c0 < kBlock ? cols - c0 : kBlock);
  double* f = F + row * cols + c0;
  if (m == 0) {
    for (int e = threadIdx.x; e < n; e += kThreads) __builtin_nontemporal_store(0.0, f + e);
    return;
  }
  block_prefix_lds(L, P + row * cols + c0, n);
  const uint64_t* sl = slots + row * shots + bptr[k];
  for (uint32_t j = threadIdx.x; j < m; j += kThreads) count_target_lds(L, __builtin_nontemporal_load(sl + j), n);
  __syncthreads();
  write_counts_lds(L, f, n, shots);
  __syncthreads();  // the workgroup's next block reuses the LDS
}

// Rows of one block: the whole row in one workgroup, from entries to
// frequencies, without sums, buckets or slots in memory (one launch instead
// of six: a table of 300 x 77 with 5000 shots a row, and its chi-square, take
// 25 us instead of 46).
__global__ void __launch_bounds__(kThreads) shots_row_kernel(const double* __restrict__ P, int64_t cols,
                                                             int64_t shots, uint64_t seed,
                                                             double* __restrict__ F) {
  __shared__ ResolveLds L;
  const int64_t row = blockIdx.x;
  const int n = (int)cols;
  block_prefix_lds(L, P + row * cols, n);
  const uint64_t T = L.C[((n - 1) / kPer) * kPad + (n - 1) % kPer];
  if (T != 0)
    for (int64_t s = threadIdx.x; s < shots; s += kThreads) {
      uint64_t t;
      uint32_t blk;
      shot_target(&T, 1, T, seed, row, s, t, blk);
      count_target_lds(L, t, n);
    }
  __syncthreads();
  write_counts_lds(L, F + row * cols, n, shots);
}

// Rows of one block with too few rows for a workgroup each to fill the chip:
// a workgroup takes `per` shots of row blockIdx.y, forms the row's prefix
// again (at most 16 KB, against thousands of shots searched in it), counts in
// LDS and adds to the row's counters in memory, cleared before and turned
// into frequencies after.  By buckets one workgroup resolved the whole row: 4
// rows of 1233 with 510851 shots a row took 1960 us, now 33.
__global__ void __launch_bounds__(kThreads) shots_row_clear_kernel(uint32_t* __restrict__ cnt, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) cnt[i] = 0;
}

__global__ void __launch_bounds__(kThreads) shots_row_part_kernel(const double* __restrict__ P, int64_t cols,
                                                                  int64_t shots, int64_t per, uint64_t seed,
                                                                  uint32_t* __restrict__ cnt) {
  __shared__ ResolveLds L;
  const int64_t row = blockIdx.y, s0 = (int64_t)blockIdx.x * per, s1 = s0 + per < shots ? s0 + per : shots;
  const int n = (int)cols;
  block_prefix_lds(L, P + row * cols, n);
  const uint64_t T = L.C[((n - 1) / kPer) * kPad + (n - 1) % kPer];
  if (T != 0)
    for (int64_t s = s0 + threadIdx.x; s < s1; s += kThreads) {
      uint64_t t;
      uint32_t blk;
      shot_target(&T, 1, T, seed, row, s, t, blk);
      count_target_lds(L, t, n);
    }
  __syncthreads();
  for (int e = threadIdx.x; e < n; e += kThreads)
    if (const uint32_t c = L.cnt[e]) atomicAdd(cnt + row * cols + e, c);
}

__global__ void __launch_bounds__(kThreads) shots_row_freq_kernel(const uint32_t* __restrict__ cnt, int64_t n,
                                                                  int64_t shots, double* __restrict__ F) {
  const double ds = (double)shots;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads)
    F[i] = freq_of(cnt[i], ds);
}

// Every block, one workgroup each (grid (nblk, rows)): for tables with many
// shots per block on average.
__global__ void __launch_bounds__(kThreads) shots_resolve_kernel(const double* __restrict__ P, int64_t cols,
                                                                 int64_t nblk, int64_t shots,
                                                                 const uint32_t* __restrict__ bcnt,
                                                                 const uint32_t* __restrict__ bptr,
                                                                 const uint64_t* __restrict__ slots,
                                                                 double* __restrict__ F) {
  __shared__ ResolveLds L;
  const int64_t k = (int64_t)blockIdx.y * nblk + blockIdx.x;
  resolve_block_lds(L, P, cols, nblk, shots, k, bcnt[k], bptr, slots, F);
}

// Only the blocks with more than kFewShots shots, after
// shots_resolve_few_kernel: each workgroup reads the shot counts of
// kManyChunk blocks (k = row * nblk + blk) at once, lists the heavy ones in
// LDS and resolves them, so a table with few such blocks costs one pass
// over the counts.
constexpr int kManyChunk = 64;
constexpr int64_t kManyGrid = 1 << 20;

__global__ void __launch_bounds__(kThreads) shots_resolve_listed_kernel(const double* __restrict__ P, int64_t cols,
                                                                        int64_t nblk, int64_t total, int64_t shots,
                                                                        const uint32_t* __restrict__ bcnt,
                                                                        const uint32_t* __restrict__ bptr,
                                                                        const uint64_t* __restrict__ slots,
                                                                        double* __restrict__ F) {
  __shared__ ResolveLds L;
  __shared__ uint32_t many[kManyChunk];
  __shared__ uint32_t nmany;
  for (int64_t base = (int64_t)blockIdx.x * kManyChunk; base < total; base += (int64_t)gridDim.x * kManyChunk) {
    if (threadIdx.x == 0) nmany = 0;
    __syncthreads();
    if (threadIdx.x < kManyChunk && base + threadIdx.x < total && bcnt[base + threadIdx.x] > (uint32_t)kFewShots)
      many[atomicAdd(&nmany, 1u)] = threadIdx.x;
    __syncthreads();
    const uint32_t listed = nmany;
    for (uint32_t q = 0; q < listed; ++q) {
      const int64_t k = base + many[q];
      resolve_block_lds(L, P, cols, nblk, shots, k, bcnt[k], bptr, slots, F);
    }
    __syncthreads();  // every thread has read nmany and the list before they change
  }
}

// Eq. 3, terms with a + b = 0 taken as 0: per-block partial sums in a fixed
// order (four strided streams a thread, then a tree), then one block sums
// the partials the same way.  Bound by reading a and b once: 9.7 GB in
// 1.55-1.65 ms (1.8 with 8-byte loads).  A thread takes
// pairs of neighbours, 16 bytes a load where both arrays are aligned (VEC);
// the order of the additions does not depend on the alignment.
constexpr int kChiBlocks = 2048;

template <bool VEC>
__global__ void __launch_bounds__(kThreads) chi2_partial_kernel(const double* __restrict__ a,
                                                                const double* __restrict__ b, int64_t n,
                                                                double* __restrict__ part) {
  __shared__ double sh[kThreads];
  // two strided streams of pairs per thread, each element summed on its own,
  // then combined
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const int64_t step = (int64_t)gridDim.x * blockDim.x, pairs = n >> 1;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  auto pair = [](const double* p, int64_t q) -> d2_t {
    if constexpr (VEC) return __builtin_nontemporal_load(reinterpret_cast<const d2_t*>(p) + q);
    else return d2_t{__builtin_nontemporal_load(p + 2 * q), __builtin_nontemporal_load(p + 2 * q + 1)};
  };
  auto add = [](double& s, double x, double y) {
    const double d = x - y, t = x + y;
    if (t != 0.0) s += d * d / t;
  };
  for (; i + step < pairs; i += 2 * step) {
    const d2_t x0 = pair(a, i), y0 = pair(b, i), x1 = pair(a, i + step), y1 = pair(b, i + step);
    add(acc[0], x0[0], y0[0]);
    add(acc[1], x0[1], y0[1]);
    add(acc[2], x1[0], y1[0]);
    add(acc[3], x1[1], y1[1]);
  }
  if (i < pairs) {
    const d2_t x = pair(a, i), y = pair(b, i);
    add(acc[0], x[0], y[0]);
    add(acc[1], x[1], y[1]);
  }
  if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) add(acc[2], a[n - 1], b[n - 1]);
  const double s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int h = kThreads / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void __launch_bounds__(kThreads) chi2_final_kernel(const double* __restrict__ part, int nparts,
                                                              double* __restrict__ out) {
  __shared__ double sh[kThreads];
  double s = 0.0;
  for (int i = threadIdx.x; i < nparts; i += kThreads) s += part[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int h = kThreads / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sh[0];
}

// bytes: what every call needs; `runs` (the run sums) and `with_runs` bytes in
// all where blocks may resolve a wave each, which smaller workspaces leave out
struct ShotsWs {
  int64_t bend = 0, bcnt = 0, bptr = 0, bfill = 0, slots = 0, bytes = 0, runs = 0, with_runs = 0;
};

// What cq_sample_shots_workspace_size asks for together with the two tables at
// most: beyond it (of the card's 288 GB) the run sums are left out.
constexpr int64_t kShotsBytes = (int64_t)240 << 30;

cq_status hip_error(hipError_t e, const char* what) {
  return fail(CQ_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

int64_t al256(int64_t x) { return (x + 255) / 256 * 256; }

ShotsWs shots_ws(int64_t rows, int64_t cols, int64_t shots) {
  ShotsWs w;
  const int64_t nblk = (cols + kBlock - 1) / kBlock, nb = rows * nblk;
  w.bend = 0;
  w.bcnt = al256(nb * 8);
  w.bptr = w.bcnt + al256(nb * 4);
  w.bfill = w.bptr + al256(nb * 4);
  w.slots = w.bfill + al256(nb * 4);
  w.bytes = w.slots + al256(rows * shots * 8);
  if (nblk > 1 && shots <= (int64_t)kSparseShots * nblk && nb >= kSparseBlocks) {
    w.runs = w.bytes;
    w.with_runs = w.runs + al256(nb * kRuns * 8);
  }
  return w;
}

cq_status shots_check(int64_t rows, int64_t cols, int64_t shots) {
  if (rows < 1 || cols < 1 || shots < 1) return fail(CQ_ERR_ARG, "rows, cols and shots must be positive");
  if (rows > 65535) return fail(CQ_ERR_SHAPE, "more than 65535 rows");
  if (cols > ((int64_t)1 << 34) / rows) return fail(CQ_ERR_SHAPE, "table larger than 2^34 entries");
  if (shots > 0xffffffffLL) return fail(CQ_ERR_SHAPE, "2^32 or more shots per row");
  if (shots > ((int64_t)1 << 34) / rows) return fail(CQ_ERR_SHAPE, "more than 2^34 shots in total");
  return CQ_OK;
}

}  // namespace

}  // namespace cq

using namespace cq;

extern "C" cq_status cq_sample_shots_workspace_size(int64_t rows, int64_t cols, int64_t shots, size_t* bytes) {
  if (!bytes) return fail(CQ_ERR_ARG, "null argument");
  cq_status st = shots_check(rows, cols, shots);
  if (st != CQ_OK) return st;
  const ShotsWs w = shots_ws(rows, cols, shots);
  *bytes = (size_t)(w.with_runs && 16 * rows * cols + w.with_runs <= kShotsBytes ? w.with_runs : w.bytes);
  return CQ_OK;
}

extern "C" cq_status cq_sample_shots(const double* probs, int64_t rows, int64_t cols, int64_t shots, uint64_t seed,
                                     double* freqs, void* workspace, size_t workspace_bytes,
                                     hipStream_t stream) {
  if (!probs || !freqs) return fail(CQ_ERR_ARG, "null argument");
  cq_status st = shots_check(rows, cols, shots);
  if (st != CQ_OK) return st;
  const ShotsWs w = shots_ws(rows, cols, shots);
  if (!workspace || (int64_t)workspace_bytes < w.bytes) return fail(CQ_ERR_WORKSPACE, "workspace too small");
  char* ws = static_cast<char*>(workspace);
  uint64_t* bend = reinterpret_cast<uint64_t*>(ws + w.bend);
  uint64_t* runs = reinterpret_cast<uint64_t*>(ws + w.runs);
  uint32_t* bcnt = reinterpret_cast<uint32_t*>(ws + w.bcnt);
  uint32_t* bptr = reinterpret_cast<uint32_t*>(ws + w.bptr);
  uint32_t* bfill = reinterpret_cast<uint32_t*>(ws + w.bfill);
  uint64_t* slots = reinterpret_cast<uint64_t*>(ws + w.slots);
  const int64_t nblk = (cols + kBlock - 1) / kBlock;  // <= 2^23 by the limits
  if (nblk == 1 && (shots <= kRowShots || rows >= kRowRows)) {
    hipLaunchKernelGGL(shots_row_kernel, dim3((unsigned)rows), dim3(kThreads), 0, stream, probs, cols, shots, seed,
                       freqs);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "shot sampling launch");
    return CQ_OK;
  }
  if (nblk == 1) {
    // no more than 2048 workgroups unless there are more rows; the counters
    // take the place of the slots (8 bytes a shot, shots > kRowShots >= the
    // columns)
    static_assert(kRowShots * 8 >= kBlock * 4, "counters fit the slots");
    int64_t per = kPartShots;
    while (per < shots && rows * ((shots + per - 1) / per) > 2048) per *= 2;
    uint32_t* cnt = reinterpret_cast<uint32_t*>(slots);
    const int64_t n = rows * cols;
    const dim3 gn((unsigned)((n + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(shots_row_clear_kernel, gn, dim3(kThreads), 0, stream, cnt, n);
    hipLaunchKernelGGL(shots_row_part_kernel, dim3((unsigned)((shots + per - 1) / per), (unsigned)rows), dim3(kThreads),
                       0, stream, probs, cols, shots, per, seed, cnt);
    hipLaunchKernelGGL(shots_row_freq_kernel, gn, dim3(kThreads), 0, stream, cnt, n, shots, freqs);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "shot sampling launch");
    return CQ_OK;
  }
  const dim3 gt((unsigned)nblk, (unsigned)rows);
  // shots of a thread: few enough for two shot groups a compute unit where
  // the table has them (20 x 10^6 outcomes with 10^5 shots a row: 226 us
  // against 258 with one)
  int per = kMaxShotsPerThread;
  while (per > 4 && rows * ((shots + (int64_t)per * kThreads - 1) / ((int64_t)per * kThreads)) < 512) per >>= 1;
  const dim3 gs((unsigned)((shots + (int64_t)per * kThreads - 1) / ((int64_t)per * kThreads)), (unsigned)rows);
  const bool sparse = w.with_runs && (int64_t)workspace_bytes >= w.with_runs;
  if (sparse)
    hipLaunchKernelGGL(shots_bsum_kernel<true>, gt, dim3(kThreads), 0, stream, probs, cols, nblk, bend, runs, bcnt,
                       bfill);
  else
    hipLaunchKernelGGL(shots_bsum_kernel<false>, gt, dim3(kThreads), 0, stream, probs, cols, nblk, bend, runs, bcnt,
                       bfill);
  hipLaunchKernelGGL(shots_bend_kernel, dim3((unsigned)rows), dim3(kScanThreads), 0, stream, bend, nblk);
  hipLaunchKernelGGL(shots_count_kernel, gs, dim3(kThreads), 0, stream, (const uint64_t*)bend, nblk, shots, seed,
                     per, bcnt);
  hipLaunchKernelGGL(shots_bptr_kernel, dim3((unsigned)rows), dim3(kScanThreads), 0, stream, bcnt, bptr, nblk);
  hipLaunchKernelGGL(shots_scatter_kernel, gs, dim3(kThreads), 0, stream, (const uint64_t*)bend, nblk, shots,
                     seed, per, (const uint32_t*)bptr, bfill, slots);
  if (shots >= (int64_t)kFewShots * nblk) {
    // many shots per block on average: every block resolves in LDS
    hipLaunchKernelGGL(shots_resolve_kernel, gt, dim3(kThreads), 0, stream, probs, cols, nblk, shots,
                       (const uint32_t*)bcnt, (const uint32_t*)bptr, (const uint64_t*)slots, freqs);
  } else {
    const int64_t total = rows * nblk;  // <= 2^23 blocks and a row more
    if (sparse)
      hipLaunchKernelGGL(shots_resolve_sparse_kernel, dim3((unsigned)((total + kThreads / 64 - 1) / (kThreads / 64))),
                         dim3(kThreads), 0, stream, probs, cols, nblk, total, shots, (const uint64_t*)runs,
                         (const uint32_t*)bcnt, (const uint32_t*)bptr, (const uint64_t*)slots, freqs);
    else
      hipLaunchKernelGGL(shots_resolve_few_kernel, gt, dim3(kThreads), 0, stream, probs, cols, nblk, shots,
                         (const uint32_t*)bcnt, (const uint32_t*)bptr, (const uint64_t*)slots, freqs);
    if (shots > kFewShots) {
      const int64_t chunks = (total + kManyChunk - 1) / kManyChunk;
      const unsigned grid = (unsigned)(chunks < kManyGrid ? chunks : kManyGrid);
      hipLaunchKernelGGL(shots_resolve_listed_kernel, dim3(grid), dim3(kThreads), 0, stream, probs, cols, nblk,
                         total, shots, (const uint32_t*)bcnt, (const uint32_t*)bptr, (const uint64_t*)slots, freqs);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_error(e, "shot sampling launch");
  return CQ_OK;
}

extern "C" cq_status cq_chi2_workspace_size(size_t* bytes) {
  if (!bytes) return fail(CQ_ERR_ARG, "null argument");
  *bytes = (size_t)kChiBlocks * sizeof(double);
  return CQ_OK;
}

extern "C" cq_status cq_chi2(const double* a, const double* b, int64_t n, double* result, void* workspace,
                             size_t workspace_bytes, hipStream_t stream) {
  if (!a || !b || !result) return fail(CQ_ERR_ARG, "null argument");
  if (n < 1) return fail(CQ_ERR_ARG, "n must be positive");
  if (!workspace || workspace_bytes < (size_t)kChiBlocks * sizeof(double))
    return fail(CQ_ERR_WORKSPACE, "workspace too small");
  double* part = static_cast<double*>(workspace);
  if (((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15) == 0)
    hipLaunchKernelGGL(chi2_partial_kernel<true>, dim3(kChiBlocks), dim3(kThreads), 0, stream, a, b, n, part);
  else
    hipLaunchKernelGGL(chi2_partial_kernel<false>, dim3(kChiBlocks), dim3(kThreads), 0, stream, a, b, n, part);
  hipLaunchKernelGGL(chi2_final_kernel, dim3(1), dim3(kThreads), 0, stream, (const double*)part, kChiBlocks, result);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_error(e, "chi-square launch");
  return CQ_OK;
}
