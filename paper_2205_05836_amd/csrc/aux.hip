// Layout permutes and entry attribution.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "kernels.hpp"

namespace cq {

namespace {

// Element kinds of a permute's source and destination.
enum Kind { kF64 = 0, kF32 = 1, kBF16 = 2, kF16 = 3 };


__device__ inline float h16_to_f(uint16_t x, bool f16) {
  return f16 ? float(__builtin_bit_cast(_Float16, x)) : float(__builtin_bit_cast(__bf16, x));
}
__device__ inline uint16_t f_to_h16(float x, bool f16) {
  return f16 ? __builtin_bit_cast(uint16_t, _Float16(x)) : __builtin_bit_cast(uint16_t, __bf16(x));
}

// Binary exponent e of a column maximum m = f * 2^e, f in [0.5, 1) (0 for 0).
__device__ inline int colmax_exp(uint64_t bits) {
  const int be = (int)((bits >> 52) & 0x7ff);
  return be == 0 ? 0 : be - 1022;
}

__device__ inline int fac_exp(const PermArgs& p, int64_t off) {
  int e = 0;
  for (int c = 0; c < p.nfac; ++c)
    e += colmax_exp(p.colmax[c][(off >> p.fac_shift[c]) & ((1ll << p.fac_bits[c]) - 1)]);
  return e;
}

// Element `off` of the source as the destination's element: 16-bit planes are
// copied bit for bit when both sides use them, else alpha and the column-scale
// undo apply in FP64.  F64 and F32 destinations; 16-bit planes as hi | lo << 16.
template <int DK> struct PermElem { typedef uint32_t type; };
template <> struct PermElem<kF64> { typedef double type; };
template <> struct PermElem<kF32> { typedef float type; };

template <int SK, int DK>
__device__ inline typename PermElem<DK>::type perm_load(const PermArgs& p, int64_t off) {
  if constexpr (SK >= kBF16 && DK == SK) {
    const uint32_t h = static_cast<const uint16_t*>(p.src)[off];
    return p.dst_lo ? h | (uint32_t) static_cast<const uint16_t*>(p.src_lo)[off] << 16 : h;
  } else {
    double v;
    if constexpr (SK == kF64) v = static_cast<const double*>(p.src)[off];
    else if constexpr (SK == kF32) v = static_cast<const float*>(p.src)[off];
    else {
      v = h16_to_f(static_cast<const uint16_t*>(p.src)[off], SK == kF16);
      if (p.src_lo) v += h16_to_f(static_cast<const uint16_t*>(p.src_lo)[off], SK == kF16);
    }
    v *= p.alpha;
    if (p.nfac) v = ldexp(v, fac_exp(p, off));
    if constexpr (DK == kF64) return v;
    else if constexpr (DK == kF32) return float(v);
    else {
      const float x = float(v);
      const uint16_t h = f_to_h16(x, DK == kF16);
      return h | (uint32_t)f_to_h16(x - h16_to_f(h, DK == kF16), DK == kF16) << 16;
    }
  }
}

template <int DK>
__device__ inline void perm_store(const PermArgs& p, int64_t i, typename PermElem<DK>::type x) {
  if constexpr (DK == kF64) static_cast<double*>(p.dst)[i] = x;
  else if constexpr (DK == kF32) static_cast<float*>(p.dst)[i] = x;
  else {
    static_cast<uint16_t*>(p.dst)[i] = (uint16_t)x;
    if (p.dst_lo) static_cast<uint16_t*>(p.dst_lo)[i] = (uint16_t)(x >> 16);
  }
}

// Generic axis permutation with conversion: one destination element per
// thread iteration, destination written contiguously.
template <int SK, int DK>
__device__ inline void permute_body(const PermArgs& p) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < p.total; i += step) {
    int64_t r = i, off = 0;
    for (int a = p.naxes - 1; a >= 0; --a) {
      const int l = p.log2[a];
      off += (r & (((int64_t)1 << l) - 1)) * p.sstride[a];
      r >>= l;
    }
    perm_store<DK>(p, i, perm_load<SK, DK>(p, off));
  }
}

// A permutation of index bits, in tiles of 2^TB elements: the tile's bits hold
// the lowest ones of the source and of the destination, so a workgroup reads
// runs of the source, exchanges through LDS and writes runs of the
// destination.  The generic form gathers single elements: 2^26 floats in an
// order that mixes all bits moved 0.5 GB in 530 us, this form in 165;
// 2^20 floats 9.8 us, now 5.2.
// Bit j of an element's number in source order (ascending source address) is
// source bit sbit[j] and tile bit pos[j]; bit j of a tile position is
// destination bit dbit[j]; bit j of the tile number adds osrc[j] to the source
// and odst[j] to the destination bits.  (32-bit members: a member read by a
// uniform index is one aligned scalar load.)
struct PermTileMap {
  int nouter;
  int sbit[12], pos[12], dbit[12];
  int osrc[kMaxPermAxes], odst[kMaxPermAxes];
};

// LDS word of tile position d: a run of the source often has its bits at
// positions five and above, which would all share a bank
__device__ inline int perm_slot(int d) { return d ^ ((d >> 5) & 31); }

template <int SK, int DK, int TB>
__global__ void __launch_bounds__(256) permute_tile_kernel(PermArgs p, PermTileMap m) {
  constexpr int PER = 1 << (TB - 8);
  typedef typename PermElem<DK>::type T;
  __shared__ T tile[1 << TB];
  const int tid = threadIdx.x;
  int64_t s0 = 0, d0 = 0;
  for (int j = 0; j < m.nouter; ++j) {
    const int64_t bit = (blockIdx.x >> j) & 1;
    s0 += bit << m.osrc[j];
    d0 += bit << m.odst[j];
  }
  int64_t dt = d0;
  int pt = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int64_t bit = (tid >> j) & 1;
    s0 += bit << m.sbit[j];
    pt |= (int)bit << m.pos[j];
    dt += bit << m.dbit[j];
  }
  T v[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    int64_t so = s0;
#pragma unroll
    for (int j = 8; j < TB; ++j) so += (int64_t)((i >> (j - 8)) & 1) << m.sbit[j];
    v[i] = perm_load<SK, DK>(p, so);
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    int po = pt;
#pragma unroll
    for (int j = 8; j < TB; ++j) po |= ((i >> (j - 8)) & 1) << m.pos[j];
    tile[perm_slot(po)] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    int64_t d = dt;
#pragma unroll
    for (int j = 8; j < TB; ++j) d += (int64_t)((i >> (j - 8)) & 1) << m.dbit[j];
    perm_store<DK>(p, d, tile[perm_slot(i * 256 + tid)]);
  }
}

template <int SK, int DK>
__global__ void __launch_bounds__(256) permute_kernel(PermArgs p) {
  permute_body<SK, DK>(p);
}

// blockIdx.z selects the instance
template <int SK, int DK>
__global__ void __launch_bounds__(256) permute_ind_kernel(const PermArgs* __restrict__ p, int64_t slot) {
  permute_body<SK, DK>(*inst_ptr(p, slot));
}

// FP64 -> FP32 or 16-bit planes (hi = rn16(x), lo = rn16(x - hi)); with
// rexp, row i >> cols_log2 is first scaled by its power of two.
template <int DK>
__device__ inline void prep_body(const double* __restrict__ src, void* dst, void* dst_lo, int64_t n,
                                 const int32_t* __restrict__ rexp = nullptr, int cols_log2 = 0,
                                 const uint64_t* __restrict__ colmax = nullptr) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  const int64_t cmask = ((int64_t)1 << cols_log2) - 1;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
    // column scaling as operand_convert_kernel: 2^-e of the column maximum, plus the row exponent
    const float x = colmax ? float(ldexp(src[i], -colmax_exp(colmax[i & cmask]) +
                                                     (rexp ? rexp[i >> cols_log2] : 0)))
                           : rexp ? float(ldexp(src[i], rexp[i >> cols_log2])) : float(src[i]);
    if constexpr (DK == kF32) {
      static_cast<float*>(dst)[i] = x;
    } else {
      const uint16_t h = f_to_h16(x, DK == kF16);
      static_cast<uint16_t*>(dst)[i] = h;
      if (dst_lo) static_cast<uint16_t*>(dst_lo)[i] = f_to_h16(x - h16_to_f(h, DK == kF16), DK == kF16);
    }
  }
}

// blockIdx.y selects the argument block, blockIdx.z the instance
template <int DK>
__global__ void __launch_bounds__(256) prep_ind_kernel(const PrepArgs* __restrict__ a, int64_t slot) {
  const PrepArgs p = inst_ptr(a, slot)[blockIdx.y];
  prep_body<DK>(p.src, p.dst, p.dst_lo, p.n, p.rexp, p.cols_log2, p.colmax);
}

// Operand preparation of a full-definition call: each kernel serves every
// operand in one launch, a run of workgroups each (block0), so a call pays one
// launch a stage instead of one a stage and operand.  At the sizes where that
// matters (a 25-qubit chain in three, scaled split planes) the stages were 15
// of the call's 17 launches and 88 of its 129 us; see the figures below.
struct OperandSet {
  int n;
  int balanced;
  OperandIn in[CQ_MAX_SUBCIRCUITS];
  ExpSumLaunch ex[2];
  int ex_block0[2], ex_blocks[2];
};

// The operand of this workgroup (uniform) and the workgroups it has.
__device__ inline int operand_of(const OperandSet& s, int nblocks, int& blocks) {
  int c = 0;
  for (int i = 1; i < s.n; ++i)
    if ((int)blockIdx.x >= s.in[i].block0) c = i;
  blocks = (c + 1 < s.n ? s.in[c + 1].block0 : nblocks) - s.in[c].block0;
  return c;
}

// Clears the maxima that the next stages fold into with atomics.
__global__ void __launch_bounds__(256) operand_clear_kernel(OperandSet s, int rows) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int c = 0; c < s.n; ++c) {
    const OperandIn& in = s.in[c];
    if (rows && in.rowmax)
      for (int64_t i = i0; i < in.rows; i += step) in.rowmax[i] = 0ull;
    if (in.colmax)
      for (int64_t i = i0; i < (int64_t)1 << in.cols_log2; i += step) in.colmax[i] = 0ull;
  }
}

// max_b |src[l][b]| per row.  A wave takes 64 consecutive entries at a time:
// rows of at most 64 columns share a wave (a reduction over each row's lanes),
// longer rows have a wave each, or 2^split workgroups where the rows alone would
// leave the chip idle (4 rows of 2^20 columns: 4 waves walked 32 MiB); those
// fold with one atomic a workgroup into maxima cleared before.
__global__ void __launch_bounds__(256) operand_rowmax_kernel(OperandSet s, int clear) {
  int nb;
  const OperandIn& in = s.in[operand_of(s, gridDim.x, nb)];
  const int64_t blk = (int)blockIdx.x - in.block0;
  if (clear && in.colmax)
    for (int64_t i = blk * 256 + threadIdx.x; i < (int64_t)1 << in.cols_log2; i += (int64_t)nb * 256)
      in.colmax[i] = 0ull;
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)nb * 4;
  const int cl = in.cols_log2;
  if (cl <= 6) {
    const int64_t n = in.rows << cl;
    for (int64_t w = blk * 4 + (threadIdx.x >> 6); w * 64 < n; w += waves) {
      const int64_t i = w * 64 + lane;
      double m = i < n ? fabs(in.src[i]) : 0.0;
      m = fmax(0.0, m);
      for (int o = (1 << cl) >> 1; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
      if (i < n && (lane & ((1 << cl) - 1)) == 0) in.rowmax[i >> cl] = (uint64_t)__double_as_longlong(m);
    }
    return;
  }
  const int64_t units = in.rows << in.split;
  const int64_t len = (int64_t)1 << (cl - in.split);  // a multiple of 64
  // a wave a unit, or a workgroup where rows are split: one atomic a workgroup
  // (with one a wave and 2^11 parts a row the atomics on 4 rows took 90 us)
  const int wave = threadIdx.x >> 6, per = in.split ? 4 : 1;
  __shared__ double part[4];
  for (int64_t u = in.split ? blk : blk * 4 + wave; u < units; u += in.split ? nb : waves) {
    const int64_t sub = len / per;
    const double* p = in.src + u * len + (in.split ? wave * sub : 0) + lane;
    double m = 0.0;
    int64_t c = 0;
    for (; c + 512 <= sub; c += 512) {
      double v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = p[c + 64 * j];
#pragma unroll
      for (int j = 0; j < 8; ++j) m = fmax(m, fabs(v[j]));
    }
    for (; c < sub; c += 64) m = fmax(m, fabs(p[c]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    if (in.split == 0) {
      if (lane == 0) in.rowmax[u] = (uint64_t)__double_as_longlong(m);
      continue;
    }
    if (lane == 0) part[wave] = m;
    __syncthreads();
    if (threadIdx.x == 0)
      atomicMax(reinterpret_cast<unsigned long long*>(in.rowmax + (u >> in.split)),
                (unsigned long long)__double_as_longlong(fmax(fmax(part[0], part[1]), fmax(part[2], part[3]))));
    __syncthreads();
  }
}

// Column maxima of the rows as scaled by the balance: a thread folds `split`
// rows of one column, eight loads in flight, then one atomic (a plain store
// where one thread holds the whole column).  64 rows a thread in one chain of
// loads left 4^5 x 2^7 entries 2048 threads and 12 us.
constexpr int kColRows = 16;
__global__ void __launch_bounds__(256) operand_colmax_kernel(OperandSet s) {
  int nb;
  const OperandIn& in = s.in[operand_of(s, gridDim.x, nb)];
  const int cl = in.cols_log2, per = in.split;
  const int64_t cols = (int64_t)1 << cl;
  const int64_t total = (in.rows + per - 1) / per * cols;
  for (int64_t t = ((int64_t)blockIdx.x - in.block0) * 256 + threadIdx.x; t < total; t += (int64_t)nb * 256) {
    const int64_t col = t & (cols - 1), r0 = (t >> cl) * per;
    const int64_t r1 = r0 + per < in.rows ? r0 + per : in.rows;
    double m = 0.0;
    for (int64_t r = r0; r < r1; r += 8) {
      double x[8];
      int e[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {  // the last row again past the end: a maximum does not change
        const int64_t q = r + j < r1 ? r + j : r1 - 1;
        x[j] = in.src[(q << cl) + col];
        e[j] = in.rexp ? in.rexp[q] : 0;
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) m = fmax(m, fabs(ldexp(x[j], e[j])));
    }
    if (per >= in.rows) in.colmax[col] = (uint64_t)__double_as_longlong(m);
    else atomicMax(reinterpret_cast<unsigned long long*>(in.colmax + col),
                   (unsigned long long)__double_as_longlong(m));
  }
}

// y as a 16-bit hi part: through FP32 (x = float(y)), or, for scaled columns,
// in one rounding -- the two differ where x is a tie of the 16-bit type, and
// each form of operand keeps its own.
template <int DK>
__device__ inline uint16_t hi_part(double y, float x, bool scaled) {
  if constexpr (DK == kF16) return scaled ? __builtin_bit_cast(uint16_t, _Float16(y)) : f_to_h16(x, true);
  else return scaled ? __builtin_bit_cast(uint16_t, __bf16(y)) : f_to_h16(x, false);
}

// y rounded to FP32.  The empty statement keeps that rounding: without it the
// compiler turns a following conversion to 16 bits into one rounding of y.
__device__ inline float to_f32(double y) {
  float x = float(y);
  asm("" : "+v"(x));
  return x;
}

template <int DK>
__device__ inline void store_planes(const OperandIn& in, int64_t i, double y) {
  const float x = to_f32(y);
  if constexpr (DK == kF32) {
    static_cast<float*>(in.dst)[i] = x;
  } else {
    const uint16_t h = hi_part<DK>(y, x, in.colmax != nullptr);
    static_cast<uint16_t*>(in.dst)[i] = h;
    if (in.dst_lo) static_cast<uint16_t*>(in.dst_lo)[i] = f_to_h16(x - h16_to_f(h, DK == kF16), DK == kF16);
  }
}

// FP64 -> FP32 or 16-bit planes (hi = rn16(x), lo = rn16(x - hi)), row l scaled
// by 2^rexp[l] and column b by 2^-e of its maximum (exact); bound by memory.
// Four elements a thread (two 16-byte loads, one 8- or 16-byte store a plane)
// where `wide` says that rows hold them and the addresses are aligned.  The
// last workgroups sum the output exponents, which need the maxima alone.
template <int DK>
__global__ void __launch_bounds__(256) operand_convert_kernel(OperandSet s, int nblocks) {
  typedef double d2_t __attribute__((ext_vector_type(2)));
  typedef float f4_t __attribute__((ext_vector_type(4)));
  typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
  if ((int)blockIdx.x >= nblocks) {
    const int q = (int)blockIdx.x >= s.ex_block0[1] ? 1 : 0;
    const ExpSumLaunch& x = s.ex[q];
    const int64_t step = (int64_t)s.ex_blocks[q] * 256;
    for (int64_t r = ((int64_t)blockIdx.x - s.ex_block0[q]) * 256 + threadIdx.x; r < x.count; r += step) {
      int e = 0;
      for (int c = 0; c < x.n; ++c)
        e += colmax_exp(x.colmax[c][(r >> x.shift[c]) & ((1ll << x.bits[c]) - 1)]);
      x.out[r] = e;
    }
    return;
  }
  int nb;
  const OperandIn& in = s.in[operand_of(s, nblocks, nb)];
  const int64_t n = in.rows << in.cols_log2;
  const int cl = in.cols_log2;
  const int64_t cmask = ((int64_t)1 << cl) - 1;
  const int64_t t0 = ((int64_t)blockIdx.x - in.block0) * 256 + threadIdx.x, step = (int64_t)nb * 256;
  if (!in.wide) {
    for (int64_t i = t0; i < n; i += step) {
      int e = in.rexp ? in.rexp[i >> cl] : 0;
      if (in.colmax) e -= colmax_exp(in.colmax[i & cmask]);
      store_planes<DK>(in, i, ldexp(in.src[i], e));
    }
    return;
  }
  for (int64_t i = t0; i < n >> 2; i += step) {
    const d2_t v0 = reinterpret_cast<const d2_t*>(in.src)[2 * i];
    const d2_t v1 = reinterpret_cast<const d2_t*>(in.src)[2 * i + 1];
    const double d[4] = {v0[0], v0[1], v1[0], v1[1]};
    int e[4];
    const int er = in.rexp ? in.rexp[(4 * i) >> cl] : 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = er;
    if (in.colmax) {
      const uint64_t* cm = in.colmax + ((4 * i) & cmask);
#pragma unroll
      for (int u = 0; u < 4; ++u) e[u] -= colmax_exp(cm[u]);
    }
    double y[4];
    float x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      y[u] = ldexp(d[u], e[u]);
      x[u] = to_f32(y[u]);
    }
    if constexpr (DK == kF32) {
      reinterpret_cast<f4_t*>(in.dst)[i] = f4_t{x[0], x[1], x[2], x[3]};
    } else {
      u16x4 h, l;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        h[u] = hi_part<DK>(y[u], x[u], in.colmax != nullptr);
        l[u] = f_to_h16(x[u] - h16_to_f(h[u], DK == kF16), DK == kF16);
      }
      reinterpret_cast<u16x4*>(in.dst)[i] = h;
      if (in.dst_lo) reinterpret_cast<u16x4*>(in.dst_lo)[i] = l;
    }
  }
}

// Binary exponent of a positive finite x (x = f * 2^e, f in [1, 2)).
__device__ inline int bexp(double x) { return ilogb(x); }

__device__ inline unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long w = __shfl_xor(v, o, 64);
    v = w > v ? w : v;
  }
  return v;
}

__device__ inline int wave_max_i32(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

// The largest v of a wave whose lanes are all active, the same in every lane:
// lane moves of the vector ALU within rows of 16 lanes, then scalars (a
// shuffle is an LDS access a step).
__device__ __forceinline__ int wave_max_full(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0xb1, 0xf, 0xf, false));   // lane ^ 1
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x4e, 0xf, 0xf, false));   // lane ^ 2
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false));  // mirrored in 8 lanes
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xf, 0xf, false));  // mirrored in 16
  return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
             max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

constexpr int kBalanceRounds = 4;
constexpr int kBalThreads = 1024;
constexpr int kBalLog = 10;            // log2 kBalThreads
constexpr int kBalFixed = kBalLog / 2;  // digit positions fixed per thread
constexpr int kBalUnroll = 4;

// The offset per subcircuit that brings its largest scaled row (smax) to the
// floor of their mean; they sum to zero.
__device__ inline void balance_offsets(int n_sub, const int* smax, int* goff) {
  int n = 0, last = -1;
  long long sum = 0;
  for (int c = 0; c < n_sub; ++c)
    if (smax[c] != INT_MIN) {
      sum += smax[c];
      ++n;
      last = c;
    }
  const long long mean = n ? (sum >= 0 ? sum / n : -((-sum + n - 1) / n)) : 0;
  long long tot = 0;
  for (int c = 0; c < n_sub; ++c) {
    goff[c] = smax[c] == INT_MIN ? 0 : (int)(mean - smax[c]);
    tot += goff[c];
  }
  if (last >= 0) goff[last] -= (int)tot;
}

// The balance of few rows (kBalSmallRows over all subcircuits), in one
// workgroup.  Only the binary exponents of the maxima are used, and a scaled
// row's exponent is its own plus its digits' shares (exact while it stays a
// finite normal number: entries within 2^+-200 of one, whatever the shares), so
// the rows are read once, as exponents held in LDS, and a round is additions:
// every thread adds its rows' shares, a wave a (subcircuit, position) folds
// the four digits' rows, a thread a cut makes the step.  Reading the rows from
// memory and comparing FP64 maxima in every round (below) took 34 us for 1104
// rows in three subcircuits.  What is left is latency (barriers, LDS lookups):
// 12.3 us with shuffled maxima, four barriers a round and every subcircuit's
// first rows on wave 0; 10.2 with lane moves, three barriers, rows spread.
// Rows that a round scales past the range of a double count as infinite (no
// step), or as zero.
constexpr int kBalSmallRows = 8192;
constexpr int kExpNone = -16384, kExpInf = 16384;

__device__ __forceinline__ void balance_small(const BalanceArgs& b) {
  __shared__ int16_t ex[kBalSmallRows], cur[kBalSmallRows];
  __shared__ int pm[CQ_MAX_SUBCIRCUITS * CQ_MAX_LOCAL_CUTS][4];
  // of a row with digit d there; positions from the low end of the row number,
  // zeros past the subcircuit's last (where the digit is 0)
  __shared__ int share[CQ_MAX_SUBCIRCUITS * CQ_MAX_LOCAL_CUTS][4];
  __shared__ int smax[CQ_MAX_SUBCIRCUITS], goff[CQ_MAX_SUBCIRCUITS];
  __shared__ int changed[kBalanceRounds];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the thread's first row of a subcircuit whose rows begin at `base`: small
  // subcircuits fall to different waves
  const auto first = [&](int base) { return (tid - base) & (kBalThreads - 1); };
  int base = 0;
  for (int c = 0; c < b.n_sub; ++c) {
    const int rows = 1 << (2 * b.k[c]);
    for (int l = first(base); l < rows; l += kBalThreads) {
      const double x = __longlong_as_double((long long)b.rowmax[c][l]);
      ex[base + l] = (int16_t)(x > 0.0 ? isfinite(x) ? bexp(x) : kExpInf : kExpNone);
    }
    base += rows;
  }
  if (tid < CQ_MAX_SUBCIRCUITS * CQ_MAX_LOCAL_CUTS * 4) (&share[0][0])[tid] = 0;
  if (tid < CQ_MAX_SUBCIRCUITS) smax[tid] = INT_MIN;
  if (tid < kBalanceRounds) changed[tid] = 0;
  // the cut of this thread, and where its two sides are
  int u = 0, w = 0;
  if (tid < b.K) {
    u = b.up[tid] * CQ_MAX_LOCAL_CUTS + b.k[b.up[tid]] - 1 - b.pos_up[tid];
    w = b.down[tid] * CQ_MAX_LOCAL_CUTS + b.k[b.down[tid]] - 1 - b.pos_down[tid];
  }
  const auto row_exp = [&](int c, int l) {
    int e = 0;
#pragma unroll
    for (int q = 0; q < CQ_MAX_LOCAL_CUTS; ++q) e += share[c * CQ_MAX_LOCAL_CUTS + q][(l >> (2 * q)) & 3];
    return e;
  };
  __syncthreads();
  for (int round = 0; round < kBalanceRounds; ++round) {
    base = 0;
    for (int c = 0; c < b.n_sub; ++c) {
      const int rows = 1 << (2 * b.k[c]);
      for (int l = first(base); l < rows; l += kBalThreads) {
        const int x = ex[base + l];
        int y = x;
        if (x > kExpNone && x < kExpInf) {
          y = x + row_exp(c, l);
          y = y > 1023 ? kExpInf : y < -1074 ? kExpNone : y;
        }
        cur[base + l] = (int16_t)y;
      }
      base += rows;
    }
    __syncthreads();
    int task = 0;
    base = 0;
    for (int c = 0; c < b.n_sub; ++c) {
      const int k = b.k[c];
      for (int p = 0; p < k; ++p, ++task) {
        if ((task & (kBalThreads / 64 - 1)) != wave) continue;
        const int sh = 2 * p, low = (1 << sh) - 1;
        int m[4] = {kExpNone, kExpNone, kExpNone, kExpNone};
        for (int q = lane; q < 1 << (2 * k - 2); q += 64) {
          const int l = base + (((q & ~low) << 2) | (q & low));
#pragma unroll
          for (int d = 0; d < 4; ++d) m[d] = max(m[d], (int)cur[l + (d << sh)]);
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) m[d] = wave_max_full(m[d]);
        if (lane < 4) pm[c * CQ_MAX_LOCAL_CUTS + p][lane] = lane == 0 ? m[0] : lane == 1 ? m[1] : lane == 2 ? m[2] : m[3];
      }
      base += 1 << (2 * k);
    }
    __syncthreads();
    // as below: half the difference of the two sides, less the mean over the
    // digits, on the upstream side (the downstream side carries its negative)
    if (tid < b.K) {
      int st[4], sum = 0;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int mu = pm[u][d], md = pm[w][d];
        st[d] = 0;
        if (mu > kExpNone && mu < kExpInf && md > kExpNone && md < kExpInf) st[d] = (md - mu) / 2;
        sum += st[d];
      }
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        int e = share[u][d] + st[d] - sum / 4;
        e = e > 200 ? 200 : (e < -200 ? -200 : e);
        if (e != share[u][d]) {
          share[u][d] = e;
          share[w][d] = -e;
          changed[round] = 1;
        }
      }
    }
    __syncthreads();
    if (!changed[round]) break;
  }
  // every subcircuit's largest scaled row, and the offsets
  base = 0;
  for (int c = 0; c < b.n_sub; ++c) {
    const int rows = 1 << (2 * b.k[c]);
    int sm = INT_MIN;
    for (int l = first(base); l < rows; l += kBalThreads) {
      const int x = ex[base + l];
      if (x > kExpNone && x < kExpInf) sm = max(sm, x + row_exp(c, l));
    }
    sm = wave_max_full(sm);
    if (lane == 0 && sm != INT_MIN) atomicMax(&smax[c], sm);
    base += rows;
  }
  __syncthreads();
  if (tid == 0) balance_offsets(b.n_sub, smax, goff);
  __syncthreads();
  base = 0;
  for (int c = 0; c < b.n_sub; ++c) {
    const int rows = 1 << (2 * b.k[c]);
    for (int l = first(base); l < rows; l += kBalThreads) b.rexp[c][l] = row_exp(c, l) + goff[c];
    base += rows;
  }
}

// One workgroup: per (subcircuit, digit position, digit) the largest row
// maximum (LDS), then e_j(d) per cut and digit, then every row's exponent.
// The largest row of a subcircuit sits at each digit's maximum over the other
// positions, so the exponents carry an offset per subcircuit (the same for
// all its rows); a final constant per subcircuit, summing to zero over the
// subcircuits (every term of Eq. 1 takes one row of each), brings every
// subcircuit's largest scaled row to their common mean binary exponent.
// Row maxima are FP64 bit patterns of values >= 0, so their unsigned order is
// the value order.  Thread t reads rows l = 1024 i + t: the digits held in the
// low 10 bits of l (the last five positions) are fixed per thread, so one
// running maximum serves them, and their share of a row's exponent is one
// number per thread; the digits above come from i, the same for the whole
// workgroup, and each thread keeps a maximum per (position, digit) for those.
// A handful of LDS atomics per thread remain (a contended atomic per row and
// position took over a millisecond for 4^8 rows), and four rows are loaded
// before any is used.
__device__ __forceinline__ void balance_body(const BalanceArgs& b) {
  constexpr int kHi = CQ_MAX_LOCAL_CUTS > kBalFixed ? CQ_MAX_LOCAL_CUTS - kBalFixed : 1;
  __shared__ unsigned long long pmax[CQ_MAX_SUBCIRCUITS][CQ_MAX_LOCAL_CUTS][4];
  __shared__ int ej[CQ_MAX_CUTS][4];
  __shared__ int stp[CQ_MAX_CUTS][4];
  __shared__ int smax[CQ_MAX_SUBCIRCUITS];
  __shared__ int goff[CQ_MAX_SUBCIRCUITS];
  __shared__ int changed;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  int64_t all = 0;
  for (int c = 0; c < b.n_sub; ++c) all += (int64_t)1 << (2 * b.k[c]);
  if (all <= kBalSmallRows) {
    balance_small(b);
    return;
  }
  for (int i = tid; i < CQ_MAX_CUTS * 4; i += blockDim.x) (&ej[0][0])[i] = 0;
  if (tid < CQ_MAX_SUBCIRCUITS) smax[tid] = INT_MIN;
  // exponent share of position p (digit d) in a row of subcircuit c
  auto share = [&](int c, int p, int d) {
    const int j = b.cut_of[c][p];
    return b.up[j] == c ? ej[j][d] : -ej[j][d];
  };
  // the positions fixed by tid, and those taken from i
  auto share_lo = [&](int c, int k, int nhi) {
    int e = 0;
    for (int p = nhi; p < k; ++p) e += share(c, p, (tid >> (2 * (k - 1 - p))) & 3);
    return e;
  };
  auto share_hi = [&](int c, int nhi, int64_t i) {
    int e = 0;
    for (int q = 0; q < nhi; ++q) e += share(c, q, (int)((i >> (2 * (nhi - 1 - q))) & 3));
    return e;
  };
  // Each round measures the per-digit maxima of the rows as scaled by the
  // current exponents and moves every cut's pair of exponents to meet them.
  // In a subcircuit with many cuts the largest row with digit d at one
  // position is decided by the other positions' extreme digits (one row out
  // of 4^(k-1) when the labels are far apart), so a single round leaves much
  // of the spread; a few rounds remove it.
  __syncthreads();
  for (int round = 0; round < kBalanceRounds; ++round) {
    for (int i = tid; i < CQ_MAX_SUBCIRCUITS * CQ_MAX_LOCAL_CUTS * 4; i += blockDim.x)
      (&pmax[0][0][0])[i] = 0ull;
    if (tid == 0) changed = 0;
    __syncthreads();
    for (int c = 0; c < b.n_sub; ++c) {
      const int k = b.k[c];
      const int64_t rows = (int64_t)1 << (2 * k);
      const int64_t iters = (rows + kBalThreads - 1) >> kBalLog;
      const int nhi = k > kBalFixed ? k - kBalFixed : 0;  // positions 0..nhi-1 take their digit from i
      const int elo = share_lo(c, k, nhi);
      unsigned long long tm = 0ull;
      unsigned long long hm[kHi][4];
#pragma unroll
      for (int q = 0; q < kHi; ++q)
#pragma unroll
        for (int d = 0; d < 4; ++d) hm[q][d] = 0ull;
      for (int64_t i0 = 0; i0 < iters; i0 += kBalUnroll) {
        unsigned long long v[kBalUnroll];
#pragma unroll
        for (int u = 0; u < kBalUnroll; ++u) {
          const int64_t l = ((i0 + u) << kBalLog) + tid;
          v[u] = ((i0 + u < iters) & (l < rows)) ? b.rowmax[c][l] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < kBalUnroll; ++u) {
          const int64_t i = i0 + u;
          unsigned long long x = v[u];
          if (x)
            x = (unsigned long long)__double_as_longlong(
                ldexp(__longlong_as_double((long long)x), elo + share_hi(c, nhi, i)));
          tm = x > tm ? x : tm;
#pragma unroll
          for (int q = 0; q < kHi; ++q) {
            const int d = q < nhi ? (int)((i >> (2 * (nhi - 1 - q))) & 3) : -1;
#pragma unroll
            for (int e = 0; e < 4; ++e) hm[q][e] = ((d == e) & (x > hm[q][e])) ? x : hm[q][e];
          }
        }
      }
      for (int p = nhi; p < k; ++p) {
        const int d = (tid >> (2 * (k - 1 - p))) & 3;
        if (tm) atomicMax(&pmax[c][p][d], tm);
      }
#pragma unroll
      for (int q = 0; q < kHi; ++q) {
        if (q >= nhi) break;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const unsigned long long w = wave_max_u64(hm[q][e]);
          if (lane == 0 && w) atomicMax(&pmax[c][q][e], w);
        }
      }
    }
    __syncthreads();
    for (int i = tid; i < b.K * 4; i += blockDim.x) {
      const int j = i >> 2, d = i & 3;
      const double mu = __longlong_as_double((long long)pmax[b.up[j]][b.pos_up[j]][d]);
      const double md = __longlong_as_double((long long)pmax[b.down[j]][b.pos_down[j]][d]);
      int step = 0;
      if (mu > 0.0 && md > 0.0 && isfinite(mu) && isfinite(md)) {
        const int diff = bexp(md) - bexp(mu);
        step = diff >= 0 ? diff / 2 : -((-diff) / 2);  // round toward zero: exact halves
      }
      stp[j][d] = step;
    }
    __syncthreads();
    // A step common to a cut's four digits only moves scale between its two
    // subcircuits (the final offsets undo that); applied round after round
    // it overshoots in a subcircuit with many cuts, so only the part that
    // differs between digits is applied.
    for (int i = tid; i < b.K * 4; i += blockDim.x) {
      const int j = i >> 2, d = i & 3;
      const int sum = stp[j][0] + stp[j][1] + stp[j][2] + stp[j][3];
      const int mean = sum >= 0 ? sum / 4 : -((-sum) / 4);
      int e = ej[j][d] + stp[j][d] - mean;
      e = e > 200 ? 200 : (e < -200 ? -200 : e);
      if (e != ej[j][d]) {
        ej[j][d] = e;
        changed = 1;
      }
    }
    __syncthreads();
    const int more = changed;
    __syncthreads();  // every thread has read the flag before the next round clears it
    if (!more) break;
  }
  // every subcircuit's largest scaled row (binary exponent)
  for (int c = 0; c < b.n_sub; ++c) {
    const int k = b.k[c];
    const int64_t rows = (int64_t)1 << (2 * k);
    const int64_t iters = (rows + kBalThreads - 1) >> kBalLog;
    const int nhi = k > kBalFixed ? k - kBalFixed : 0;
    const int elo = share_lo(c, k, nhi);
    int sm = INT_MIN;
    for (int64_t i0 = 0; i0 < iters; i0 += kBalUnroll) {
      unsigned long long v[kBalUnroll];
#pragma unroll
      for (int u = 0; u < kBalUnroll; ++u) {
        const int64_t l = ((i0 + u) << kBalLog) + tid;
        v[u] = ((i0 + u < iters) & (l < rows)) ? b.rowmax[c][l] : 0ull;
      }
#pragma unroll
      for (int u = 0; u < kBalUnroll; ++u) {
        const double x = __longlong_as_double((long long)v[u]);
        if (x > 0.0 && isfinite(x)) sm = max(sm, bexp(x) + elo + share_hi(c, nhi, i0 + u));
      }
    }
    sm = wave_max_i32(sm);
    if (lane == 0 && sm != INT_MIN) atomicMax(&smax[c], sm);
  }
  __syncthreads();
  if (tid == 0) balance_offsets(b.n_sub, smax, goff);
  __syncthreads();
  // every row's exponent: its digits' shares plus its subcircuit's offset
  for (int c = 0; c < b.n_sub; ++c) {
    const int k = b.k[c];
    const int64_t rows = (int64_t)1 << (2 * k);
    const int nhi = k > kBalFixed ? k - kBalFixed : 0;
    const int elo = share_lo(c, k, nhi) + goff[c];
    for (int64_t i = 0; (i << kBalLog) < rows; ++i) {
      const int64_t l = (i << kBalLog) + tid;
      if (l < rows) b.rexp[c][l] = elo + share_hi(c, nhi, i);
    }
  }
}

__global__ void __launch_bounds__(kBalThreads) balance_kernel(BalanceArgs b) { balance_body(b); }

// The balance of one instance of a dynamic-definition batch (grid z), from
// its program; nothing when the recursion converts nothing.
__global__ void __launch_bounds__(kBalThreads) balance_ind_kernel(const DDProgram* P, const DDLevel* lv,
                                                                  int64_t slot) {
  P = inst_ptr(P, slot);
  lv = inst_ptr(lv, slot);
  if (!P->balance) return;
  bool any = false;
  for (int c = 0; c < P->n_sub; ++c) any = any | (lv->prep[c].n > 0);
  if (!any) return;
  balance_body(P->bal);
}

// Column maxima of the reduced entries for the column scaling: subcircuit
// blockIdx.y of instance blockIdx.z, 64 columns a workgroup, its four waves
// taking every fourth row; values carry the balance's row exponents, as the
// conversion applies them.
__global__ void __launch_bounds__(256) colmax_ind_kernel(const DDProgram* P, const DDLevel* lv, int64_t slot) {
  __shared__ double part[4][64];
  P = inst_ptr(P, slot);
  lv = inst_ptr(lv, slot);
  const int c = blockIdx.y;
  if (!P->cscale || c >= P->n_sub) return;
  const PrepArgs& pa = lv->prep[c];
  const int64_t cols = (int64_t)1 << pa.cols_log2;
  if (pa.n <= 0 || (int64_t)blockIdx.x * 64 >= cols) return;
  const int64_t rows = P->rows[c];
  const int32_t* rexp = P->balance ? P->bal.rexp[c] : nullptr;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t b = (int64_t)blockIdx.x * 64 + lane;
  double m = 0.0;
  if (b < cols)
    for (int64_t r = w; r < rows; r += 4) {
      const double x = pa.src[(r << pa.cols_log2) + b];
      m = fmax(m, fabs(rexp ? ldexp(x, rexp[r]) : x));
    }
  part[w][lane] = m;
  __syncthreads();
  if (w == 0 && b < cols)
    P->colmax[c][b] = (uint64_t)__double_as_longlong(
        fmax(fmax(part[0][lane], part[1][lane]), fmax(part[2][lane], part[3][lane])));
}

// Output exponents of the last GEMM (step `step`): blockIdx.y 0 its rows
// (z * M + m), 1 its columns (n); each the sum over the group's subcircuits of
// the exponent of the column that bits shift .. shift + na_c - 1 select.
__global__ void __launch_bounds__(256) expsum_ind_kernel(const DDProgram* P, const DDState* st,
                                                         const DDLevel* lv, int step, int64_t slot) {
  P = inst_ptr(P, slot);
  st = inst_ptr(st, slot);
  lv = inst_ptr(lv, slot);
  if (!P->cscale) return;
  const GemmArgs& g = lv->gemm[step];
  if (g.tiles <= 0) return;
  const int q = blockIdx.y;
  const int64_t count = q == 0 ? g.tiles / (g.tilesM * g.tilesN) * g.M : g.N;
  int32_t* const out = q == 0 ? P->rowexp : P->colexp;
  // each member's bit field, the same for every row: its shift and width
  const int n = P->fac_n[q];
  int sh[CQ_MAX_SUBCIRCUITS], sub[CQ_MAX_SUBCIRCUITS];
  int64_t mk[CQ_MAX_SUBCIRCUITS];
#pragma unroll
  for (int i = 0; i < CQ_MAX_SUBCIRCUITS; ++i) {
    sh[i] = 0;
    sub[i] = 0;
    mk[i] = 0;
    if (i < n) {
      const SymLog& sl = P->fac_shift[q][i];
      int s = sl.c0;
      for (int c = 0; c < CQ_MAX_SUBCIRCUITS; ++c)
        if ((sl.mask >> c) & 1u) s += st->na[c];
      sh[i] = s;
      sub[i] = P->fac_sub[q][i];
      mk[i] = ((int64_t)1 << st->na[sub[i]]) - 1;
    }
  }
  // four consecutive rows a thread, one 16-byte store where the address
  // allows it; a member whose field starts at bit 2 or above has the same
  // column for all four
  const int64_t stepg = (int64_t)gridDim.x * blockDim.x * 4;
  for (int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4; r < count; r += stepg) {
    int e[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < CQ_MAX_SUBCIRCUITS; ++i) {
      if (i >= n) continue;
      const uint64_t* cm = P->colmax[sub[i]];
      if (sh[i] >= 2) {
        const int v = colmax_exp(cm[(r >> sh[i]) & mk[i]]);
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] += v;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] += colmax_exp(cm[((r + j) >> sh[i]) & mk[i]]);
      }
    }
    if (r + 4 <= count && (reinterpret_cast<uintptr_t>(out + r) & 15) == 0) {
      *reinterpret_cast<int4*>(out + r) = make_int4(e[0], e[1], e[2], e[3]);
    } else {
      for (int j = 0; j < 4 && r + j < count; ++j) out[r + j] = e[j];
    }
  }
}

// Tile maxima of the row exponents over the 128-row tiles of each batch
// (z * tilesM + mt), for the tile bounds when A is shared across batches
// (else the bounds weight every element by its own exponents and this
// exits); one wave a tile, its lanes taking every 64th row (coalesced), then
// a wave maximum.
__global__ void __launch_bounds__(256) exptmax_ind_kernel(const DDProgram* P, const DDLevel* lv, int step,
                                                          int64_t slot) {
  P = inst_ptr(P, slot);
  lv = inst_ptr(lv, slot);
  if (!P->cscale) return;
  const GemmArgs& g = lv->gemm[step];
  if (g.tiles <= 0) return;
  const int64_t Z = g.tiles / (g.tilesM * g.tilesN);
  if (g.sAz != 0 || Z == 1) return;
  const int64_t count = Z * g.tilesM;
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
  // t is the same for every lane of a wave, so every lane reaches the shuffles
  for (int64_t t = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); t < count; t += waves) {
    int e = INT_MIN;
    const int64_t z = t / g.tilesM, m0 = (t - z * g.tilesM) * 128;
    const int64_t m1 = m0 + 128 < g.M ? m0 + 128 : g.M;
    for (int64_t m = m0 + lane; m < m1; m += 64) e = max(e, P->rowexp[z * g.M + m]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) e = max(e, __shfl_xor(e, o));
    if (lane == 0) P->rowtmax[t] = e;
  }
}

// Row maxima of the reduced entries for the balance: subcircuit blockIdx.y of
// instance blockIdx.z, one wave per row of its current 2^cols_log2 columns
// (zeros for a subcircuit the recursion does not convert).
__global__ void __launch_bounds__(256) rowmax_ind_kernel(const DDProgram* P, const DDLevel* lv, int64_t slot) {
  P = inst_ptr(P, slot);
  lv = inst_ptr(lv, slot);
  const int c = blockIdx.y;
  if (!P->balance || c >= P->n_sub) return;
  const PrepArgs& pa = lv->prep[c];
  const bool live = pa.n > 0;
  const int64_t rows = P->rows[c];
  const int64_t cols = (int64_t)1 << pa.cols_log2;
  uint64_t* const rm = const_cast<uint64_t*>(P->bal.rowmax[c]);
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t r = wave; r < rows; r += waves) {
    double m = 0.0;
    if (live) {
      const double* row = pa.src + (r << pa.cols_log2);
      for (int64_t col = lane; col < cols; col += 64) m = fmax(m, fabs(row[col]));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    if (lane == 0) rm[r] = (uint64_t)__double_as_longlong(m);
  }
}

// ---------------------------------------------------------------------------
// Attribution (Section 3.1).  Two separable passes, both FP64:
//  1. measured ends: U[j][lm][b] = sum_m prod_u sigma(lm_u, m_u)
//                                  * V[j][basis(lm)][compose(b, m)]
//  2. initialised ends: E[row(li, lm)][b] = sum_j prod_t alpha(li_t, j_t) U[j][lm][b]
// Thread per output element; b is the fastest index so stores are contiguous.
// ---------------------------------------------------------------------------

struct AttrArgs {
  const double* V;
  double* U;
  double* E;
  int r, o, n, w, k;
  int out_pos[CQ_MAX_WIDTH];
  int meas_pos[CQ_MAX_WIDTH];
  int64_t init_w[CQ_MAX_WIDTH];
  int64_t meas_w[CQ_MAX_WIDTH];
};

// Measurement basis of a label: I and Z -> Z basis (0), X -> 1, Y -> 2.
__device__ inline int basis_of(int l) { return l == 3 ? 0 : l; }

// alpha(label, prepared state) for states |0>, |1>, |+>, |+i> = 0..3; only
// called on the support (I, Z: |0>, |1>; X: also |+>; Y: also |+i>).
__device__ inline double alpha_coef(int l, int d) {
  if (d >= 2) return 2.0;
  if (l == 0) return 1.0;
  if (l == 3) return d == 0 ? 1.0 : -1.0;
  return -1.0;
}

__global__ void __launch_bounds__(256) attr_meas_kernel(AttrArgs a) {
  const int64_t nb = (int64_t)1 << a.n;
  const int64_t nlm = (int64_t)1 << (2 * a.o);
  const int64_t total = ((int64_t)1 << (2 * a.r)) * nlm * nb;
  int64_t pow3o = 1;
  for (int u = 0; u < a.o; ++u) pow3o *= 3;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += step) {
    const int64_t b = i % nb;
    const int64_t lm = (i / nb) % nlm;
    const int64_t j = i / (nb * nlm);
    int64_t x0 = 0;
    for (int q = 0; q < a.n; ++q)
      if ((b >> (a.n - 1 - q)) & 1) x0 |= (int64_t)1 << a.out_pos[q];
    int64_t beta = 0;
    for (int u = 0; u < a.o; ++u) beta = 3 * beta + basis_of((lm >> (2 * (a.o - 1 - u))) & 3);
    const double* Vj = a.V + ((j * pow3o + beta) << a.w);
    double sum = 0.0;
    for (int m = 0; m < (1 << a.o); ++m) {
      int64_t x = x0;
      bool neg = false;
      for (int u = 0; u < a.o; ++u) {
        if ((m >> (a.o - 1 - u)) & 1) {
          x |= (int64_t)1 << a.meas_pos[u];
          if (((lm >> (2 * (a.o - 1 - u))) & 3) != 0) neg = !neg;
        }
      }
      const double v = Vj[x];
      sum += neg ? -v : v;
    }
    a.U[i] = sum;
  }
}

__global__ void __launch_bounds__(256) attr_init_kernel(AttrArgs a) {
  const int64_t nb = (int64_t)1 << a.n;
  const int64_t nlm = (int64_t)1 << (2 * a.o);
  const int64_t nli = (int64_t)1 << (2 * a.r);
  const int64_t total = nli * nlm * nb;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += step) {
    const int64_t b = i % nb;
    const int64_t lm = (i / nb) % nlm;
    const int64_t li = i / (nb * nlm);
    // support of each init digit: I, Z -> {0, 1}; X -> {0, 1, 2}; Y -> {0, 1, 3}
    int64_t combos = 1;
    for (int t = 0; t < a.r; ++t) {
      const int l = (li >> (2 * (a.r - 1 - t))) & 3;
      combos *= (l == 1 || l == 2) ? 3 : 2;
    }
    double sum = 0.0;
    for (int64_t c = 0; c < combos; ++c) {
      int64_t rem = c, j = 0;
      double coef = 1.0;
      // mixed radix over the supports, last init slot fastest
      for (int t = a.r - 1; t >= 0; --t) {
        const int l = (li >> (2 * (a.r - 1 - t))) & 3;
        const int sz = (l == 1 || l == 2) ? 3 : 2;
        int d = (int)(rem % sz);
        rem /= sz;
        if (d == 2) d = (l == 1) ? 2 : 3;
        j += (int64_t)d << (2 * (a.r - 1 - t));
        coef *= alpha_coef(l, d);
      }
      sum += coef * a.U[(j * nlm + lm) * nb + b];
    }
    int64_t row = 0;
    for (int t = 0; t < a.r; ++t) row += ((li >> (2 * (a.r - 1 - t))) & 3) * a.init_w[t];
    for (int u = 0; u < a.o; ++u) row += ((lm >> (2 * (a.o - 1 - u))) & 3) * a.meas_w[u];
    a.E[row * nb + b] = sum;
  }
}

// Register forms of the two passes for few cut ends (the common case): a
// thread owns one (j, b) -- or one (lm, b) -- reads each input element once
// and produces every label of its group by butterflies in registers, so V and
// U each cross HBM once.
//  * measured ends, O <= 2: the 3^O x 2^O values V[j][beta][compose(b, m)]
//    give all 4^O labels lm;
//  * initialised ends, R <= 3: per init digit, (|0>, |1>, |+>, |+i>) ->
//    (I, X, Y, Z) = (d0 + d1, -d0 - d1 + 2 d2, -d0 - d1 + 2 d3, d0 - d1).
template <int O>
__global__ void __launch_bounds__(256) attr_meas_reg_kernel(AttrArgs a) {
  constexpr int NB = O == 0 ? 1 : (O == 1 ? 3 : 9);   // 3^O bases
  constexpr int NM = 1 << O;                          // outcomes of the measured bits
  constexpr int NL = 1 << (2 * O);                    // labels
  const int64_t nb = (int64_t)1 << a.n;
  const int64_t total = ((int64_t)1 << (2 * a.r)) * nb;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += step) {
    const int64_t b = i & (nb - 1);
    const int64_t j = i >> a.n;
    int64_t x0 = 0;
    for (int q = 0; q < a.n; ++q)
      if ((b >> (a.n - 1 - q)) & 1) x0 |= (int64_t)1 << a.out_pos[q];
    double v[NB][NM];
#pragma unroll
    for (int beta = 0; beta < NB; ++beta)
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        int64_t x = x0;
#pragma unroll
        for (int u = 0; u < O; ++u)
          if ((m >> (O - 1 - u)) & 1) x |= (int64_t)1 << a.meas_pos[u];
        v[beta][m] = a.V[((j * NB + beta) << a.w) + x];
      }
#pragma unroll
    for (int lm = 0; lm < NL; ++lm) {
      int beta = 0;
#pragma unroll
      for (int u = 0; u < O; ++u) beta = 3 * beta + basis_of((lm >> (2 * (O - 1 - u))) & 3);
      double sum = 0.0;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        bool neg = false;
#pragma unroll
        for (int u = 0; u < O; ++u)
          if (((m >> (O - 1 - u)) & 1) && ((lm >> (2 * (O - 1 - u))) & 3) != 0) neg = !neg;
        sum += neg ? -v[beta][m] : v[beta][m];
      }
      a.U[(j * NL + lm) * nb + b] = sum;
    }
  }
}

template <int R>
__global__ void __launch_bounds__(256) attr_init_reg_kernel(AttrArgs a) {
  constexpr int NJ = 1 << (2 * R);
  const int64_t nb = (int64_t)1 << a.n;
  const int64_t nlm = (int64_t)1 << (2 * a.o);
  const int64_t total = nlm * nb;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += step) {
    const int64_t b = i & (nb - 1);
    const int64_t lm = i >> a.n;
    double u[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) u[j] = a.U[(j * nlm + lm) * nb + b];
#pragma unroll
    for (int t = 0; t < R; ++t) {
      const int sd = 1 << (2 * (R - 1 - t));  // stride of init digit t
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if ((j / sd) % 4 != 0) continue;
        const double d0 = u[j], d1 = u[j + sd], d2 = u[j + 2 * sd], d3 = u[j + 3 * sd];
        u[j] = d0 + d1;                       // I
        u[j + sd] = 2.0 * d2 - d0 - d1;       // X
        u[j + 2 * sd] = 2.0 * d3 - d0 - d1;   // Y
        u[j + 3 * sd] = d0 - d1;              // Z
      }
    }
    int64_t mrow = 0;
    for (int q = 0; q < a.o; ++q) mrow += ((lm >> (2 * (a.o - 1 - q))) & 3) * a.meas_w[q];
#pragma unroll
    for (int li = 0; li < NJ; ++li) {
      int64_t row = mrow;
#pragma unroll
      for (int t = 0; t < R; ++t) row += ((li >> (2 * (R - 1 - t))) & 3) * a.init_w[t];
      a.E[row * nb + b] = u[li];
    }
  }
}

// Three or four measured ends: the 2^O outcome values of one (init string j,
// basis string beta, column b) give, by O sum/difference butterflies, the
// values of all 2^z labels measured in that basis (z digits Z, each I or Z;
// an X or Y digit keeps its difference).  The basis is the grid's y, so which
// of the 2^O butterfly results are labels is the same for the whole workgroup.
// Bound by reading V once.  The measured bits of the outcome index may sit
// anywhere: STAGE takes 64 columns a wave, loads their 64 * 2^O values in
// address order (16 bytes a lane; the 6 lowest output bits and the measured
// bits hold every index bit below the seventh, so a run is at least 512
// bytes), and regroups them per column through LDS.  Loading each column's
// values where they are makes a wave touch 64 lines per load when the
// measured bits are the lowest ones, and the lines leave the 32 KB L1 before
// their other values are asked for.  Fewer than 64 columns take that plain
// form (the table is small then).
// A wave's LDS writes are read by its other lanes (a wave's LDS operations
// run in order; this keeps the compiler from moving them across).
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

constexpr int kAttrPad = 66;  // doubles between two outcomes' rows of 64 columns in LDS

template <int O, bool STAGE>
__global__ void __launch_bounds__(256) attr_meas_wht_kernel(AttrArgs a) {
  constexpr int NM = 1 << O;
  typedef double d2_t __attribute__((ext_vector_type(2)));
  __shared__ double sh[STAGE ? 4 : 1][STAGE ? NM * kAttrPad : 1];
  const int64_t nb = (int64_t)1 << a.n;
  int64_t nbasis = 1;
#pragma unroll
  for (int u = 0; u < O; ++u) nbasis *= 3;
  const int beta = blockIdx.y;
  // per butterfly result m: its label lm (or none: an X or Y digit's sum)
  int digit[O];
  {
    int rest = beta;
#pragma unroll
    for (int u = O - 1; u >= 0; --u) {
      digit[u] = rest % 3;
      rest /= 3;
    }
  }
  const int64_t total = ((int64_t)1 << (2 * a.r)) << a.n;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // the grid covers whole waves of columns when STAGE (nb >= 64), so a wave
  // enters and leaves the loop together
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += step) {
    const int64_t bl = i & (nb - 1), j = i >> a.n;
    const double* Vj = a.V + ((j * nbasis + beta) << a.w);
    double v[NM];
    if constexpr (STAGE) {
      // wave's first column deposited around the measured bits (its low 6 bits are 0)
      int64_t x0 = bl - lane;
#pragma unroll
      for (int u = O - 1; u >= 0; --u)  // measured positions ascend from the last slot to the first
        x0 = ((x0 >> a.meas_pos[u]) << (a.meas_pos[u] + 1)) | (x0 & (((int64_t)1 << a.meas_pos[u]) - 1));
      // bit t of a value's number in address order: the t-th lowest of the
      // wave's index bits, a column bit or an outcome bit
      int64_t xl = 0, xq[NM / 2];
      int sl = 0, sq[NM / 2], s1 = 0;
#pragma unroll
      for (int q = 0; q < NM / 2; ++q) {
        xq[q] = 0;
        sq[q] = 0;
      }
      int pos = 0, um = O - 1, bc = 0;  // next position, next measured slot, next column bit
#pragma unroll
      for (int t = 0; t < 6 + O; ++t) {
        const bool meas = um >= 0 && (bc >= 6 || a.meas_pos[um >= 0 ? um : 0] == pos);
        if (meas) pos = a.meas_pos[um];
        const int place = meas ? kAttrPad << (O - 1 - um) : 1 << bc;
        if (t == 0) {
          s1 = place;
        } else if (t < 7) {
          xl |= (int64_t)((lane >> (t - 1)) & 1) << pos;
          sl += ((lane >> (t - 1)) & 1) * place;
        } else {
#pragma unroll
          for (int q = 0; q < NM / 2; ++q)
            if ((q >> (t - 7)) & 1) {
              xq[q] |= (int64_t)1 << pos;
              sq[q] += place;
            }
        }
        um -= meas ? 1 : 0;
        bc += meas ? 0 : 1;
        ++pos;
      }
      double* S = sh[wave];
      d2_t ld[NM / 2];
#pragma unroll
      for (int q = 0; q < NM / 2; ++q) ld[q] = *reinterpret_cast<const d2_t*>(Vj + (x0 | xl | xq[q]));
#pragma unroll
      for (int q = 0; q < NM / 2; ++q) {
        S[sl + sq[q]] = ld[q][0];
        S[sl + sq[q] + s1] = ld[q][1];
      }
      wave_lds_fence();
#pragma unroll
      for (int m = 0; m < NM; ++m) v[m] = S[m * kAttrPad + lane];
      wave_lds_fence();  // the next columns overwrite S
    } else {
      int64_t x0 = bl;
#pragma unroll
      for (int u = O - 1; u >= 0; --u)
        x0 = ((x0 >> a.meas_pos[u]) << (a.meas_pos[u] + 1)) | (x0 & (((int64_t)1 << a.meas_pos[u]) - 1));
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        int64_t x = x0;
#pragma unroll
        for (int u = 0; u < O; ++u)
          if ((m >> (O - 1 - u)) & 1) x |= (int64_t)1 << a.meas_pos[u];
        v[m] = Vj[x];
      }
    }
#pragma unroll
    for (int h = 1; h < NM; h <<= 1)
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        if (m & h) continue;
        const double x = v[m], y = v[m | h];
        v[m] = x + y;
        v[m | h] = x - y;
      }
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      int lm = 0;
      bool label = true;
#pragma unroll
      for (int u = 0; u < O; ++u) {
        const int bit = (m >> (O - 1 - u)) & 1;
        label = label & (digit[u] == 0 || bit == 1);
        lm = 4 * lm + (digit[u] == 0 ? 3 * bit : digit[u]);
      }
      if (label) a.U[((j << (2 * O)) + lm) * nb + bl] = v[m];
    }
  }
}

// Four initialised ends: the 4^4 init strings of one (lm, b) are spread over
// the four 16-lane groups of a wave by the first digit, 64 to a lane, so three
// digits transform in registers and the first by cross-lane reads; U is read
// and E written in runs of 16 columns (128 bytes).  Bound by U and E crossing
// once each; one thread per entry re-read each U value for every label row in
// its support (4^8 rows of 2^10 columns with both passes: 15.7 ms then, 0.88
// ms with this kernel and the one above; 3.25 GB cannot be done without).
__global__ void __launch_bounds__(256) attr_init4_kernel(AttrArgs a) {
  const int64_t nb = (int64_t)1 << a.n;
  const int64_t total = nb << (2 * a.o);  // (lm, b)
  const int lane = threadIdx.x & 63, grp = lane >> 4, l16 = lane & 15;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t i0 = wave * 16; i0 < total; i0 += waves * 16) {
    const int64_t i = i0 + l16;
    const bool in = i < total;
    const double* src = a.U + (int64_t)grp * 64 * total + (in ? i : total - 1);
    double u[64];
#pragma unroll
    for (int j = 0; j < 64; ++j) u[j] = src[j * total];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const int sd = 1 << (2 * (2 - t));  // stride of init digit t + 1
#pragma unroll
      for (int j = 0; j < 64; ++j) {
        if ((j / sd) % 4 != 0) continue;
        const double d0 = u[j], d1 = u[j + sd], d2 = u[j + 2 * sd], d3 = u[j + 3 * sd];
        u[j] = d0 + d1;                       // I
        u[j + sd] = 2.0 * d2 - d0 - d1;       // X
        u[j + 2 * sd] = 2.0 * d3 - d0 - d1;   // Y
        u[j + 3 * sd] = d0 - d1;              // Z
      }
    }
    const int64_t b = i & (nb - 1), lm = i >> a.n;
    int64_t mrow = (int64_t)grp * a.init_w[0];
    for (int q = 0; q < a.o; ++q) mrow += ((lm >> (2 * (a.o - 1 - q))) & 3) * a.meas_w[q];
    // group 1 (X) takes 2 d2 - d0 - d1 and group 2 (Y) 2 d3 - d0 - d1
    const int other = (grp == 1 ? 32 : grp == 2 ? 48 : 0) + l16;
    const bool two = grp == 1 || grp == 2;
#pragma unroll
    for (int j = 0; j < 64; ++j) {
      const double d0 = __shfl(u[j], l16), d1 = __shfl(u[j], 16 + l16), d = __shfl(u[j], other);
      const double x = two ? 2.0 * d - d0 : d0;
      const double y = grp == 0 ? x + d1 : x - d1;
      const int64_t row = mrow + (j >> 4) * a.init_w[1] + ((j >> 2) & 3) * a.init_w[2] + (j & 3) * a.init_w[3];
      if (in) a.E[(row << a.n) + b] = y;
    }
  }
}

// Both passes in one kernel for up to two measured and two initialised cut
// ends (the dynamic-definition subcircuits): a thread owns one output column
// b and walks the 3^O measurement bases; for each basis it loads the
// 4^R x 2^O variant values V[j][basis][compose(b, m)] it needs (each element
// of V is read once overall), forms U[j][lm] for the labels lm measured in
// that basis, runs the init butterflies over j in registers and writes the
// 4^R entries of each such lm.  U never reaches memory, so HBM sees V once
// and E once.  Same operations in the same order as the two register passes.
template <int R, int O>
__global__ void __launch_bounds__(256) attr_fused_kernel(AttrArgs a) {
  constexpr int NJ = 1 << (2 * R);                   // init digit strings
  constexpr int NB = O == 0 ? 1 : (O == 1 ? 3 : 9);  // 3^O bases
  constexpr int NM = 1 << O;                         // outcomes of the measured bits
  constexpr int NL = 1 << (2 * O);                   // measured labels
  const int64_t nb = (int64_t)1 << a.n;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < nb; b += step) {
    int64_t x0 = 0;
    for (int q = 0; q < a.n; ++q)
      if ((b >> (a.n - 1 - q)) & 1) x0 |= (int64_t)1 << a.out_pos[q];
    int64_t xm[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      int64_t x = x0;
#pragma unroll
      for (int u = 0; u < O; ++u)
        if ((m >> (O - 1 - u)) & 1) x |= (int64_t)1 << a.meas_pos[u];
      xm[m] = x;
    }
#pragma unroll
    for (int beta = 0; beta < NB; ++beta) {
      double v[NJ][NM];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int m = 0; m < NM; ++m) v[j][m] = a.V[(((int64_t)j * NB + beta) << a.w) + xm[m]];
#pragma unroll
      for (int lm = 0; lm < NL; ++lm) {
        int bl = 0;
#pragma unroll
        for (int u = 0; u < O; ++u) bl = 3 * bl + basis_of((lm >> (2 * (O - 1 - u))) & 3);
        if (bl != beta) continue;
        double uj[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          double sum = 0.0;
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            bool neg = false;
#pragma unroll
            for (int u = 0; u < O; ++u)
              if (((m >> (O - 1 - u)) & 1) && ((lm >> (2 * (O - 1 - u))) & 3) != 0) neg = !neg;
            sum += neg ? -v[j][m] : v[j][m];
          }
          uj[j] = sum;
        }
#pragma unroll
        for (int t = 0; t < R; ++t) {
          const int sd = 1 << (2 * (R - 1 - t));  // stride of init digit t
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            if ((j / sd) % 4 != 0) continue;
            const double d0 = uj[j], d1 = uj[j + sd], d2 = uj[j + 2 * sd], d3 = uj[j + 3 * sd];
            uj[j] = d0 + d1;                       // I
            uj[j + sd] = 2.0 * d2 - d0 - d1;       // X
            uj[j + 2 * sd] = 2.0 * d3 - d0 - d1;   // Y
            uj[j + 3 * sd] = d0 - d1;              // Z
          }
        }
        int64_t mrow = 0;
#pragma unroll
        for (int q = 0; q < O; ++q) mrow += ((lm >> (2 * (O - 1 - q))) & 3) * a.meas_w[q];
#pragma unroll
        for (int li = 0; li < NJ; ++li) {
          int64_t row = mrow;
#pragma unroll
          for (int t = 0; t < R; ++t) row += ((li >> (2 * (R - 1 - t))) & 3) * a.init_w[t];
          a.E[row * nb + b] = uj[li];
        }
      }
    }
  }
}

// Indirect launches size their grid for the largest shape and loop; a
// moderate cap keeps the empty workgroups of smaller shapes cheap.
unsigned grid_ind(int64_t total) {
  int64_t b = (total + 255) / 256;
  if (b > 4096) b = 4096;
  if (b < 1) b = 1;
  return (unsigned)b;
}

unsigned grid_for(int64_t total) {
  int64_t b = (total + 255) / 256;
  if (b > 1 << 20) b = 1 << 20;
  if (b < 1) b = 1;
  return (unsigned)b;
}


int kind_of(DType t, bool f16) {
  if (t == DType::F64) return kF64;
  if (t == DType::F32) return kF32;
  return f16 ? kF16 : kBF16;
}

// tb: bits of a tile (10 for doubles), 0 for the generic kernel
template <int SK, int DK>
void permute_dispatch(dim3 grid, const PermArgs& a, int tb, const PermTileMap& m, hipStream_t s) {
  if constexpr (DK != kF64)
    if (tb == 12) {
      hipLaunchKernelGGL((permute_tile_kernel<SK, DK, 12>), grid, dim3(256), 0, s, a, m);
      return;
    }
  if (tb == 10) hipLaunchKernelGGL((permute_tile_kernel<SK, DK, 10>), grid, dim3(256), 0, s, a, m);
  else hipLaunchKernelGGL((permute_kernel<SK, DK>), grid, dim3(256), 0, s, a);
}

template <int SK>
void permute_dispatch_dst(int dk, dim3 grid, const PermArgs& a, int tb, const PermTileMap& m, hipStream_t s) {
  switch (dk) {
    case kF64: permute_dispatch<SK, kF64>(grid, a, tb, m, s); break;
    case kF32: permute_dispatch<SK, kF32>(grid, a, tb, m, s); break;
    case kBF16: permute_dispatch<SK, kBF16>(grid, a, tb, m, s); break;
    default: permute_dispatch<SK, kF16>(grid, a, tb, m, s); break;
  }
}

template <int SK>
void permute_ind_dispatch_dst(int dk, dim3 grid, const PermArgs* a, int64_t slot, hipStream_t s) {
  switch (dk) {
    case kF64: hipLaunchKernelGGL((permute_ind_kernel<SK, kF64>), grid, dim3(256), 0, s, a, slot); break;
    case kF32: hipLaunchKernelGGL((permute_ind_kernel<SK, kF32>), grid, dim3(256), 0, s, a, slot); break;
    case kBF16: hipLaunchKernelGGL((permute_ind_kernel<SK, kBF16>), grid, dim3(256), 0, s, a, slot); break;
    default: hipLaunchKernelGGL((permute_ind_kernel<SK, kF16>), grid, dim3(256), 0, s, a, slot); break;
  }
}

}  // namespace

hipError_t launch_permute_indirect(const PermArgs* dev, DType ts, DType td, bool f16,
                                   int64_t max_total, hipStream_t stream, InstSpan span) {
  if (max_total <= 0 || span.n <= 0) return hipSuccess;
  const dim3 grid(grid_ind(max_total), 1, (unsigned)span.n);
  const int sk = kind_of(ts, f16), dk = kind_of(td, f16);
  switch (sk) {
    case kF64: permute_ind_dispatch_dst<kF64>(dk, grid, dev, span.stride, stream); break;
    case kF32: permute_ind_dispatch_dst<kF32>(dk, grid, dev, span.stride, stream); break;
    case kBF16: permute_ind_dispatch_dst<kBF16>(dk, grid, dev, span.stride, stream); break;
    default: permute_ind_dispatch_dst<kF16>(dk, grid, dev, span.stride, stream); break;
  }
  return hipGetLastError();
}

hipError_t launch_prep_indirect(const PrepArgs* dev, int count, DType t, bool f16, int64_t max_n,
                                hipStream_t stream, InstSpan span) {
  if (max_n <= 0 || count <= 0 || span.n <= 0) return hipSuccess;
  const dim3 grid(grid_ind(max_n), (unsigned)count, (unsigned)span.n);
  if (t == DType::F32)
    hipLaunchKernelGGL((prep_ind_kernel<kF32>), grid, dim3(256), 0, stream, dev, span.stride);
  else if (f16)
    hipLaunchKernelGGL((prep_ind_kernel<kF16>), grid, dim3(256), 0, stream, dev, span.stride);
  else
    hipLaunchKernelGGL((prep_ind_kernel<kBF16>), grid, dim3(256), 0, stream, dev, span.stride);
  return hipGetLastError();
}

namespace {
constexpr int kPermBigBits = 22;

// The tile map of a permutation of `bits` index bits in tiles of 2^tb: false
// when it is not one (a source stride that is no power of two, or that two
// bits share), is smaller than a tile, or has more tiles than a launch has
// workgroups of 256 (fewer than 2^32 threads), which the generic kernel takes.
// The tile takes source and destination bits in turn from the lowest.
bool perm_tile_map(const PermLaunch& p, int bits, int tb, PermTileMap& m) {
  if (bits < tb || bits > kMaxPermAxes || bits - tb > 23) return false;
  int src_of[64], dst_of[64];  // source bit of a destination bit, and back (-1: none)
  std::fill(dst_of, dst_of + 64, -1);
  int b = 0;
  for (int x = p.naxes - 1; x >= 0; --x)
    for (int l = 0; l < p.log2[x]; ++l, ++b) {
      const int64_t st = p.sstride[x];
      if (st <= 0 || (st & (st - 1)) || st > ((int64_t)1 << 60) >> l) return false;
      const int sb = __builtin_ctzll((unsigned long long)st) + l;
      if (dst_of[sb] >= 0) return false;
      src_of[b] = sb;
      dst_of[sb] = b;
    }
  bool in[64] = {};  // destination bits of the tile
  int n = 0, ds = 0, ss = 0;
  while (n < tb) {
    while (ds < bits && in[ds]) ++ds;
    if (ds < bits && n < tb) in[ds] = true, ++n;
    while (ss < 64 && (dst_of[ss] < 0 || in[dst_of[ss]])) ++ss;
    if (ss < 64 && n < tb) in[dst_of[ss]] = true, ++n;
  }
  int pos_of[64];
  m.nouter = 0;
  n = 0;
  for (int d = 0; d < bits; ++d) {
    if (in[d]) {
      pos_of[d] = n;
      m.dbit[n++] = d;
    } else {
      m.osrc[m.nouter] = src_of[d];
      m.odst[m.nouter++] = d;
    }
  }
  n = 0;
  for (int sb = 0; sb < 64; ++sb)
    if (dst_of[sb] >= 0 && in[dst_of[sb]]) {
      m.sbit[n] = sb;
      m.pos[n++] = pos_of[dst_of[sb]];
    }
  return true;
}
}  // namespace

hipError_t launch_permute(const PermLaunch& p, hipStream_t stream) {
  PermArgs a;
  a.src = p.src.p;
  a.src_lo = p.src.t == DType::H16X2 ? p.src.lo : nullptr;
  a.dst = p.dst;
  a.dst_lo = p.td == DType::H16X2 ? p.dst_lo : nullptr;
  a.naxes = p.naxes;
  int bits = 0;
  for (int i = 0; i < p.naxes; ++i) {
    a.log2[i] = p.log2[i];
    a.sstride[i] = p.sstride[i];
    bits += p.log2[i];
  }
  a.total = (int64_t)1 << bits;
  a.alpha = p.alpha;
  a.nfac = p.nfac;
  for (int c = 0; c < CQ_MAX_SUBCIRCUITS; ++c) {
    a.colmax[c] = p.colmax[c];
    a.fac_shift[c] = p.fac_shift[c];
    a.fac_bits[c] = p.fac_bits[c];
  }
  const int sk = kind_of(p.src.t, p.f16), dk = kind_of(p.td, p.f16);
  // tiles of 2^10 elements give 2^20 elements 1024 workgroups; larger ones
  // read and write longer runs, except doubles, whose runs are twice as long
  // and whose tiles would leave four workgroups a CU (2^10 against 2^12: 2^20
  // floats 5.2 us against 8, 2^24 33 against 26.5, 2^26 204 against 165, 2^26
  // doubles 270 against 338)
  PermTileMap m;
  const int tb = bits >= kPermBigBits && p.td != DType::F64 ? 12 : 10;
  const bool tiled = perm_tile_map(p, bits, tb, m);
  const dim3 grid(tiled ? 1u << (bits - tb) : grid_for(a.total));
  switch (sk) {
    case kF64: permute_dispatch_dst<kF64>(dk, grid, a, tiled ? tb : 0, m, stream); break;
    case kF32: permute_dispatch_dst<kF32>(dk, grid, a, tiled ? tb : 0, m, stream); break;
    case kBF16: permute_dispatch_dst<kBF16>(dk, grid, a, tiled ? tb : 0, m, stream); break;
    default: permute_dispatch_dst<kF16>(dk, grid, a, tiled ? tb : 0, m, stream); break;
  }
  return hipGetLastError();
}

hipError_t launch_dd_balance(const DDProgram* prog, const DDLevel* lv, int n_sub, int64_t max_rows,
                             hipStream_t stream, InstSpan span) {
  if (n_sub <= 0 || max_rows <= 0 || span.n <= 0) return hipSuccess;
  int64_t gx = (max_rows * 64 + 255) / 256;
  if (gx > 1024) gx = 1024;
  hipLaunchKernelGGL(rowmax_ind_kernel, dim3((unsigned)gx, (unsigned)n_sub, (unsigned)span.n), dim3(256), 0,
                     stream, prog, lv, span.stride);
  hipLaunchKernelGGL(balance_ind_kernel, dim3(1, 1, (unsigned)span.n), dim3(kBalThreads), 0, stream, prog, lv,
                     span.stride);
  return hipGetLastError();
}

hipError_t launch_dd_colmax(const DDProgram* prog, const DDLevel* lv, int n_sub, int64_t max_cols,
                            hipStream_t stream, InstSpan span) {
  if (n_sub <= 0 || max_cols <= 0 || span.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(colmax_ind_kernel, dim3((unsigned)((max_cols + 63) / 64), (unsigned)n_sub, (unsigned)span.n),
                     dim3(256), 0, stream, prog, lv, span.stride);
  return hipGetLastError();
}

hipError_t launch_dd_expsum(const DDProgram* prog, const DDState* st, const DDLevel* lv, int step,
                            int64_t max_rows, int64_t max_cols, hipStream_t stream, InstSpan span) {
  if (span.n <= 0) return hipSuccess;
  const int64_t most = max_rows > max_cols ? max_rows : max_cols;
  hipLaunchKernelGGL(expsum_ind_kernel, dim3(grid_ind(most), 2, (unsigned)span.n), dim3(256), 0, stream, prog,
                     st, lv, step, span.stride);
  // one wave a tile: a few tiles a wave at most
  hipLaunchKernelGGL(exptmax_ind_kernel, dim3(grid_ind(most / 2 + 1), 1, (unsigned)span.n), dim3(256), 0, stream,
                     prog, lv, step, span.stride);
  return hipGetLastError();
}

// The workgroups of one operand in a launch: one for every 256 work items, at
// most 2^17 (the kernels loop).
int operand_blocks(int64_t items) {
  const int64_t b = (items + 255) / 256;
  return (int)(b < 1 ? 1 : b > 1 << 17 ? 1 << 17 : b);
}

hipError_t launch_balance(const BalanceLaunch& b, hipStream_t stream) {
  OperandSet s;
  s.n = b.n_in;
  s.balanced = b.balanced;
  for (int c = 0; c < CQ_MAX_SUBCIRCUITS; ++c) s.in[c] = b.in[c];
  for (int q = 0; q < 2; ++q) s.ex[q] = b.ex[q];
  int blocks = 0;
  bool scaled = false;
  int64_t most = 1;  // maxima of one operand
  for (int c = 0; c < s.n; ++c) {
    scaled = scaled || s.in[c].colmax;
    most = std::max(most, std::max(s.in[c].rows, (int64_t)1 << s.in[c].cols_log2));
  }
  const dim3 clear((unsigned)operand_blocks(most));
  if (b.stage == BalanceLaunch::kExponents) {
    bool atomics = false;
    for (int c = 0; c < s.n; ++c) {
      OperandIn& in = s.in[c];
      const int64_t n = in.rows << in.cols_log2;
      in.block0 = blocks;
      in.split = 0;
      if (in.cols_log2 > 6) {
        // rows are split until 2048 workgroups (8 a CU) have work, or a part
        // is down to 2048 entries (one round of loads in flight)
        while ((in.rows << in.split) < 2048 && in.cols_log2 - in.split > 11) ++in.split;
        atomics = atomics || in.split > 0;
        const int64_t units = in.rows << in.split;
        blocks += operand_blocks(in.split ? units * 256 : units * 64);
      } else {
        blocks += operand_blocks(n);
      }
    }
    if (s.n > 0) {
      if (atomics) hipLaunchKernelGGL(operand_clear_kernel, clear, dim3(256), 0, stream, s, 1);
      hipLaunchKernelGGL(operand_rowmax_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, s,
                         scaled && !atomics ? 1 : 0);
    }
    hipLaunchKernelGGL(balance_kernel, dim3(1), dim3(kBalThreads), 0, stream, static_cast<const BalanceArgs&>(b));
    return hipGetLastError();
  }
  if (s.n <= 0) return hipSuccess;
  if (scaled) {
    bool atomics = false;
    for (int c = 0; c < s.n; ++c) {
      OperandIn& in = s.in[c];
      in.split = kColRows;
      in.block0 = blocks;
      atomics = atomics || in.rows > kColRows;
      blocks += operand_blocks((in.rows + kColRows - 1) / kColRows << in.cols_log2);
    }
    // the balance's first stage has cleared them already
    if (atomics && !s.balanced) hipLaunchKernelGGL(operand_clear_kernel, clear, dim3(256), 0, stream, s, 0);
    hipLaunchKernelGGL(operand_colmax_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, s);
  }
  blocks = 0;
  const auto al = [](const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; };
  for (int c = 0; c < s.n; ++c) {
    OperandIn& in = s.in[c];
    const int64_t n = in.rows << in.cols_log2;
    in.wide = n % 4 == 0 && ((!in.rexp && !in.colmax) || in.cols_log2 >= 2) && al(in.src, 16) &&
              al(in.dst, b.t == DType::F32 ? 16 : 8) && (!in.dst_lo || al(in.dst_lo, 8));
    in.block0 = blocks;
    blocks += operand_blocks(in.wide ? n / 4 : n);
  }
  int grid = blocks;
  for (int q = 0; q < 2; ++q) {
    s.ex_block0[q] = grid;
    s.ex_blocks[q] = s.ex[q].count > 0 ? operand_blocks(s.ex[q].count) : 0;
    grid += s.ex_blocks[q];
  }
  if (b.t == DType::F32)
    hipLaunchKernelGGL((operand_convert_kernel<kF32>), dim3((unsigned)grid), dim3(256), 0, stream, s, blocks);
  else if (b.f16)
    hipLaunchKernelGGL((operand_convert_kernel<kF16>), dim3((unsigned)grid), dim3(256), 0, stream, s, blocks);
  else
    hipLaunchKernelGGL((operand_convert_kernel<kBF16>), dim3((unsigned)grid), dim3(256), 0, stream, s, blocks);
  return hipGetLastError();
}

hipError_t launch_attribute(const AttrLaunch& l, hipStream_t stream) {
  AttrArgs a;
  a.V = l.V;
  a.U = l.U;
  a.E = l.E;
  a.r = l.r;
  a.o = l.o;
  a.n = l.n;
  a.w = l.w;
  a.k = l.k;
  for (int i = 0; i < CQ_MAX_WIDTH; ++i) {
    a.out_pos[i] = l.out_pos[i];
    a.meas_pos[i] = l.meas_pos[i];
    a.init_w[i] = l.init_w[i];
    a.meas_w[i] = l.meas_w[i];
  }
  if (l.r <= 2 && l.o <= 2) {
    const dim3 gf(grid_for((int64_t)1 << l.n));
#define CQ_ATTR_FUSED(R, O)                                                          \
  if (l.r == R && l.o == O) {                                                        \
    hipLaunchKernelGGL((attr_fused_kernel<R, O>), gf, dim3(256), 0, stream, a);     \
    return hipGetLastError();                                                        \
  }
    CQ_ATTR_FUSED(0, 0) CQ_ATTR_FUSED(0, 1) CQ_ATTR_FUSED(0, 2)
    CQ_ATTR_FUSED(1, 0) CQ_ATTR_FUSED(1, 1) CQ_ATTR_FUSED(1, 2)
    CQ_ATTR_FUSED(2, 0) CQ_ATTR_FUSED(2, 1) CQ_ATTR_FUSED(2, 2)
#undef CQ_ATTR_FUSED
  }
  // two passes through U (in slabs of columns whose U stays in the 256 MB
  // last-level cache the 4^8 x 2^10 case took 0.90-0.96 ms against 0.88)
  const int64_t nb = (int64_t)1 << l.n;
  const dim3 gt(grid_for(nb << (2 * (l.r + l.o)))), gm(grid_for(nb << (2 * l.r))), gi(grid_for(nb << (2 * l.o)));
  const bool stage = l.n >= 6 && (reinterpret_cast<uintptr_t>(l.V) & 15) == 0;
  switch (l.o) {
    case 0: hipLaunchKernelGGL(attr_meas_reg_kernel<0>, gm, dim3(256), 0, stream, a); break;
    case 1: hipLaunchKernelGGL(attr_meas_reg_kernel<1>, gm, dim3(256), 0, stream, a); break;
    case 2: hipLaunchKernelGGL(attr_meas_reg_kernel<2>, gm, dim3(256), 0, stream, a); break;
    case 3:
      if (stage) hipLaunchKernelGGL((attr_meas_wht_kernel<3, true>), dim3(gm.x, 27), dim3(256), 0, stream, a);
      else hipLaunchKernelGGL((attr_meas_wht_kernel<3, false>), dim3(gm.x, 27), dim3(256), 0, stream, a);
      break;
    case 4:
      if (stage) hipLaunchKernelGGL((attr_meas_wht_kernel<4, true>), dim3(gm.x, 81), dim3(256), 0, stream, a);
      else hipLaunchKernelGGL((attr_meas_wht_kernel<4, false>), dim3(gm.x, 81), dim3(256), 0, stream, a);
      break;
    default: hipLaunchKernelGGL(attr_meas_kernel, gt, dim3(256), 0, stream, a); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch (l.r) {
    case 0: hipLaunchKernelGGL(attr_init_reg_kernel<0>, gi, dim3(256), 0, stream, a); break;
    case 1: hipLaunchKernelGGL(attr_init_reg_kernel<1>, gi, dim3(256), 0, stream, a); break;
    case 2: hipLaunchKernelGGL(attr_init_reg_kernel<2>, gi, dim3(256), 0, stream, a); break;
    case 3: hipLaunchKernelGGL(attr_init_reg_kernel<3>, gi, dim3(256), 0, stream, a); break;
    case 4: hipLaunchKernelGGL(attr_init4_kernel, dim3(grid_for((nb << (2 * l.o)) * 4)), dim3(256), 0, stream, a); break;
    default: hipLaunchKernelGGL(attr_init_kernel, gt, dim3(256), 0, stream, a); break;
  }
  return hipGetLastError();
}

}  // namespace cq
