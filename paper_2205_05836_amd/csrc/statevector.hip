// State-vector simulation on the device: the noiseless output distribution
// of a circuit of one-qubit unitaries and CZ gates (the ground truth of
// Section 2), and every variant of a subcircuit (Section 3.1: each cut-end
// initialisation |0>, |1>, |+>, |+i> and each measurement basis Z, X, Y).
//
// Amplitudes are FP64 complex, qubit 0 the most significant index bit.
// Gates run in passes: gates whose qubits fit one tile of index bits are
// applied together to tiles of amplitudes held in registers (one workgroup a
// tile, the tile's other index bits fixed), so the state makes one HBM round
// trip per pass instead of one per gate.  A pass may take a later gate that
// commutes with every gate it overtakes (no shared qubit).
//
// A state that starts as a basis state is zero wherever a qubit that no gate
// has acted on differs from its start, so a pass reads and writes only the
// amplitudes whose untouched bits agree with it: 2^t of 2^n while t qubits
// are touched.  The passes are therefore planned so that the touched set
// grows as late as possible (plan_passes).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "internal.hpp"
#include "kernels.hpp"
#include "svplan.hpp"

namespace cq {

namespace {

constexpr int kSvThreads = 256;
constexpr int kLdsTile = 1 << (kMinTileBits - 1);

// A gate of a pass in one word (whole words, so that uniform reads of the
// arguments are aligned scalar loads): bits 0-5 CQ_GATE_U or CQ_GATE_CZ, 6-7
// the form (CQ_GATE_U), 8-15 and 16-23 tile-local bit positions (the second
// for CZ only), 24-31 the matrix (CQ_GATE_U).
typedef uint32_t TileOp;
__host__ __device__ inline int op_kind(TileOp g) { return (int)(g & 0x3fu); }
__host__ __device__ inline int op_form(TileOp g) { return (int)((g >> 6) & 3u); }
__host__ __device__ inline int op_a(TileOp g) { return (int)((g >> 8) & 0xffu); }
__host__ __device__ inline int op_b(TileOp g) { return (int)((g >> 16) & 0xffu); }
__host__ __device__ inline int op_u(TileOp g) { return (int)(g >> 24); }

// One launch: the tile's index bits by local position, the bits that number
// the tiles, and the gates.  mode 0 writes amplitudes back, mode 1 writes
// weight * |amplitude|^2 to `probs` in the same index order.  State blockIdx.y of a
// batch starts as the basis string whose bit init_bit[t] is bit r - 1 - t of
// blockIdx.y (all other bits 0) and lies bstride elements after state 0.
struct TileGroup {
  int32_t k;       // tile bits
  int32_t nops;
  int32_t mode;
  int32_t nouter;  // bits that number the tiles
  int32_t first;   // the state is still its basis string: nothing is read
  int32_t r;
  uint64_t before;  // bits touched before and after the pass: amplitudes whose
  uint64_t after;   // untouched bits differ from the start are zero and not stored
  uint64_t full;    // all index bits
  uint64_t tile;    // the tile's index bits
  uint64_t fixed;   // bits neither in the tile nor numbering tiles (kept at the start's)
  int64_t bstride;
  uint32_t init_bit[CQ_MAX_LOCAL_CUTS];
  uint32_t bits[kMaxTileBits];
  uint32_t outer[CQ_MAX_SV_QUBITS];
  TileOp ops[kMaxOps];
  // (re, im) of u00, u01, u10, u11, or of the two ratios of the normalised form
  double u[kMaxU][8];
  double weight;
};

static_assert(sizeof(TileGroup) + 2 * sizeof(void*) <= 4096, "kernel arguments exceed 4 KiB");

__device__ inline uint64_t start_string(const TileGroup& G, uint32_t y) {
  uint64_t s = 0;
  for (int t = 0; t < G.r; ++t) s |= (uint64_t)((y >> (G.r - 1 - t)) & 1u) << G.init_bit[t];
  return s;
}

struct Complex {
  double re, im;
};

__device__ inline Complex cmul(double ur, double ui, Complex x) {
  return {ur * x.re - ui * x.im, ur * x.im + ui * x.re};
}

// Registers narrower than a full tile: the whole state in LDS, a barrier per
// gate (every amplitude is read and written).
__global__ void __launch_bounds__(kSvThreads) sv_tile_kernel(double2* psi, double* probs, TileGroup G) {
  __shared__ double2 S[kLdsTile];
  psi += blockIdx.y * G.bstride;
  const uint64_t start = start_string(G, blockIdx.y);
  const int n = 1 << G.k;
  for (int t = threadIdx.x; t < n; t += kSvThreads)
    S[t] = G.first ? make_double2((uint64_t)t == start ? 1.0 : 0.0, 0.0) : psi[t];
  __syncthreads();
  for (int gi = 0; gi < G.nops; ++gi) {
    const TileOp g = G.ops[gi];
    if (op_kind(g) == CQ_GATE_U) {
      const double* u = G.u[op_u(g)];
      const int ga = op_a(g);
      const int half = n >> 1, m = 1 << ga;
      for (int p = threadIdx.x; p < half; p += kSvThreads) {
        const int i0 = ((p >> ga) << (ga + 1)) | (p & (m - 1)), i1 = i0 | m;
        const Complex x0{S[i0].x, S[i0].y}, x1{S[i1].x, S[i1].y};
        const Complex a0 = cmul(u[0], u[1], x0), b0 = cmul(u[2], u[3], x1);
        const Complex a1 = cmul(u[4], u[5], x0), b1 = cmul(u[6], u[7], x1);
        S[i0] = make_double2(a0.re + b0.re, a0.im + b0.im);
        S[i1] = make_double2(a1.re + b1.re, a1.im + b1.im);
      }
    } else {
      const int both = (1 << op_a(g)) | (1 << op_b(g));
      for (int t = threadIdx.x; t < n; t += kSvThreads)
        if ((t & both) == both) S[t] = make_double2(-S[t].x, -S[t].y);
    }
    __syncthreads();
  }
  for (int t = threadIdx.x; t < n; t += kSvThreads) {
    const double2 v = S[t];
    if (G.mode == 0) psi[t] = v;
    else probs[t] = v.x * v.x + v.y * v.y;
  }
}

// Full tiles keep the amplitudes in registers: with 2^TB amplitudes and T
// threads, thread t holds local indices t + T e, so the local bits are six
// lane bits, then the wave bits, then the register bits.  A one-qubit gate on
// a register bit pairs two of the thread's own elements; on a lane bit the
// partner comes by a lane move of the vector ALU or by exchanging halves of two
// registers (cross-lane reads went through LDS, the busiest unit: with them and
// general unitaries the last pass of the 30-qubit circuit, 36 unitaries on 2^30
// amplitudes, took 17.5 ms, 14.7 now; it is bound by vector issue, of which the
// products are a third); on a wave bit it goes through LDS.  The host places the pass's busiest qubits on register bits.
// Tiles of 11 bits run as 256 threads of 8 amplitudes, of 12 bits as 256 of 16
// (13 bits as 512 of 16 leave one workgroup a compute unit: the 30-qubit
// circuit took 30.3 ms against 24.6).
template <int TB>
struct TileShape {
  static constexpr int LogT = 8;
  static constexpr int T = 1 << LogT;
  static constexpr int NE = 1 << (TB - LogT);
};

__device__ inline double2 u_row(double r0, double i0, double r1, double i1, double2 x, double2 y) {
  // (r0 + i i0) x + (r1 + i i1) y
  return make_double2(r0 * x.x - i0 * x.y + r1 * y.x - i1 * y.y, r0 * x.y + i0 * x.x + r1 * y.y + i1 * y.x);
}

// x + (r + i i) y
__device__ inline double2 add_scaled(double2 x, double r, double i, double2 y) {
  return make_double2(x.x + r * y.x - i * y.y, x.y + r * y.y + i * y.x);
}

// A one-qubit unitary on a pair in registers.  The normalised form costs four
// FMA an amplitude, the general one eight (see normalize).
template <int F>
__device__ inline void u_pair(double2& x0, double2& x1, const double* u) {
  const double2 a = x0, b = x1;
  if constexpr (F == kNormal) {
    x0 = add_scaled(a, u[0], u[1], b);
    x1 = add_scaled(b, u[2], u[3], a);
  } else {
    x0 = u_row(u[0], u[1], u[2], u[3], a, b);
    x1 = u_row(u[4], u[5], u[6], u[7], a, b);
  }
}

template <int F, int R, int NE>
__device__ inline void u_reg(double2 (&v)[NE], const double* u) {
#pragma unroll
  for (int e = 0; e < NE; ++e)
    if (!(e & (1 << R))) u_pair<F>(v[e], v[e | (1 << R)], u);
}

// Lane bit 5 or 4 of elements a and b changes places with the choice between
// them: a lane then holds both values of the bit of one element (its own for
// the low half, the partner's for the high one).  Applying it again undoes it.
template <int M>
__device__ inline void lane_swap(double2& a, double2& b) {
  uint64_t p[2] = {__builtin_bit_cast(uint64_t, a.x), __builtin_bit_cast(uint64_t, a.y)};
  uint64_t q[2] = {__builtin_bit_cast(uint64_t, b.x), __builtin_bit_cast(uint64_t, b.y)};
  uint32_t pw[4] = {(uint32_t)p[0], (uint32_t)(p[0] >> 32), (uint32_t)p[1], (uint32_t)(p[1] >> 32)};
  uint32_t qw[4] = {(uint32_t)q[0], (uint32_t)(q[0] >> 32), (uint32_t)q[1], (uint32_t)(q[1] >> 32)};
  // in place (the builtin copies its operands first); a swap wants two wait
  // states after a vector write of its operands
#define CQ_SWAP4(op)                                                                                              \
  asm volatile("s_nop 1\n\t" op " %0, %4\n\t" op " %1, %5\n\t" op " %2, %6\n\t" op " %3, %7"                    \
               : "+v"(pw[0]), "+v"(pw[1]), "+v"(pw[2]), "+v"(pw[3]), "+v"(qw[0]), "+v"(qw[1]), "+v"(qw[2]), "+v"(qw[3]))
  if constexpr (M == 32) CQ_SWAP4("v_permlane32_swap_b32");
  else CQ_SWAP4("v_permlane16_swap_b32");
#undef CQ_SWAP4
  for (int i = 0; i < 2; ++i) {
    p[i] = (uint64_t)pw[2 * i] | (uint64_t)pw[2 * i + 1] << 32;
    q[i] = (uint64_t)qw[2 * i] | (uint64_t)qw[2 * i + 1] << 32;
  }
  a = make_double2(__builtin_bit_cast(double, p[0]), __builtin_bit_cast(double, p[1]));
  b = make_double2(__builtin_bit_cast(double, q[0]), __builtin_bit_cast(double, q[1]));
}

// x of lane ^ M, M < 16: by a lane move of the vector ALU, for M = 4 (which
// needs two of those) by a swizzle.
template <int M>
__device__ inline uint32_t lane_xor(uint32_t x) {
  static_assert(M == 1 || M == 2 || M == 4 || M == 8, "within a row");
  if constexpr (M == 4) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 0x101f);
  else return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, M == 1 ? 0xb1 : M == 2 ? 0x4e : 0x128, 0xf, 0xf, true);
}

template <int M>
__device__ inline double lane_xor(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  return __builtin_bit_cast(double, (uint64_t)lane_xor<M>((uint32_t)b) | (uint64_t)lane_xor<M>((uint32_t)(b >> 32)) << 32);
}

// An element whose partner (the other value of its pair) sits elsewhere:
// bit 0 takes u00 * mine + u01 * partner, bit 1 u11 * mine + u10 * partner,
// or in the normalised form mine + ratio * partner.  The coefficients are
// picked once per gate, so each element costs one row, not two and a select.
struct ExchangeCoef {
  double ar, ai, br, bi;  // coefficient of mine, of the partner; or the ratio in a
};

// A coefficient every lane reads alike, taken through the first lane so that
// the per-lane choice below selects values, not addresses (a per-lane
// address would turn each coefficient into a vector load that the gate
// then waits for).
__device__ inline double uniform_coef(const double* p) {
  const uint64_t b = __builtin_bit_cast(uint64_t, *p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}

template <int F>
__device__ inline ExchangeCoef exchange_coef(const double* u, int bit) {
  if constexpr (F != kGeneral) {
    const double r0 = uniform_coef(u + 0), i0 = uniform_coef(u + 1), r1 = uniform_coef(u + 2), i1 = uniform_coef(u + 3);
    return ExchangeCoef{bit ? r1 : r0, bit ? i1 : i0, 0.0, 0.0};
  } else {
    const ExchangeCoef c0{uniform_coef(u + 0), uniform_coef(u + 1), uniform_coef(u + 2), uniform_coef(u + 3)};
    const ExchangeCoef c1{uniform_coef(u + 6), uniform_coef(u + 7), uniform_coef(u + 4), uniform_coef(u + 5)};
    return bit ? c1 : c0;
  }
}

template <int F>
__device__ inline double2 u_exchange(const ExchangeCoef& c, double2 mine, double2 y) {
  if constexpr (F == kNormal) return add_scaled(mine, c.ar, c.ai, y);
  else return u_row(c.ar, c.ai, c.br, c.bi, mine, y);
}

// A gate on lane bit log2 M.
template <int F, int M, int NE>
__device__ inline void u_lane(double2 (&v)[NE], const double* u, int lane) {
  if constexpr (M >= 16) {
#pragma unroll
    for (int e = 0; e < NE; e += 2) {
      lane_swap<M>(v[e], v[e + 1]);
      u_pair<F>(v[e], v[e + 1], u);
      lane_swap<M>(v[e], v[e + 1]);
    }
  } else {
    const ExchangeCoef c = exchange_coef<F>(u, (lane & M) ? 1 : 0);
#pragma unroll
    for (int e = 0; e < NE; ++e)
      v[e] = u_exchange<F>(c, v[e], make_double2(lane_xor<M>(v[e].x), lane_xor<M>(v[e].y)));
  }
}

__device__ inline double flip_sign(double x, uint32_t bit31) {
  return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, x) ^ ((uint64_t)bit31 << 32));
}

// A one-qubit unitary on local bit ga; S is the workgroup's exchange buffer of
// 8 elements a thread.
template <int TB, int F>
__device__ __forceinline__ void reg_unitary(double2 (&v)[TileShape<TB>::NE], const double* u, int ga, int tid,
                                            int lane, double2* S) {
  constexpr int T = TileShape<TB>::T, LogT = TileShape<TB>::LogT, NE = TileShape<TB>::NE;
  if (ga >= LogT) {
    switch (ga - LogT) {
      case 0: u_reg<F, 0, NE>(v, u); break;
      case 1: u_reg<F, 1, NE>(v, u); break;
      case 2: u_reg<F, 2, NE>(v, u); break;
      default:
        if constexpr (NE > 8) u_reg<F, 3, NE>(v, u);
        break;
    }
  } else if (ga < 6) {
    switch (ga) {
      case 0: u_lane<F, 1, NE>(v, u, lane); break;
      case 1: u_lane<F, 2, NE>(v, u, lane); break;
      case 2: u_lane<F, 4, NE>(v, u, lane); break;
      case 3: u_lane<F, 8, NE>(v, u, lane); break;
      case 4: u_lane<F, 16, NE>(v, u, lane); break;
      default: u_lane<F, 32, NE>(v, u, lane); break;
    }
  } else {
    const ExchangeCoef c = exchange_coef<F>(u, (tid >> ga) & 1);
    const int m = 1 << ga;
#pragma unroll
    for (int h = 0; h < NE; h += 8) {
      __syncthreads();  // the previous exchange has read S
#pragma unroll
      for (int e = 0; e < 8; ++e) S[tid + e * T] = v[h + e];
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 8; ++e) v[h + e] = u_exchange<F>(c, v[h + e], S[(tid + e * T) ^ m]);
    }
  }
}

// The pass's gates on a thread's elements; S is the workgroup's exchange
// buffer of 8 elements a thread.
template <int TB>
__device__ __forceinline__ void reg_apply(double2 (&v)[TileShape<TB>::NE], const TileGroup& G, int tid, int lane,
                                          double2* S) {
  constexpr int T = TileShape<TB>::T, LogT = TileShape<TB>::LogT, NE = TileShape<TB>::NE;
  // bit e of bit_of(q): bit q of e
  auto bit_of = [](int q) -> uint32_t { return (uint32_t)(0xff00f0f0ccccaaaaull >> (16 * q)) & 0xffffu; };
  for (int gi = 0; gi < G.nops; ++gi) {
    const TileOp g = G.ops[gi];
    if (op_kind(g) == CQ_GATE_CZ) {
      // A run of CZs is diagonal: element tid + T e changes sign by the
      // parity, over the run's pairs, of the product of the pair's two bits;
      // bit e of `sg` collects it.
      uint32_t sg = 0;
      int j = gi;
      for (TileOp o = g; op_kind(o) == CQ_GATE_CZ;) {
        const int a = op_a(o), b = op_b(o);
        const uint32_t ma = a < LogT ? 0u - (((uint32_t)tid >> a) & 1u) : bit_of(a - LogT);
        const uint32_t mb = b < LogT ? 0u - (((uint32_t)tid >> b) & 1u) : bit_of(b - LogT);
        sg ^= ma & mb;
        if (++j == G.nops) break;
        o = G.ops[j];
      }
      gi = j - 1;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const uint32_t s = (sg << (31 - e)) & 0x80000000u;
        v[e] = make_double2(flip_sign(v[e].x, s), flip_sign(v[e].y, s));
      }
      continue;
    }
    if (op_form(g) == kNormal) reg_unitary<TB, kNormal>(v, G.u[op_u(g)], op_a(g), tid, lane, S);
    else reg_unitary<TB, kGeneral>(v, G.u[op_u(g)], op_a(g), tid, lane, S);
  }
}

template <int TB>
__global__ void __launch_bounds__(TileShape<TB>::T, TB == 12 ? 2 : 4) sv_reg_kernel(double2* psi, double* probs, TileGroup G) {
  constexpr int T = TileShape<TB>::T, LogT = TileShape<TB>::LogT, NE = TileShape<TB>::NE;
  __shared__ double2 S[T * 8];
  psi += blockIdx.y * G.bstride;
  const uint64_t start = start_string(G, blockIdx.y);
  uint64_t base = start & G.fixed;
  const uint64_t w = blockIdx.x;
  for (int i = 0; i < G.nouter; ++i) base |= ((w >> i) & 1ull) << G.outer[i];
  const int tid = threadIdx.x, lane = tid & 63;
  // local index tid + T e: its low bits are tid's (one per-thread part of the
  // address), the others e's (a part every thread shares), so no per-element
  // address has to stay live from the load to the store
  uint64_t tpart = base;
  for (int i = 0; i < LogT; ++i) tpart |= (uint64_t)((tid >> i) & 1) << G.bits[i];
  auto epart = [&](int e) -> uint64_t {
    uint64_t a = 0;
    for (int i = LogT; i < TB; ++i) a |= (uint64_t)((e >> (i - LogT)) & 1) << G.bits[i];
    return a;
  };
  // bits whose value decides whether an amplitude is stored before / after
  const uint64_t off0 = G.full & ~G.before, off1 = G.full & ~G.after;
  const bool zero = ((base ^ start) & off0 & ~G.tile) != 0;  // nothing of this tile is stored: all zero
  double2 v[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const uint64_t a = tpart | epart(e);
    v[e] = make_double2(0.0, 0.0);
    if (((a ^ start) & off0) == 0) {
      if (G.first) v[e].x = 1.0;
      else v[e] = psi[a];
    }
  }
  if (!zero) reg_apply<TB>(v, G, tid, lane, S);
  if (G.mode == 0) {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const uint64_t a = tpart | epart(e);
      if (((a ^ start) & off1) == 0) psi[a] = v[e];
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) probs[tpart | epart(e)] = G.weight * (v[e].x * v[e].x + v[e].y * v[e].y);
}

// Variants by linearity.  An init string prepares each init slot t in
// ket(d_t) = |0>, |1>, (|0> + |1>) / sqrt 2 or (|0> + i|1>) / sqrt 2, so its
// post-circuit state is a sum of the post-circuit states S_c of the 2^r
// computational init strings (slot t in |c_t>, c_t bit r - 1 - t of c), which
// sit bstride elements apart; and a measured slot's rotation combines the two
// halves of that slot's bit with weights that are powers of i over sqrt 2.
// Every variant is therefore |sum of amplitudes times powers of i|^2 over a
// power of 2.  A thread owns the 2^o outcomes around one setting of the other
// bits: it holds the 2^R x 2^O amplitudes of the last R <= 2 init and
// O <= 2 measured slots, forms each basis by additions in registers and writes
// that basis's 4^R init strings, so every S_c is read once and every variant
// written once (bound by that write).  Further slots are the grid's y: their
// digits (and outcome) choose which amplitudes are added on loading.
struct CombineArgs {
  int32_t w, r, o;
  int32_t vec;  // the last measured slot is index bit 0 and probs is 16-byte aligned
  int64_t bstride;
  double weight;  // of every |amplitude|^2
  uint32_t meas_bit[CQ_MAX_LOCAL_CUTS];  // index bit of measured slot u
};

__device__ inline double2 add_phase(double2 x, double2 y, int p) {  // x + i^p y
  switch (p & 3) {
    case 0: return make_double2(x.x + y.x, x.y + y.y);
    case 1: return make_double2(x.x - y.y, x.y + y.x);
    case 2: return make_double2(x.x - y.x, x.y - y.y);
    default: return make_double2(x.x + y.y, x.y - y.x);
  }
}

// The amplitude of init digit d from the two halves: |0>, |1>, + and +i
// (without the 1 / sqrt 2).
__device__ inline double2 init_amp(int d, double2 x0, double2 x1) {
  return d == 0 ? x0 : d == 1 ? x1 : add_phase(x0, x1, d - 2);
}

template <int R, int O>
__global__ void __launch_bounds__(kSvThreads) sv_combine_kernel(const double2* __restrict__ psi,
                                                                double* __restrict__ probs, CombineArgs A) {
  constexpr int NC = 1 << R, NM = 1 << O, NJ = 1 << (2 * R), NB = O == 0 ? 1 : (O == 1 ? 3 : 9);
  // the outer slots of this workgroup: offsets to the amplitudes and to the
  // outputs; every bit that takes both values doubles the amplitudes to add
  // (term q of them: offset off[q], times i^ph[q])
  constexpr int kMaxTerms = 1 << (CQ_MAX_LOCAL_CUTS - 2);
  __shared__ int64_t off[kMaxTerms];
  __shared__ int ph[kMaxTerms];
  const int ro = A.r - R, oo = A.o - O;
  int64_t dst = 0, jo = 0, bo = 0;
  int nt = 0;
  double outer_scale = A.weight;
  {
    unsigned y = blockIdx.y;
    const int q = threadIdx.x;
    int64_t src = 0, w4 = 1, w3 = 1;
    int p = 0;
    for (int s = ro - 1; s >= 0; --s) {
      const int d = y & 3;
      y >>= 2;
      const int64_t step = A.bstride << (A.r - 1 - s);
      if (d == 1) src += step;
      if (d >= 2) {
        if ((q >> nt) & 1) {
          src += step;
          p += d - 2;
        }
        ++nt;
        outer_scale *= 0.5;
      }
      jo += d * w4;
      w4 *= 4;
    }
    for (int u = oo - 1; u >= 0; --u) {
      const int m = y & 1;
      y >>= 1;
      const int d = (int)(y % 3);
      y /= 3;
      const int64_t step = (int64_t)1 << A.meas_bit[u];
      if (m) dst += step;
      if (d == 0) {
        if (m) src += step;
      } else {
        // X: x0 + (-1)^m x1; Y: x0 - i x1 (m = 0), x0 + i x1 (m = 1)
        if ((q >> nt) & 1) {
          src += step;
          p += d == 1 ? 2 * m : (m ? 1 : 3);
        }
        ++nt;
        outer_scale *= 0.5;
      }
      bo += d * w3;
      w3 *= 3;
    }
    if (q < 1 << nt) {
      off[q] = src;
      ph[q] = p;
    }
  }
  __syncthreads();
  const int64_t t = ((int64_t)blockIdx.z * gridDim.x + blockIdx.x) * kSvThreads + threadIdx.x;
  if (t >= (int64_t)1 << (A.w - A.o)) return;
  int64_t x0 = t;  // around the measured bits, which ascend from the last slot to the first
  for (int u = A.o - 1; u >= 0; --u)
    x0 = ((x0 >> A.meas_bit[u]) << (A.meas_bit[u] + 1)) | (x0 & (((int64_t)1 << A.meas_bit[u]) - 1));
  int64_t xm[NM];  // index bits of the inner outcomes
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    xm[m] = 0;
#pragma unroll
    for (int u = 0; u < O; ++u)
      if ((m >> (O - 1 - u)) & 1) xm[m] |= (int64_t)1 << A.meas_bit[oo + u];
  }
  double2 s[NC][NM];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int m = 0; m < NM; ++m) s[c][m] = psi[off[0] + c * A.bstride + (x0 | xm[m])];
  for (int q = 1; q < 1 << nt; ++q)
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int m = 0; m < NM; ++m) s[c][m] = add_phase(s[c][m], psi[off[q] + c * A.bstride + (x0 | xm[m])], ph[q]);
  int64_t nbasis = 1;
  for (int u = 0; u < A.o; ++u) nbasis *= 3;
  double* const out = probs + (dst | x0);
#pragma unroll 1
  for (int b = 0; b < NB; ++b) {
    double2 v[NC][NM];
    double scale = outer_scale;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int m = 0; m < NM; ++m) v[c][m] = s[c][m];
#pragma unroll
    for (int u = 0; u < O; ++u) {
      const int d = (O == 2 && u == 0) ? b / 3 : b % 3;
      if (d == 0) continue;
      scale *= 0.5;
      const int h = 1 << (O - 1 - u);
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          if (m & h) continue;
          const double2 y0 = v[c][m], y1 = v[c][m | h];
          v[c][m] = d == 1 ? add_phase(y0, y1, 0) : add_phase(y0, y1, 3);
          v[c][m | h] = d == 1 ? add_phase(y0, y1, 2) : add_phase(y0, y1, 1);
        }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      double p[NM];
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        double2 a;
        double sc = scale;
        if constexpr (R == 0) {
          a = v[0][m];
        } else if constexpr (R == 1) {
          a = init_amp(j, v[0][m], v[1][m]);
          if (j >= 2) sc *= 0.5;
        } else {
          const int d0 = j >> 2, d1 = j & 3;  // slot 0 is the state's high bit
          a = init_amp(d1, init_amp(d0, v[0][m], v[NC / 2][m]), init_amp(d0, v[NC / 4][m], v[NC - 1][m]));
          if (d0 >= 2) sc *= 0.5;
          if (d1 >= 2) sc *= 0.5;
        }
        p[m] = (a.x * a.x + a.y * a.y) * sc;
      }
      double* const row = out + ((((jo << (2 * R)) + j) * nbasis + bo * NB + b) << A.w);
      if (O >= 1 && A.vec) {
#pragma unroll
        for (int m = 0; m < NM; m += 2)
          if constexpr (NM >= 2) *reinterpret_cast<double2*>(row + xm[m]) = make_double2(p[m], p[m + 1]);
      } else {
#pragma unroll
        for (int m = 0; m < NM; ++m) row[xm[m]] = p[m];
      }
    }
  }
}

cq_status sv_hip_error(hipError_t e, const char* what) {
  return fail(CQ_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

cq_status check_gates(int32_t n, const cq_gate* gates, int32_t n_gates) {
  if (n_gates < 0) return fail(CQ_ERR_ARG, "negative gate count");
  if (n_gates > 0 && !gates) return fail(CQ_ERR_ARG, "null gate array");
  for (int i = 0; i < n_gates; ++i) {
    const cq_gate& g = gates[i];
    if (g.kind != CQ_GATE_U && g.kind != CQ_GATE_CZ) return fail(CQ_ERR_ARG, "unknown gate kind");
    if (g.q0 < 0 || g.q0 >= n) return fail(CQ_ERR_ARG, "gate qubit out of range");
    if (g.kind == CQ_GATE_CZ && (g.q1 < 0 || g.q1 >= n || g.q1 == g.q0))
      return fail(CQ_ERR_ARG, "CZ qubits out of range or equal");
    if (g.kind == CQ_GATE_U)
      for (double v : g.u)
        if (!std::isfinite(v)) return fail(CQ_ERR_ARG, "non-finite gate matrix");
  }
  return CQ_OK;
}

TileGroup tile_group(const GateSet& s, const PlanShape& sh, const Pass& pass, int mode) {
  TileGroup G{};
  const int n = s.n, k = std::min(n, sh.tile), low = std::min(n, sh.low);
  uint64_t mask = pass.mask | ((1ull << low) - 1);
  for (const uint64_t pool : {pass.after, ~(uint64_t)0})  // fill with touched bits first
    for (int b = 0; b < n && __builtin_popcountll(mask) < k; ++b) mask |= (pool >> b & 1) << b;
  G.k = k;
  G.mode = mode;
  G.before = pass.before;
  G.after = mode ? (1ull << n) - 1 : pass.after;
  G.full = (1ull << n) - 1;
  G.tile = mask;
  // local positions: ascending global bits for partial tiles; for full
  // tiles the lowest bits first (coalesced lanes), then the other bits by
  // one-qubit gate count, busiest first, on the register positions, then the
  // lane positions left, then the wave positions
  std::vector<int> order;
  for (int b = 0; b < n; ++b)
    if (mask >> b & 1) order.push_back(b);
  if (k >= kMinTileBits) {
    int uses[64] = {};
    for (int i : pass.gates)
      if (s.g[i].kind == CQ_GATE_U) ++uses[n - 1 - s.g[i].q0];
    std::vector<int> rest(order.begin() + low, order.end());
    std::stable_sort(rest.begin(), rest.end(), [&](int x, int y) { return uses[x] > uses[y]; });
    const int logt = TileShape<kMaxTileBits>::LogT;
    std::vector<int> slot;
    for (int i = logt; i < k; ++i) slot.push_back(i);
    for (int i = low; i < logt; ++i) slot.push_back(i);
    std::vector<int> placed(k, -1);
    for (int i = 0; i < low; ++i) placed[i] = order[i];
    for (int i = 0; i < (int)rest.size(); ++i) placed[slot[i]] = rest[i];
    order = placed;
  }
  int local[64];
  int no = 0;
  for (int i = 0; i < k; ++i) {
    local[order[i]] = i;
    G.bits[i] = (uint32_t)order[i];
  }
  for (int b = 0; b < n; ++b)
    if (!(mask >> b & 1)) {
      if (G.after >> b & 1) G.outer[no++] = (uint32_t)b;
      else G.fixed |= 1ull << b;
    }
  G.nouter = no;
  G.weight = (double)s.weight;
  G.nops = (int)pass.gates.size();
  int nu = 0;
  for (int j = 0; j < G.nops; ++j) {
    const cq_gate& g = s.g[pass.gates[j]];
    const uint32_t a = (uint32_t)g.kind | (uint32_t)local[n - 1 - g.q0] << 8;
    if (g.kind == CQ_GATE_CZ) {
      G.ops[j] = a | (uint32_t)local[n - 1 - g.q1] << 16;
    } else {
      G.ops[j] = a | (uint32_t)s.form[pass.gates[j]] << 6 | (uint32_t)nu << 24;
      for (int c = 0; c < 8; ++c) G.u[nu][c] = g.u[c];
      ++nu;
    }
  }
  return G;
}

// One tile pass: the register kernel for full tiles, the LDS kernel for
// registers narrower than a tile.
hipError_t launch_tiles(const TileGroup& G, double2* psi, double* probs, unsigned states, hipStream_t stream) {
  const dim3 grid((unsigned)(1ull << G.nouter), states);
  switch (G.k) {
    case 11: hipLaunchKernelGGL(sv_reg_kernel<11>, grid, dim3(TileShape<11>::T), 0, stream, psi, probs, G); break;
    case 12: hipLaunchKernelGGL(sv_reg_kernel<12>, grid, dim3(TileShape<12>::T), 0, stream, psi, probs, G); break;
    default: hipLaunchKernelGGL(sv_tile_kernel, grid, dim3(kSvThreads), 0, stream, psi, probs, G); break;
  }
  return hipGetLastError();
}

// Applies the (normalised) gates in the planned passes to a batch of states, one
// for each string of init_bits, that start as basis strings (see TileGroup).
// With probs (one state) the last pass writes weight * |amplitude|^2 there; else
// it leaves every amplitude in psi, and the weight to whoever squares them.
hipError_t run_gates(const GateSet& s, const PlanShape& sh, const std::vector<Pass>& passes, double2* psi,
                     double* probs, const std::vector<int>& init_bits, hipStream_t stream) {
  for (size_t i = 0; i < passes.size(); ++i) {
    const bool last = i + 1 == passes.size();
    TileGroup G = tile_group(s, sh, passes[i], last && probs ? 1 : 0);
    G.bstride = (int64_t)1 << s.n;
    G.first = i == 0;
    G.r = (int32_t)init_bits.size();
    for (int t = 0; t < G.r; ++t) G.init_bit[t] = (uint32_t)init_bits[t];
    const hipError_t e = launch_tiles(G, psi, probs, 1u << G.r, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int R, int O>
void launch_combine(const CombineArgs& A, const double2* psi, double* probs, hipStream_t stream) {
  const int64_t nx = (((int64_t)1 << (A.w - A.o)) + kSvThreads - 1) / kSvThreads;
  unsigned ny = 1u << (2 * (A.r - R));
  for (int u = 0; u < A.o - O; ++u) ny *= 6;
  // x and z number the columns: a dimension holds fewer than 2^32 threads
  const unsigned nz = nx > 1 << 23 ? (unsigned)(nx >> 23) : 1u;
  hipLaunchKernelGGL((sv_combine_kernel<R, O>), dim3((unsigned)(nx / nz), ny, nz), dim3(kSvThreads), 0, stream, psi,
                     probs, A);
}

// r: the init slots whose 2^r computational strings psi holds, the last of `si`
hipError_t combine(const SubInfo& si, int r, const double2* psi, double* probs, double weight, hipStream_t stream) {
  CombineArgs A{};
  A.weight = weight;
  A.w = si.width;
  A.r = r;
  A.o = si.o();
  A.bstride = (int64_t)1 << si.width;
  for (int u = 0; u < A.o; ++u) A.meas_bit[u] = (uint32_t)(si.width - 1 - si.meas_slots[u]);
  A.vec = A.o > 0 && A.meas_bit[A.o - 1] == 0 && (reinterpret_cast<uintptr_t>(probs) & 15) == 0;
  switch (std::min(A.r, 2) * 3 + std::min(A.o, 2)) {
    case 0: launch_combine<0, 0>(A, psi, probs, stream); break;
    case 1: launch_combine<0, 1>(A, psi, probs, stream); break;
    case 2: launch_combine<0, 2>(A, psi, probs, stream); break;
    case 3: launch_combine<1, 0>(A, psi, probs, stream); break;
    case 4: launch_combine<1, 1>(A, psi, probs, stream); break;
    case 5: launch_combine<1, 2>(A, psi, probs, stream); break;
    case 6: launch_combine<2, 0>(A, psi, probs, stream); break;
    case 7: launch_combine<2, 1>(A, psi, probs, stream); break;
    default: launch_combine<2, 2>(A, psi, probs, stream); break;
  }
  return hipGetLastError();
}

// What cq_variants_workspace_size asks for together with the variants at most:
// beyond it (of the card's 288 GB) fewer states are batched.
constexpr size_t kVariantBytes = (size_t)240 << 30;

}  // namespace

}  // namespace cq

using namespace cq;

extern "C" cq_status cq_simulate_workspace_size(int32_t n, size_t* bytes) {
  if (!bytes) return fail(CQ_ERR_ARG, "null argument");
  if (n < 1 || n > CQ_MAX_SV_QUBITS) return fail(CQ_ERR_SHAPE, "qubit count out of range");
  *bytes = (size_t)16 << n;
  return CQ_OK;
}

extern "C" cq_status cq_simulate_probabilities(int32_t n, const cq_gate* gates, int32_t n_gates, double* probs,
                                               void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (!probs) return fail(CQ_ERR_ARG, "null argument");
  if (n < 1 || n > CQ_MAX_SV_QUBITS) return fail(CQ_ERR_SHAPE, "qubit count out of range");
  cq_status st = check_gates(n, gates, n_gates);
  if (st != CQ_OK) return st;
  if (!workspace || workspace_bytes < ((size_t)16 << n)) return fail(CQ_ERR_WORKSPACE, "workspace too small");
  GateSet circuit = gate_set(n, gates, n_gates, 0);
  normalize(circuit, true);
  std::vector<Pass> passes;
  const PlanShape shape = best_plan(circuit, 1, passes);
  const hipError_t e = run_gates(circuit, shape, passes, static_cast<double2*>(workspace), probs, {}, stream);
  if (e != hipSuccess) return sv_hip_error(e, "state-vector launch");
  return CQ_OK;
}

extern "C" cq_status cq_variants_workspace_size(const cq_subcircuit* sub, size_t* bytes) {
  if (!bytes) return fail(CQ_ERR_ARG, "null argument");
  SubInfo si;
  cq_status st = build_subinfo(sub, si);
  if (st != CQ_OK) return st;
  if (si.width < 1) return fail(CQ_ERR_SHAPE, "subcircuit has no slots");
  size_t variants = ((size_t)8 << si.width) << (2 * si.r());
  for (int u = 0; u < si.o(); ++u) variants *= 3;
  int r = si.r();
  while (r > 0 && variants + (((size_t)16 << si.width) << r) > kVariantBytes) --r;
  *bytes = ((size_t)16 << si.width) << r;
  return CQ_OK;
}

extern "C" cq_status cq_variant_probabilities(const cq_subcircuit* sub, const cq_gate* gates, int32_t n_gates,
                                              double* variants, void* workspace, size_t workspace_bytes,
                                              hipStream_t stream) {
  if (!variants) return fail(CQ_ERR_ARG, "null argument");
  SubInfo si;
  cq_status st = build_subinfo(sub, si);
  if (st != CQ_OK) return st;
  const int w = si.width;
  if (w < 1) return fail(CQ_ERR_SHAPE, "subcircuit has no slots");
  st = check_gates(w, gates, n_gates);
  if (st != CQ_OK) return st;
  if (!workspace || workspace_bytes < ((size_t)16 << w)) return fail(CQ_ERR_WORKSPACE, "workspace too small");
  double2* psi = static_cast<double2*>(workspace);
  const int r = si.r(), o = si.o();
  uint64_t rotated = 0;
  for (int q : si.meas_slots) rotated |= 1ull << (w - 1 - q);
  // As many of the last init slots as the workspace holds strings for go as one
  // batch of computational strings, from which one pass writes every variant of
  // theirs; the slots before them are prepared by a unitary each, one string of
  // digits after another (none with a workspace of 2^r states).
  int inner = r;
  while (((size_t)16 << w) << inner > workspace_bytes) --inner;
  const int outer = r - inner;
  std::vector<int> init_bits;
  for (int t = outer; t < r; ++t) init_bits.push_back(w - 1 - si.init_slots[t]);
  const double h = 1.0 / std::sqrt(2.0);
  const double prepare[4][8] = {{1, 0, 0, 0, 0, 0, 1, 0},    // |0>
                                {0, 0, 1, 0, 1, 0, 0, 0},    // |1>
                                {h, 0, h, 0, h, 0, -h, 0},   // |+>
                                {h, 0, h, 0, 0, h, 0, -h}};  // |+i>
  std::vector<cq_gate> all((size_t)outer + n_gates);
  std::copy(gates, gates + n_gates, all.begin() + outer);
  int64_t stride = (int64_t)1 << (w + 2 * inner);  // variants of a string
  for (int u = 0; u < o; ++u) stride *= 3;
  std::vector<Pass> passes;
  PlanShape shape;
  for (int64_t j = 0; j < (int64_t)1 << (2 * outer); ++j) {
    for (int t = 0; t < outer; ++t) {
      all[t].kind = CQ_GATE_U;
      all[t].q0 = si.init_slots[t];
      for (int c = 0; c < 8; ++c) all[t].u[c] = prepare[(j >> (2 * (outer - 1 - t))) & 3][c];
    }
    GateSet circuit = gate_set(w, all.data(), (int)all.size(), rotated);
    normalize(circuit, false);
    if (j == 0) shape = best_plan(circuit, 1 << inner, passes);
    hipError_t e = run_gates(circuit, shape, passes, psi, nullptr, init_bits, stream);
    if (e == hipSuccess)
      e = combine(si, inner, psi, variants + j * stride, (double)circuit.weight, stream);
    if (e != hipSuccess) return sv_hip_error(e, "variant launch");
  }
  return CQ_OK;
}
