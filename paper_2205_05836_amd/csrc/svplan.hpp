// The host side of the state-vector simulation: which gates matter, the form
// each one-qubit unitary is applied in, and the passes.  No device code.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "cutqc.h"

namespace cq {

constexpr int kMinTileBits = 11;  // narrower registers take the LDS kernel
constexpr int kMaxTileBits = 12;
constexpr int kMaxOps = 160;  // gates of a pass
constexpr int kMaxU = 36;     // one-qubit unitaries among them

// Forms of a one-qubit unitary (normalize).
enum Form { kGeneral = 0, kNormal = 1 };

// One pass of a plan: its gates (indices into the gate list, circuit order),
// the qubits they act on as index bits, and the bits touched before and
// after it.
struct Pass {
  std::vector<int> gates;
  uint64_t mask = 0, before = 0, after = 0;
};

struct GateSet {
  int n = 0;
  std::vector<cq_gate> g;
  std::vector<uint64_t> mask;
  std::vector<int> form;  // Form of each one-qubit unitary
  long double weight = 1.0L;  // |factor|^2 that the final amplitudes lack
};

inline uint64_t gate_mask(int n, const cq_gate& g) {
  return (1ull << (n - 1 - g.q0)) | (g.kind == CQ_GATE_CZ ? 1ull << (n - 1 - g.q1) : 0ull);
}

// The gates that matter to probabilities: a CZ none of whose qubits sees a
// later one-qubit gate (of the list, or of the rotations on `rotated`, index
// bits) commutes to the end, where it only changes phases.
inline GateSet gate_set(int n, const cq_gate* gates, int n_gates, uint64_t rotated) {
  GateSet s;
  s.n = n;
  uint64_t live = rotated;
  std::vector<int> keep;
  for (int i = n_gates - 1; i >= 0; --i) {
    const uint64_t m = gate_mask(n, gates[i]);
    if (gates[i].kind == CQ_GATE_U) live |= m;
    else if ((m & live) == 0) continue;
    keep.push_back(i);
  }
  for (auto it = keep.rbegin(); it != keep.rend(); ++it) {
    s.g.push_back(gates[*it]);
    s.mask.push_back(gate_mask(n, gates[*it]));
  }
  return s;
}

// Rewrites the unitaries so that most cost four FMA an amplitude instead of
// eight: U = diag(d0, d1) [1, a; b, 1].  The diagonal commutes with the CZs
// behind the gate and is multiplied into the columns of the next unitary on
// its qubit.  A qubit's last unitary stays general, or, where only
// probabilities are asked for (`probs`) and |d0| = |d1| to rounding (as for
// every unitary matrix), leaves |d0|^2 to the final weight.  What is stored
// meanwhile is the true amplitude over the factors held back: those are kept
// within 2^-12 .. 2^12 a qubit (2^408 over 34 qubits) by a general gate, which
// also takes what has no such form or a diagonal below a 16th of the entries
// beside it.
//
// Error: the ratios are rounded, where a general gate has its entries as
// given, but an amplitude is rounded twice instead of four times.  What a
// row's rounding takes from its norm and phase is made good: the diagonal is
// the one that fits the row best with the rounded ratio, the entries of a
// general gate behind it pass on their norm, and the weight collects the
// factors in long double.  (Brickwork of Haar unitaries on 16 qubits, 8 layers
// deep, relative l2 error of the probabilities against long double: 6.4e-16,
// with general gates 6.5e-16; the sum of all probabilities 1.3e-16 off, 1.2e-16
// with general gates.  With the diagonal taken as it stands and the weight in
// double 12 layers had 10e-16 against 8.6e-16, and the sum was 5e-16 off.)  The
// rounded ratios cost a qubit's first and last gates more than the fewer
// roundings gain: 4 layers have 4.9e-16 against 4.6e-16, 6 5.5e-16 against
// 5.4e-16, 10 7.2e-16 against 7.4e-16, so qubits with fewer than kNormalGates
// unitaries keep them general.
constexpr int kNormalGates = 8;

inline void normalize(GateSet& s, bool probs) {
  typedef long double real;
  struct cx {
    real re, im;
  };
  const auto mul = [](cx x, cx y) { return cx{x.re * y.re - x.im * y.im, x.re * y.im + x.im * y.re}; };
  const auto mulc = [](cx x, cx y) { return cx{x.re * y.re + x.im * y.im, x.im * y.re - x.re * y.im}; };  // x conj(y)
  const auto norm = [](cx x) { return x.re * x.re + x.im * x.im; };
  std::vector<cx> d0(s.n, cx{1, 0}), d1(s.n, cx{1, 0});
  std::vector<int> last(s.n, -1), count(s.n, 0);
  for (size_t i = 0; i < s.g.size(); ++i)
    if (s.g[i].kind == CQ_GATE_U) {
      last[s.g[i].q0] = (int)i;
      ++count[s.g[i].q0];
    }
  s.form.assign(s.g.size(), kGeneral);
  if (s.n < kMinTileBits) return;
  const auto fits = [](real pivot, real other) {  // squared magnitudes; false for NaN
    return pivot >= (real)1 / (1 << 24) && pivot <= (real)(1 << 24) && other <= 256 * pivot;
  };
  for (size_t i = 0; i < s.g.size(); ++i) {
    cq_gate& g = s.g[i];
    const int q = g.q0;
    if (g.kind != CQ_GATE_U || count[q] < kNormalGates) continue;
    cx u[4];
    for (int c = 0; c < 4; ++c) u[c] = mul(cx{g.u[2 * c], g.u[2 * c + 1]}, (c & 1) ? d1[q] : d0[q]);
    d0[q] = d1[q] = cx{1, 0};
    const bool end = (int)i == last[q];
    bool normal = (probs || !end) && fits(norm(u[0]), norm(u[1])) && fits(norm(u[3]), norm(u[2]));
    if (normal) {
      // the ratios as the kernel has them, then the diagonal that fits the rows
      // (divisions are slow: one for both of each)
      const real m0 = norm(u[0]), m1 = norm(u[3]), inv = 1 / (m0 * m1);
      const cx x = mulc(u[1], u[0]), y = mulc(u[2], u[3]);
      const cx a{(double)(x.re * (m1 * inv)), (double)(x.im * (m1 * inv))};
      const cx b{(double)(y.re * (m0 * inv)), (double)(y.im * (m0 * inv))};
      const real na = 1 + norm(a), nb = 1 + norm(b), fit = 1 / (na * nb);
      const cx ta = mulc(u[1], a), tb = mulc(u[2], b);
      const cx p0{(u[0].re + ta.re) * (nb * fit), (u[0].im + ta.im) * (nb * fit)};
      const cx p1{(u[3].re + tb.re) * (na * fit), (u[3].im + tb.im) * (na * fit)};
      const real n0 = norm(p0), n1 = norm(p1);
      if (end) normal = std::abs(n0 - n1) <= 2e-16L * n0;
      if (normal) {
        s.form[i] = kNormal;
        if (end) s.weight *= (n0 + n1) / 2;
        d0[q] = p0;
        d1[q] = p1;
        u[0] = a;
        u[1] = b;
      }
    }
    if (normal) {
      g.u[0] = (double)u[0].re;
      g.u[1] = (double)u[0].im;
      g.u[2] = (double)u[1].re;
      g.u[3] = (double)u[1].im;
      continue;
    }
    real given = 0, rounded = 0;
    for (int c = 0; c < 4; ++c) {
      g.u[2 * c] = (double)u[c].re;
      g.u[2 * c + 1] = (double)u[c].im;
      given += norm(u[c]);
      rounded += norm(cx{g.u[2 * c], g.u[2 * c + 1]});
    }
    if (given != rounded && rounded > given / 2 && rounded < given * 2) {  // not if out of range
      const real lost = given / rounded;
      if (end) s.weight *= lost;
      else d0[q] = d1[q] = cx{std::sqrt(lost), 0};
    }
  }
}

// How a plan is laid out: tile bits, the lowest index bits every tile holds
// (gathers then read runs of 2^low amplitudes), and how many qubits join the
// allowed set when no gate inside it can run.
struct PlanShape {
  int tile = 0, low = 0, grow = 0;
};

// Passes for one shape.  A pass takes, in circuit order, every gate inside the
// allowed qubits that fits the tile and shares no qubit with an earlier gate
// left for a later pass.  The state starts as a basis string, and the allowed
// qubits start as the lowest `tile` index bits and grow, lowest first, only when
// none of their gates can run: while t qubits are touched a pass moves 2^t
// amplitudes.  The last pass writes every amplitude, also without gates.
// Returns the modelled time in microseconds, or anything above `limit` once
// that is passed.  The model, from traces: 3.5 us a launch, the bytes at the
// rate of a large copy (4.4 TB/s), and 0.33 ms for every one-qubit gate on 2^30
// amplitudes, no less than the serial time of those gates in one tile (0.8 us
// each with 11 bits, 1.4 us with 12).
//
// The order leaves the amplitudes as exact as circuit order does, but spreads
// their errors differently: what a gate rounds while few qubits are touched is
// passed on in proportion to the amplitudes that grow from it, so the large
// probabilities carry more of it.  (20 qubits, 8 layers, general gates, against
// long double: relative l2 error of the amplitudes 9.2e-16 in circuit order and
// 9.1e-16 in this one, sum of |dp| 8.5e-16 and 9.3e-16, 8.6e-16 with the
// rewritten unitaries; l2 error of the probabilities, which weighs the large
// ones, 6.3e-16 and 8.3e-16, 7.8e-16 with the rewritten ones.)
inline double plan_passes(const GateSet& s, const PlanShape& sh, int states, double limit,
                   std::vector<Pass>& out) {
  const int n = s.n;
  const uint64_t full = (1ull << n) - 1;
  const uint64_t low = (1ull << std::min(n, sh.low)) - 1;
  uint64_t allowed = (1ull << std::min(n, sh.tile)) - 1, touched = 0;
  std::vector<int> rest(s.g.size()), left;
  for (size_t i = 0; i < rest.size(); ++i) rest[i] = (int)i;
  out.clear();
  double us = 0.0;
  while (!rest.empty()) {
    Pass p;
    uint64_t blocked = 0, cur = low;
    int nu = 0;
    left.clear();
    for (size_t q = 0; q < rest.size(); ++q) {
      const int i = rest[q];
      const uint64_t m = s.mask[i];
      const int is_u = s.g[i].kind == CQ_GATE_U;
      if ((m & (blocked | ~allowed)) == 0 && (int)p.gates.size() < kMaxOps && nu + is_u <= kMaxU &&
          __builtin_popcountll(cur | m) <= sh.tile) {
        p.gates.push_back(i);
        p.mask |= m;
        cur |= m;
        nu += is_u;
      } else {
        blocked |= m;
        left.push_back(i);
        if ((allowed & ~blocked) == 0) {  // nothing after it can run
          left.insert(left.end(), rest.begin() + q + 1, rest.end());
          break;
        }
      }
    }
    if (p.gates.empty()) {
      for (int a = 0; a < sh.grow && allowed != full; ++a) allowed |= allowed + 1;  // the lowest bit not allowed yet
      continue;
    }
    p.before = touched;
    touched |= p.mask;
    p.after = touched;
    rest.swap(left);
    const double before = out.empty() ? 0.0 : std::ldexp(16.0, __builtin_popcountll(p.before));
    const double after = std::ldexp(rest.empty() ? 8.0 : 16.0, rest.empty() ? n : __builtin_popcountll(p.after));
    const double work = nu * std::max(std::ldexp(3.1e-7 * states, __builtin_popcountll(p.after)),
                                      sh.tile <= 11 ? 0.8 : 1.4);
    us += 3.5 + states * (before + after) / 4.4e6 + work;
    out.push_back(std::move(p));
    if (us > limit) break;
  }
  return us;
}

// Shapes in the order in which trying them pays (tile bits, growth; 0: every
// qubit at once), for registers of 18 to 24 qubits and for wider ones, by the
// model over line and random-pair circuits of 18 to 28 qubits and 3 to 12
// layers.  Runs of 8 amplitudes (128 bytes, one line) leave a tile one bit more
// than runs of 16; a tile's spare bits go to the lowest anyway.
constexpr int kShapes = 12;
constexpr int8_t kNarrow[kShapes][2] = {{11, 4}, {11, 6}, {11, 2}, {11, 3}, {11, 0}, {11, 1},
                                        {12, 2}, {12, 4}, {12, 1}, {12, 3}, {12, 6}, {12, 0}};
constexpr int8_t kWide[kShapes][2] = {{12, 2}, {12, 1}, {12, 4}, {11, 4}, {12, 3}, {12, 0},
                                      {11, 3}, {11, 1}, {11, 2}, {11, 0}, {12, 6}, {11, 6}};

// The cheapest plan by the model.  Wider tiles mean fewer passes; growing the
// allowed set by several qubits at a time merges passes that one at a time
// would leave nearly empty.  Laying out a shape costs the host some 0.02 us a
// gate, so shapes are tried only while that stays below a 16th of the best
// plan's modelled time: three for 18 qubits and 8 layers (135 us), which the
// model puts within 1.5% of the best of all up to 21 qubits and within 3% to 24,
// and all of them from there.  (24 shapes whatever the size took 124 us at 18
// qubits.)  Below 18 qubits launches decide: every qubit at once, either tile.
inline PlanShape best_plan(const GateSet& s, int states, std::vector<Pass>& out) {
  PlanShape best;
  double least = 1e300;
  std::vector<Pass> cand;
  int tried = 0;
  for (int q = 0; q < kShapes; ++q) {
    const int8_t* const t = s.n <= 24 ? kNarrow[q] : kWide[q];
    if (s.n < 18 && t[1] != 0) continue;
    if (t[0] > std::max(s.n, kMinTileBits)) continue;
    if (tried && tried * 0.02 * (double)s.g.size() > least / 16) break;
    const PlanShape sh{std::min(s.n, (int)t[0]), 3, t[1] ? t[1] : s.n};
    const double us = plan_passes(s, sh, states, least, cand);
    ++tried;
    if (us < least) {
      least = us;
      best = sh;
      out.swap(cand);
    }
  }
  if (out.empty()) out.push_back(Pass());
  out.back().after = (1ull << s.n) - 1;
  return best;
}

}  // namespace cq
