// The passes of random brickwork circuits (plan <qubits> <layers>): checks that
// every gate is in one pass, fits its tile and keeps its place among the gates
// it shares a qubit with, then prints the least host time of 20 plannings
// (gate selection, forms and passes) and the modelled device time of the
// passes, both in microseconds.
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "svplan.hpp"

using namespace cq;

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  const int n = std::atoi(argv[1]), layers = std::atoi(argv[2]);
  std::mt19937_64 rng(n);
  std::uniform_real_distribution<double> angle(0.0, 6.283185307179586);
  std::vector<cq_gate> gates;
  for (int t = 0; t < layers; ++t) {
    for (int q = 0; q < n; ++q) {
      const double c = std::cos(angle(rng)), s = std::sqrt(1 - c * c), f = angle(rng), l = angle(rng);
      gates.push_back(cq_gate{CQ_GATE_U, q, 0, {c, 0, -s * std::cos(l), -s * std::sin(l), s * std::cos(f),
                                                s * std::sin(f), c * std::cos(f + l), c * std::sin(f + l)}});
    }
    for (int q = t % 2; q + 1 < n; q += 2) gates.push_back(cq_gate{CQ_GATE_CZ, q, q + 1, {}});
  }
  double least = 1e300, model = 0.0;
  for (int rep = 0; rep < 20; ++rep) {
    const auto t0 = std::chrono::steady_clock::now();
    GateSet s = gate_set(n, gates.data(), (int)gates.size(), 0);
    normalize(s, true);
    std::vector<Pass> passes;
    const PlanShape shape = best_plan(s, 1, passes);
    const std::chrono::duration<double, std::micro> d = std::chrono::steady_clock::now() - t0;
    least = std::min(least, d.count());
    if (rep) continue;
    std::vector<int> seen(s.g.size(), 0), at(n, -1);
    uint64_t touched = 0;
    for (const Pass& p : passes) {
      uint64_t mask = (1ull << std::min(n, shape.low)) - 1;
      int unitaries = 0;
      if (p.before != touched) return 3;
      for (int i : p.gates) {
        ++seen[i];
        mask |= s.mask[i];
        touched |= s.mask[i];
        unitaries += s.g[i].kind == CQ_GATE_U;
        for (int b = 0; b < n; ++b)
          if (s.mask[i] >> b & 1) {
            if (at[b] > i) return 4;
            at[b] = i;
          }
      }
      const bool last = &p == &passes.back();
      if (p.after != (last ? (1ull << n) - 1 : touched) || __builtin_popcountll(mask) > shape.tile) return 5;
      if ((int)p.gates.size() > kMaxOps || unitaries > kMaxU) return 6;
    }
    for (int c : seen)
      if (c != 1) return 7;
    std::vector<Pass> again;
    model = plan_passes(s, shape, 1, 1e300, again);
  }
  std::printf("%.1f %.1f\n", least, model);
  return 0;
}
