// Replays the state-vector kernel's arithmetic (svplan.hpp's forms, FMA by FMA)
// on random brickwork circuits, with the unitaries as the library rewrites them
// and with all of them general, and prints both errors against long double:
//   replay <qubits> <layers> <circuits> <probs 0|1>
// The relative l2 error of the probabilities and the error of their sum, rms
// over the circuits: general l2, rewritten l2, general sum, rewritten sum.
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "svplan.hpp"

using namespace cq;

namespace {

std::vector<cq_gate> brickwork(int n, int layers, std::mt19937_64& rng) {
  std::normal_distribution<double> normal;
  std::vector<cq_gate> gates;
  for (int t = 0; t < layers; ++t) {
    for (int q = 0; q < n; ++q) {
      double z[4], s = 0.0;
      for (double& x : z) s += (x = normal(rng)) * x;
      for (double& x : z) x /= std::sqrt(s);
      const std::complex<double> a(z[0], z[1]), b(z[2], z[3]), e = std::polar(1.0, 3.0 * normal(rng));
      const std::complex<double> u[4] = {a * e, -std::conj(b) * e, b, std::conj(a)};
      cq_gate g{};
      g.kind = CQ_GATE_U;
      g.q0 = q;
      for (int c = 0; c < 4; ++c) {
        g.u[2 * c] = u[c].real();
        g.u[2 * c + 1] = u[c].imag();
      }
      gates.push_back(g);
    }
    for (int q = t % 2; q + 1 < n; q += 2) {
      cq_gate g{};
      g.kind = CQ_GATE_CZ;
      g.q0 = q;
      g.q1 = q + 1;
      gates.push_back(g);
    }
  }
  return gates;
}

// Calls f(x, y) for every pair of a unitary, or flips the signs of a CZ.
template <typename Amp, typename F>
void apply(int n, const cq_gate& g, std::vector<Amp>& v, F f) {
  const size_t m = (size_t)1 << (n - 1 - g.q0);
  const size_t both = g.kind == CQ_GATE_CZ ? m | (size_t)1 << (n - 1 - g.q1) : 0;
  for (size_t x = 0; x < v.size(); ++x) {
    if (both) {
      if ((x & both) == both) v[x] = -v[x];
    } else if (!(x & m)) {
      f(v[x], v[x | m]);
    }
  }
}

typedef std::complex<double> cd;

cd row(const double* u, cd x, cd y) {
  return cd(std::fma(-u[3], y.imag(), std::fma(u[2], y.real(), std::fma(-u[1], x.imag(), u[0] * x.real()))),
            std::fma(u[3], y.real(), std::fma(u[2], y.imag(), std::fma(u[1], x.real(), u[0] * x.imag()))));
}

cd add(cd x, const double* r, cd y) {
  return cd(std::fma(-r[1], y.imag(), std::fma(r[0], y.real(), x.real())),
            std::fma(r[1], y.real(), std::fma(r[0], y.imag(), x.imag())));
}

std::vector<double> replay(const GateSet& s) {
  std::vector<cd> v((size_t)1 << s.n);
  v[0] = 1.0;
  for (size_t i = 0; i < s.g.size(); ++i) {
    const double* u = s.g[i].u;
    if (s.form[i] == kNormal)
      apply(s.n, s.g[i], v, [&](cd& x, cd& y) {
        const cd a = x;
        x = add(a, u, y);
        y = add(y, u + 2, a);
      });
    else
      apply(s.n, s.g[i], v, [&](cd& x, cd& y) {
        const cd a = x;
        x = row(u, a, y);
        y = row(u + 4, a, y);
      });
  }
  std::vector<double> p;
  for (const cd& z : v) p.push_back((double)s.weight * std::fma(z.imag(), z.imag(), z.real() * z.real()));
  return p;
}

std::vector<long double> exact(const GateSet& s) {
  typedef std::complex<long double> cl;
  std::vector<cl> v((size_t)1 << s.n);
  v[0] = 1.0L;
  for (const cq_gate& g : s.g) {
    cl u[4];
    for (int c = 0; c < 4; ++c) u[c] = cl(g.u[2 * c], g.u[2 * c + 1]);
    apply(s.n, g, v, [&](cl& x, cl& y) {
      const cl a = x;
      x = u[0] * a + u[1] * y;
      y = u[2] * a + u[3] * y;
    });
  }
  std::vector<long double> p;
  for (const cl& z : v) p.push_back(std::norm(z));
  return p;
}

void errors(const std::vector<double>& p, const std::vector<long double>& e, long double* l2, long double* sum) {
  long double d = 0, n = 0, s = 0;
  for (size_t x = 0; x < p.size(); ++x) {
    d += (p[x] - e[x]) * (p[x] - e[x]);
    n += e[x] * e[x];
    s += p[x] - e[x];
  }
  *l2 += d / n;
  *sum += s * s;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 5) return 2;
  const int n = std::atoi(argv[1]), layers = std::atoi(argv[2]), circuits = std::atoi(argv[3]);
  long double l2[2] = {0, 0}, sum[2] = {0, 0};
  for (int c = 0; c < circuits; ++c) {
    std::mt19937_64 rng(1000 * n + c);
    const std::vector<cq_gate> gates = brickwork(n, layers, rng);
    GateSet general = gate_set(n, gates.data(), (int)gates.size(), 0), rewritten = general;
    general.form.assign(general.g.size(), kGeneral);
    normalize(rewritten, std::atoi(argv[4]) != 0);
    const std::vector<long double> e = exact(general);
    errors(replay(general), e, &l2[0], &sum[0]);
    errors(replay(rewritten), e, &l2[1], &sum[1]);
  }
  std::printf("%.6Lg %.6Lg %.6Lg %.6Lg\n", std::sqrt(l2[0] / circuits), std::sqrt(l2[1] / circuits),
              std::sqrt(sum[0] / circuits), std::sqrt(sum[1] / circuits));
  return 0;
}
