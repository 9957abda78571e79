// The arithmetic of lbg_sym.hpp on the host, for tests/test_symmetry_cpu.py.
#include <cmath>
#include <random>

#include "lbg_sym.hpp"

using namespace lbg;

// The products of the arcs at the points p.
static SymProducts products(const uint32_t* u, const uint32_t* v, int64_t count, const double (&p)[kSymPoints]) {
  SymProducts s;
  sym_start(s);
  bool swapped = false;
  for (int64_t k = 0; k < count; ++k) {
    const bool side = u[k] > v[k];
    sym_take(s, side != swapped, side ? v[k] : u[k], side ? u[k] : v[k], p);
    swapped = side;
  }
  sym_finish(s, swapped);
  return s;
}

extern "C" {

double sc_mul(double a, double b) { return sym_mul(a, b); }
double sc_small(double a) { return sym_small(a); }

// The products (up, down of each point, as residues) of `count` arcs at the points x[0 .. 1].
void sc_products(const uint32_t* u, const uint32_t* v, int64_t count, const uint64_t* x, uint64_t* out) {
  double p[kSymPoints];
  for (int i = 0; i < kSymPoints; ++i) p[i] = static_cast<double>((1ull << 52) + x[i]);
  const SymProducts s = products(u, v, count, p);
  const int64_t m = static_cast<int64_t>(kSymP);
  for (int i = 0; i < kSymPoints; ++i) {
    out[2 * i] = static_cast<uint64_t>((static_cast<int64_t>(s.up[i]) % m + m) % m);
    out[2 * i + 1] = static_cast<uint64_t>((static_cast<int64_t>(s.down[i]) % m + m) % m);
  }
}

// Of `draws` draws, how often the arcs pass at one point alone, and at all of them.
void sc_passes(const uint32_t* u, const uint32_t* v, int64_t count, int64_t draws, uint64_t seed, int64_t* out) {
  std::mt19937_64 rng(seed);
  out[0] = out[1] = 0;
  for (int64_t d = 0; d < draws; ++d) {
    double p[kSymPoints];
    for (double& x : p) x = static_cast<double>((1ull << 52) + (rng() >> 13) % kSymP);
    const SymProducts s = products(u, v, count, p);
    int same = 0;
    for (int i = 0; i < kSymPoints; ++i) same += sym_equal(s.up[i], s.down[i]);
    out[0] += same > 0;
    out[1] += same == kSymPoints;
  }
}
}
