// Whether a graph is symmetric, by one pass over its arcs.
//
// A graph is symmetric when the pairs {u, v} of its arcs u -> v with u < v
// are, as a multiset, those of its arcs with u > v (self-loops are their own
// reverse).  Two multisets of numbers e in a field are equal exactly when the
// polynomials prod (x - e) are, and two different ones of degree at most m
// agree at no more than m points of the field: so both products are formed at
// a point x drawn at random, in the field of p = 2^51 - 129 elements, for
// e = 2^25 min(u, v) + max(u, v), which tells all pairs of a graph of at most
// 2^25 nodes apart.  A symmetric graph always passes.  Any other one, however
// its one-way arcs are arranged, passes with a chance of at most m / p over
// the draw, and the three points that are used are drawn independently: at
// most (m / p)^3, below 2^-60 for every m < 2^31 (2^-72 for the 2^27 arcs of
// R-MAT scale 22).  (Equality of multisets by products at a random point:
// Lipton 1989; Blum et al., Checking the correctness of memories, 1991.)
//
// The products are formed in double precision, where a multiply-add of 53
// bits is as fast as one of 24 and four times as fast as a 32-bit integer
// multiply: sym_mul is exact.  Plain C++, so that tests can run it on the host.
#pragma once

#include <stdint.h>

#ifndef __device__
#define __device__
#define __forceinline__ inline
#endif

namespace lbg {

constexpr unsigned long long kSymP = (1ull << 51) - 129;  // a prime
constexpr uint32_t kSymNodes = 1u << 25;                  // node ids are below
constexpr int kSymPoints = 3;

// a * b mod p, up to a multiple of p: for integers |a| < 2 p and |b| < p, an
// integer below 2 p in size again.  h + l is the exact product and q its
// quotient within 1.5 (h / p < 2^52 suffers two roundings of 2^-53 each, then
// one to an integer), so |h - q p| <= 1.5 p is computed exactly, and |l| <
// p / 4 (half an ulp of h < 2^103).
__device__ __forceinline__ double sym_mul(double a, double b) {
  constexpr double p = static_cast<double>(kSymP), inv = 1.0 / p;
  const double h = a * b;
  const double l = __builtin_fma(a, b, -h);
  const double q = __builtin_rint(h * inv);
  return __builtin_fma(-q, p, h) + l;
}

// The same element, at most about p / 2 in size; |a| < 2 p.
__device__ __forceinline__ double sym_small(double a) {
  constexpr double p = static_cast<double>(kSymP), inv = 1.0 / p;
  return __builtin_fma(-__builtin_rint(a * inv), p, a);
}

// 2^52 + e of a pair: e is below 2^50, so these are its bits.
__device__ __forceinline__ double sym_pair(uint32_t u, uint32_t v) {
  const uint32_t a = u < v ? u : v, b = u < v ? v : u;
  const unsigned long long bits = 0x4330000000000000ull | (static_cast<unsigned long long>(a) << 25) | b;
  return __builtin_bit_cast(double, bits);
}

// The products at the points.  up: over arcs u -> v with u < v, down: over the
// others; `swapped` says which is which, so that an arc needs one
// multiplication whatever its direction.
struct SymProducts {
  double up[kSymPoints], down[kSymPoints];
  bool swapped;
};

__device__ __forceinline__ void sym_start(SymProducts& s) {
#pragma unroll
  for (int i = 0; i < kSymPoints; ++i) s.up[i] = s.down[i] = 1.0;
  s.swapped = false;
}

// Arc u -> v, u != v, both below kSymNodes; x: the points, each an integer in
// [0, p) plus 2^52 (exact: below 2^53).
__device__ __forceinline__ void sym_arc(SymProducts& s, uint32_t u, uint32_t v, const double (&x)[kSymPoints]) {
  const bool down = u > v, swap = down != s.swapped;
  const double e = sym_pair(u, v);
  s.swapped = down;
#pragma unroll
  for (int i = 0; i < kSymPoints; ++i) {
    const double now = swap ? s.down[i] : s.up[i];
    s.down[i] = swap ? s.up[i] : s.down[i];
    s.up[i] = sym_mul(now, x[i] - e);  // |x - e| < p: both terms lie in [0, p)
  }
}

__device__ __forceinline__ void sym_finish(SymProducts& s) {
#pragma unroll
  for (int i = 0; i < kSymPoints; ++i) {
    const double a = s.up[i];
    s.up[i] = s.swapped ? s.down[i] : a;
    s.down[i] = s.swapped ? a : s.down[i];
  }
  s.swapped = false;
}

// Takes in the products of other arcs (sym_finish both).
__device__ __forceinline__ void sym_join(SymProducts& s, const double (&up)[kSymPoints],
                                         const double (&down)[kSymPoints]) {
#pragma unroll
  for (int i = 0; i < kSymPoints; ++i) {
    s.up[i] = sym_mul(s.up[i], sym_small(up[i]));
    s.down[i] = sym_mul(s.down[i], sym_small(down[i]));
  }
}

// Whether the two products of a point are the same element.
__device__ __forceinline__ bool sym_equal(double a, double b) {
  return (static_cast<long long>(a) - static_cast<long long>(b)) % static_cast<long long>(kSymP) == 0;
}

}  // namespace lbg
