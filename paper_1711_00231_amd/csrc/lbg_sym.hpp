// Whether a graph is symmetric, by one pass over its arcs.
//
// A graph is symmetric when the pairs {u, v} of its arcs u -> v with u < v
// are, as a multiset, those of its arcs with u > v (self-loops are their own
// reverse).  So the products of x - e over the ones and over the others are
// formed at points x drawn at random, in the field of p = 2^51 - 129 elements,
// for e = 2^25 min(u, v) + max(u, v), which tells all pairs of a graph of at
// most 2^25 nodes apart (equality of multisets by products at a random point:
// Lipton 1989; Blum et al., Checking the correctness of memories, 1991).  The
// graph passes when the products are equal, and not zero, at every point.  A
// symmetric one does unless a point happens to be one of its e, which costs
// the pull levels of one solve.  Take any other, and k the larger of the
// numbers of arcs that its two sides hold beyond each other: without the
// factors they share, which are not zero, the products are two different
// monic polynomials in x of degree at most k, equal at no more than k points.
// So it passes with a chance of at most (k / p)^2 over the two points, which
// are drawn independently: below 2^-96 for up to eight one-way arcs, however
// they are arranged, below 2^-48 if all of 2^27 arcs are one-way (where a
// sample of a few arcs has long found one, see sym_sample).
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
constexpr int kSymPoints = 2;

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

// 2^52 + e of a pair, a < b: e is below 2^50, so these are its bits.
__device__ __forceinline__ double sym_pair(uint32_t a, uint32_t b) {
  const uint32_t hi = 0x43300000u | (a >> 7), lo = (a << 25) | b;
  return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}

// The products at the points: up over arcs u -> v with u < v, down over those
// with u > v, or (while `swapped`) the other way round, so that an arc takes
// one multiplication and a choice, whatever its direction.
struct SymProducts {
  double up[kSymPoints], down[kSymPoints];
};

__device__ __forceinline__ void sym_start(SymProducts& s) {
#pragma unroll
  for (int i = 0; i < kSymPoints; ++i) s.up[i] = s.down[i] = 1.0;
}

// Takes in pair a < b; swap: its direction is not the last one's.  x: the
// points, each an integer in [0, p) plus 2^52 (exact: below 2^53).
__device__ __forceinline__ void sym_take(SymProducts& s, bool swap, uint32_t a, uint32_t b,
                                         const double (&x)[kSymPoints]) {
  const double e = sym_pair(a, b);
#pragma unroll
  for (int i = 0; i < kSymPoints; ++i) {
    const double now = swap ? s.down[i] : s.up[i];
    s.down[i] = swap ? s.up[i] : s.down[i];
    s.up[i] = sym_mul(now, x[i] - e);  // |x - e| < p: both lie in [0, p)
  }
}

// After the last pair.
__device__ __forceinline__ void sym_finish(SymProducts& s, bool swapped) {
#pragma unroll
  for (int i = 0; i < kSymPoints; ++i) {
    const double a = s.up[i];
    s.up[i] = swapped ? s.down[i] : a;
    s.down[i] = swapped ? a : s.down[i];
  }
}

// Takes in the products of other arcs.
__device__ __forceinline__ void sym_join(SymProducts& s, const double (&up)[kSymPoints],
                                         const double (&down)[kSymPoints]) {
#pragma unroll
  for (int i = 0; i < kSymPoints; ++i) {
    s.up[i] = sym_mul(s.up[i], sym_small(up[i]));
    s.down[i] = sym_mul(s.down[i], sym_small(down[i]));
  }
}

// Whether the two products of a point are one element, and not zero.
__device__ __forceinline__ bool sym_equal(double a, double b) {
  constexpr long long p = static_cast<long long>(kSymP);
  const long long x = static_cast<long long>(a), y = static_cast<long long>(b);
  return (x - y) % p == 0 && x % p != 0;
}

}  // namespace lbg
