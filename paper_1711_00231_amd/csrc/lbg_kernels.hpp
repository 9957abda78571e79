// Frontier-expansion kernels for level-synchronous BFS and SSSP on gfx950.
//
// One launch processes one level (BFS) or one Bellman-Ford iteration (SSSP):
// it consumes worklist L (buffer L & 1, tail counter ctr[L % 3]), appends to
// worklist L+1 (buffer (L+1) & 1, counter ctr[(L+1) % 3]) and clears
// ctr[(L+2) % 3] for the launch after it.  Launches read their work size
// from device memory, so the host can enqueue many levels without waiting;
// a launch that finds an empty worklist returns at once.
//
// Relaxation (Section II-B).  Device atomics are the scarce resource on
// MI355X (about 27 G/s chip-wide, any scope, against ~250 G/s random L2
// reads), so each path filters with plain reads before it issues one:
//  * BFS claims an undiscovered node with an atomic OR on a visited bitmap.
//    An atomic on a line invalidates that line in every XCD's L2, so the hot
//    path never reads the bitmap it claims through.  It reads one per-XCD
//    advisory filter (n/8 bytes, resident in the XCD's L2) that holds `seen`
//    (a copy of the bitmap frozen for the level, merged in when the level
//    starts) plus the claims of the XCD's own blocks (plain stores), so a
//    visited node costs one L2 read and an XCD issues about one atomic per
//    new node.  The winner writes level L+1 and sets the bit in next level's
//    `seen`, which this launch also refreshes from the current one (plain
//    stores; a bit lost to a racing store only costs one more atomic later).
//  * SSSP keeps (distance << 32 | iteration of last improvement) per node and
//    relaxes with a single 64-bit atomicMin: the returned old value says both
//    whether the arc improved the node and whether the node is already queued
//    for this iteration (the worklist condensing concern of Section II-B is
//    handled at push time, with no second atomic).  The per-arc filter reads
//    a 2-byte copy, min(distance, 0xffff), instead of the 8-byte state (a
//    quarter of the random-read footprint: 8 MiB at scale 22, half of what an
//    XCD's L2 holds); winners refresh it with plain stores, so it may lag the
//    state but never undercuts it, and 0xffff (too large, or unknown) never
//    filters.  Batched SSSP rows keep the same 2-byte copy per row: their
//    state is far larger than the last-level cache, and the copy halves the
//    random-read footprint of filtering on the 4-byte output row (measured:
//    3.5 % faster on 2,048 solves over 322 M arcs).  A frontier node's own
//    distance is always read from the state, and the epilogue writes the
//    output from the state.
// Plain reads may be stale inside a launch; values only move one way (bits
// set, distances decrease), so a stale read can only cost an extra atomic,
// never a missed update.
#pragma once

#include "lbg_device.hpp"

namespace lbg {

constexpr uint32_t kBfsInf = 0x7fffffffu;
constexpr uint32_t kSsspInf = 0xffffffffu;

// Arc e of a single SSSP solve: destination and weight, from the CSR arrays
// or from one packed word.
template <bool kPacked, bool kNarrow>
__device__ __forceinline__ void load_arc(const KArgs& a, uint32_t e, int32_t* v, uint32_t* w) {
  if (kPacked) {
    const uint32_t pa = *at<kNarrow>(a.arcs, e);
    *v = static_cast<int32_t>(pa >> a.wbits);
    *w = pa & ((1u << a.wbits) - 1u);
  } else {
    *v = *at<kNarrow>(a.cols, e);
    *w = *at<kNarrow>(a.weights, e);
  }
}


template <typename T>
__device__ __forceinline__ T ld_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Level bookkeeping, by one thread of the grid: clear the counter two levels
// ahead (the one level L+1 appends to) and account level L.
__device__ __forceinline__ void level_account(const KArgs& a, uint32_t L, unsigned long long c) {
  __hip_atomic_store(&a.ctl->ctr[(L + 2) % 3], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (static_cast<uint32_t>(c) != 0u) {
    const unsigned long long fe = (c >> 32) ? (c >> 32) : static_cast<uint32_t>(c);
    if (a.team) {
      a.ctl->levels += 1;
      a.ctl->next = L + 1;
    } else {
      a.ctl->levels = L + 1;
    }
    a.ctl->frontier_entries += fe;
    a.ctl->edges_scanned += static_cast<uint32_t>(c);
  }
}

// Shared prologue of the one-level kernels: read this level's worklist size
// and account the level.  Returns the packed (nodes, edges) tail.
__device__ __forceinline__ unsigned long long level_begin(const KArgs& a, uint32_t L) {
  const unsigned long long c = __hip_atomic_load(&a.ctl->ctr[L % 3], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
  if (blockIdx.x == 0 && threadIdx.x == 0) level_account(a, L, c);
  return c;
}

// BFS, at the start of level L: the next level's `seen` snapshot starts as
// this level's (whole grid), and each XCD's advisory filter absorbs this
// level's snapshot (by the XCD's own blocks), so one read of the filter
// answers both "visited before this level" and "claimed by this XCD".
// Plain read-modify-writes: a bit lost to a racing store costs one atomic.
__device__ __forceinline__ void refresh_seen(const KArgs& a, uint32_t L) {
  const uint32_t* cur = a.seen[L & 1];
  uint32_t* nxt = a.seen[(L + 1) & 1];
  for (uint32_t k = blockIdx.x * kBlock + threadIdx.x; k < a.words; k += gridDim.x * kBlock)
    nxt[k] = cur[k];
  uint32_t* fx = a.xfilter + static_cast<size_t>(blockIdx.x % kXcds) * a.words;
  const uint32_t xb = blockIdx.x / kXcds, nxb = (gridDim.x - blockIdx.x % kXcds + kXcds - 1) / kXcds;
  for (uint32_t k = xb * kBlock + threadIdx.x; k < a.words; k += nxb * kBlock) {
    const uint32_t sw = cur[k];
    if (sw) fx[k] |= sw;
  }
}

// Block-level reduction of the per-thread counters, then one atomic per
// block on this XCD's stats line.  Must be reached by the whole block.
// skip: arcs of worklist entries passed over without loading them (an SSSP
// node that improved again in the iteration that expands it; its arcs are
// relaxed in the next one), kept in slot 7.
__device__ __forceinline__ void add_stats(const KArgs& a, uint32_t upd, uint32_t atom, uint32_t skip = 0u) {
  if (!a.count_stats) return;  // kernel-argument uniform
  __shared__ uint32_t red[3][kWaves];
  const uint32_t su = wave_sum(upd), sa = wave_sum(atom), sk = wave_sum(skip);
  const uint32_t wid = threadIdx.x >> 6;
  if (lane_id() == 0) {
    red[0][wid] = su;
    red[1][wid] = sa;
    red[2][wid] = sk;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long tu = 0, ta = 0, tk = 0;
    for (int w = 0; w < kWaves; ++w) {
      tu += red[0][w];
      ta += red[1][w];
      tk += red[2][w];
    }
    const int x = blockIdx.x % kXcds;
    if (tu) atomicAdd(&a.ctl->xstat[x][0], tu);
    if (ta) atomicAdd(&a.ctl->xstat[x][1], ta);
    if (tk) atomicAdd(&a.ctl->xstat[x][7], tk);
  }
}

// Relax one arc u -> v.  Returns true if v must be queued for the next
// level; then *s / *d receive v's first arc and out-degree.  *upd counts
// successful improvements/discoveries, *atom the global atomics issued.
template <bool kSssp>
__device__ __forceinline__ bool relax(const KArgs& a, uint32_t L, int32_t v, uint32_t du,
                                      uint32_t w, uint32_t* upd, uint32_t* atom, int32_t* s,
                                      int32_t* d) {
  if (static_cast<uint32_t>(v) >= a.n) {  // malformed cols (see lbg_validate_csr)
    atomicOr(&a.ctl->error, kErrBadArc);
    return false;
  }
  if (!kSssp) {
    const uint32_t word = static_cast<uint32_t>(v) >> 5;
    const uint32_t bit = 1u << (v & 31);
    uint32_t* f = a.xfilter + static_cast<size_t>(blockIdx.x % kXcds) * a.words;  // holds `seen`
    const uint32_t fw = f[word];
    if (fw & bit) return false;  // this XCD already claimed (or is claiming) v
    f[word] = fw | bit;          // plain store; a lost bit only costs one more atomic
    ++*atom;
    if (atomicOr(&a.visited[word], bit) & bit) return false;  // another XCD won
    a.levels[v] = static_cast<int32_t>(L + 1);
    uint32_t* sn = a.seen[(L + 1) & 1];
    sn[word] |= bit;  // plain read-modify-write: a lost bit only costs an atomic later
    ++*upd;
  } else {
    const uint32_t alt = du + w;
    if (alt >= f16_bound(a.d16[v])) return false;
    const unsigned long long mine = (static_cast<unsigned long long>(alt) << 32) | (L + 1);
    ++*atom;
    const unsigned long long old = atomicMin(&a.dstate[v], mine);
    if (alt >= static_cast<uint32_t>(old >> 32)) return false;
    a.d16[v] = f16_of(alt);  // filter; may lag the state, never undercuts it
    ++*upd;
    if (static_cast<uint32_t>(old) == L + 1) return false;  // already queued this iteration
  }
  const int32_t s0 = a.offsets[v];
  *s = s0;
  *d = a.offsets[v + 1] - s0;
  return *d > 0;  // a node without out-arcs has nothing to expand
}

// relax() for kB arcs of one lane at once: each step (filter reads, claims
// or atomic minima, the winners' offsets) is issued for all kB arcs before
// any result is used, so a lane keeps kB requests in flight instead of one.
// v[b] < 0: no arc.  On return want[b] says whether v[b] joins the next
// worklist, with its first arc s[b] and out-degree d[b].
template <bool kSssp, int kB>
__device__ __forceinline__ void relax_batch(const KArgs& a, uint32_t L, int32_t (&v)[kB], const uint32_t (&du)[kB],
                                            const uint32_t (&w)[kB], uint32_t* upd, uint32_t* atom,
                                            int32_t (&s)[kB], int32_t (&d)[kB], bool (&want)[kB]) {
  bool bad = false;
#pragma unroll
  for (int b = 0; b < kB; ++b)
    if (v[b] >= 0 && static_cast<uint32_t>(v[b]) >= a.n) {  // malformed cols (see lbg_validate_csr)
      bad = true;
      v[b] = -1;
    }
  if (bad) atomicOr(&a.ctl->error, kErrBadArc);
  uint32_t x[kB];
  bool win[kB];
  if (!kSssp) {
    uint32_t* f = a.xfilter + static_cast<size_t>(blockIdx.x % kXcds) * a.words;  // holds `seen`
#pragma unroll
    for (int b = 0; b < kB; ++b) x[b] = v[b] >= 0 ? f[static_cast<uint32_t>(v[b]) >> 5] : ~0u;
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const uint32_t word = static_cast<uint32_t>(v[b]) >> 5, bit = 1u << (v[b] & 31);
      if (v[b] >= 0 && !(x[b] & bit)) {
        f[word] = x[b] | bit;  // plain store; a lost bit only costs one more atomic
        ++*atom;
        x[b] = atomicOr(&a.visited[word], bit);
      } else {
        x[b] = ~0u;
      }
    }
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const uint32_t word = static_cast<uint32_t>(v[b]) >> 5, bit = 1u << (v[b] & 31);
      win[b] = v[b] >= 0 && !(x[b] & bit);
      if (win[b]) {
        a.levels[v[b]] = static_cast<int32_t>(L + 1);
        a.seen[(L + 1) & 1][word] |= bit;  // plain read-modify-write: a lost bit only costs an atomic later
        ++*upd;
      }
    }
  } else {
#pragma unroll
    for (int b = 0; b < kB; ++b) x[b] = v[b] >= 0 ? f16_bound(a.d16[v[b]]) : 0u;
    unsigned long long old[kB];
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const uint32_t alt = du[b] + w[b];
      old[b] = 0ull;
      if (v[b] >= 0 && alt < x[b]) {
        ++*atom;
        old[b] = atomicMin(&a.dstate[v[b]], (static_cast<unsigned long long>(alt) << 32) | (L + 1));
      }
    }
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const uint32_t alt = du[b] + w[b];
      const bool better = v[b] >= 0 && alt < x[b] && alt < static_cast<uint32_t>(old[b] >> 32);
      if (better) {
        a.d16[v[b]] = f16_of(alt);  // filter; may lag the state, never undercuts it
        ++*upd;
      }
      win[b] = better && static_cast<uint32_t>(old[b]) != L + 1;  // not yet queued this iteration
    }
  }
#pragma unroll
  for (int b = 0; b < kB; ++b) {
    s[b] = 0;
    d[b] = 0;
    if (win[b]) {
      s[b] = a.offsets[v[b]];
      d[b] = a.offsets[v[b] + 1];
    }
  }
#pragma unroll
  for (int b = 0; b < kB; ++b) {
    d[b] -= s[b];
    want[b] = win[b] && d[b] > 0;  // a node without out-arcs has nothing to expand
  }
}

// ------------------------------------------------------------------ init --
// Output = infinity, source = 0, visited/stamp cleared, worklist 0 = {src}
// (node strategies) or src's arcs (edge strategy).
template <bool kSssp>
__device__ __forceinline__ void init_state(const KArgs& a, int32_t src, uint32_t gid, uint32_t stride) {
  for (uint32_t v = gid; v < a.n; v += stride) {
    if (kSssp) {
      a.dstate[v] = (v == static_cast<uint32_t>(src)) ? 0ull
                                                      : (static_cast<unsigned long long>(kSsspInf) << 32);
      // the balanced strategy keeps the team's flags in the output until
      // k_sssp_finish writes it
      if (!a.team) a.dist[v] = (v == static_cast<uint32_t>(src)) ? 0u : kSsspInf;
      a.d16[v] = (v == static_cast<uint32_t>(src)) ? 0 : static_cast<uint16_t>(kF16None);
    } else {
      a.levels[v] = (v == static_cast<uint32_t>(src)) ? 0 : static_cast<int32_t>(kBfsInf);
    }
  }
  if (!kSssp) {
    const uint32_t sw = static_cast<uint32_t>(src) >> 5;
    for (uint32_t w = gid; w < a.words; w += stride) {
      const uint32_t bits = (w == sw) ? (1u << (src & 31)) : 0u;
      a.visited[w] = bits;
      a.seen[0][w] = bits;
      // seen[1] must not carry another solve's bits: level 0 may OR into a
      // word of it before refreshing that word
      a.seen[1][w] = 0u;
    }
    const uint32_t fwords = a.words * kXcds;
    for (uint32_t w = gid; w < fwords; w += stride) a.xfilter[w] = 0u;
  }
  if (gid == 0) {
    a.ctl->error = 0u;
    a.ctl->levels = 0u;
    a.ctl->frontier_entries = 0ull;
    a.ctl->edges_scanned = 0ull;
    a.ctl->p_frontier_entries = 0ull;
    a.ctl->p_edges_scanned = 0ull;
    a.ctl->next = 0u;
    a.ctl->worked = 0ull;
    a.ctl->sym_run = 0u;
    a.ctl->split_at = 0u;
    a.ctl->far_seen = 0u;
  }
}

// Near-far SSSP.  Plain Bellman-Ford expands every improved node in the next
// iteration, whatever its distance, and on graphs of long shortest paths most
// of that work is done again with better distances later: 96 x the arcs of the
// 2048 x 2048 grid without shortcuts, 4.3 x with 1 % shortcuts, 3.7 x those of
// a uniform graph of 2^20 nodes (measured with the weights of those
// workloads).  So a node whose distance exceeds a threshold T is not queued
// but put in the far set, one bit per node; once the worklist is empty T grows
// by delta and a split moves the nodes of the far set with distances up to T
// to the worklist (the deferral of delta-stepping, Meyer and Sanders 2003, and
// of the near-far worklists of Davidson et al. 2014, here with a bitmap, so a
// node is held once and any order of updates is right).  Invariant: a reached
// node that has not been expanded with its present distance is in the
// worklist or in the far set.  A bit may outlive its node's move to the
// worklist (its clearing may overtake its setting); then the node is expanded
// once more.
//
// The step: 16 x the mean weight / the mean out-degree, i.e. about 16 arcs
// of a node's share of weight.  Smaller steps relax fewer arcs in more
// iterations.  Counted with a host model of the rule, arcs relaxed /
// iterations: grid with shortcuts, 1 x mean weight 1.12 / 189, 4 x (this rule)
// 1.38 / 119, 8 x 1.72 / 105; uniform 2^20, 1 x 1.27 / 41, 2 x (this rule)
// 1.33 / 35, 4 x 3.66 / 30.  While even the largest level of a step is a fraction of what
// the chip takes in one round of latency the step doubles (the grid without
// shortcuts: 4587 iterations at 4 x, 3560 with doubling).
//
// What it saves is the work of nodes reached over few heavy arcs before many
// light ones.  Where the weights hardly differ there are none, and the extra
// iterations only cost: decided by the spread of a sample of the weights
// (standard deviation / mean; 0.33 for weights 1 - 2, 0.45 for 1 - 4, 0.52 for
// 1 - 10, 0.58 for wide ranges), deferring against not, in ms.  Uniform graph
// of 10^6 nodes and 8 arcs per node: equal 0.54 / 0.38, 50 - 100 0.63 / 0.44,
// 1 - 4 0.72 / 0.62, 1 - 10 0.78 / 0.86, 1 - 100 1.00 / 1.21.  Grid of 1500 x
// 1500, 3.6 arcs per node: 1 - 2 1.03 / 1.00, 1 - 4 1.17 / 1.27.  And graphs of
// few arcs per node lose as the dense ones do (solve() in lbg.hip) when most
// of their nodes have next to none: directed R-MAT of 2^21 nodes, 8 arcs per
// node, 1.05 / 0.93 ms (half of its nodes have less than a 20th of the mean;
// a power-law tail over nodes of ordinary degree, 10^6 nodes, gains: 1.08 /
// 1.11 to 1.17 / 1.63).
constexpr double kFarSpread = 0.4, kFarSpreadDense = 0.485;  // the second from kFarDense arcs per node on
constexpr uint32_t kFarDense = 6;
constexpr uint32_t kFarIdle = 16384;  // arcs of a level that latency hides
constexpr uint32_t kFarSample = 4096;

// One workgroup: whether to defer and the first threshold, from samples of the
// weights and the out-degrees, then the other words of the team's control
// block.
__device__ __forceinline__ void near_far_init(const KArgs& a) {
  constexpr int kN = 3;
  __shared__ double red[kN][kBlock];  // weights, their squares, nodes below a quarter of the mean degree
  double x[kN] = {0.0, 0.0, 0.0};
  for (uint32_t k = threadIdx.x; k < kFarSample; k += kBlock) {
    const uint32_t e = static_cast<uint32_t>(static_cast<unsigned long long>(k) * a.m / kFarSample);
    const double w = static_cast<double>(a.arcs ? a.arcs[e] & ((1u << a.wbits) - 1u) : a.weights[e]);
    const uint32_t v = static_cast<uint32_t>(static_cast<unsigned long long>(k) * a.n / kFarSample);
    const double d = static_cast<double>(a.offsets[v + 1]) - static_cast<double>(a.offsets[v]);
    x[0] += w;
    x[1] += w * w;
    x[2] += 4.0 * d * a.n < a.m ? 1.0 : 0.0;
  }
  for (int i = 0; i < kN; ++i) red[i][threadIdx.x] = x[i];
  __syncthreads();
  for (uint32_t h = kBlock / 2; h > 0; h /= 2) {
    if (threadIdx.x < h)
      for (int i = 0; i < kN; ++i) red[i][threadIdx.x] += red[i][threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double sum = red[0][0];
    const double spread = a.m >= static_cast<unsigned long long>(kFarDense) * a.n ? kFarSpreadDense : kFarSpread;
    const bool narrow = red[1][0] * kFarSample <= (1.0 + spread * spread) * sum * sum;
    const bool skewed = 2.0 * red[2][0] >= kFarSample;
    a.ctl->plain = narrow || skewed ? 1u : 0u;
    TeamCtl* t = a.team;
    for (int k = 0; k < 4; ++k) t->join[k] = t->size[k] = 0u;
    t->epoch = 0u;
    const double step = 16.0 * sum / kFarSample * a.n / a.m;
    t->delta0 = static_cast<uint32_t>(step < 1.0 ? 1.0 : (step > 1e9 ? 1e9 : step));
    t->thr[0] = t->delta[0] = t->delta0;
    t->at[0] = 0u;
    t->most[0] = 0u;
    for (uint32_t k = 0; k < 2 * kTeamFew; ++k) t->flag[k] = 0ull;
  }
}

// A node whose distance was `was` (> T) has improved: out of the far set if
// it is queued now, into it if this is the first time it is reached.
template <bool kNarrow>
__device__ __forceinline__ void far_move(const KArgs& a, uint32_t v, uint32_t was, bool queued) {
  if (queued) {
    if (was != kSsspInf) atomicAnd(at<kNarrow>(a.far, v >> 5), ~(1u << (v & 31)));
  } else if (was == kSsspInf) {
    atomicOr(at<kNarrow>(a.far, v >> 5), 1u << (v & 31));
  }
}

// The bits of word k of the far set that stand for nodes.
__device__ __forceinline__ uint32_t far_mask(const KArgs& a, uint32_t k) {
  return k + 1 < a.words || (a.n & 31u) == 0u ? ~0u : (1u << (a.n & 31u)) - 1u;
}

// The threshold and step of a split, from those of the steps before.
__device__ __forceinline__ void far_raise(uint32_t delta0, uint32_t most, uint32_t* thr, uint32_t* delta) {
  uint32_t d = *delta;
  if (most < kFarIdle && (most == 0u || d / 4 < delta0)) d = d < 0x40000000u ? 2 * d : d;
  else if (most > 8 * kFarIdle && d > delta0) d = max(delta0, d / 2);
  *delta = d;
  *thr = *thr < kSsspInf - d ? *thr + d : kSsspInf;
}

// A sample of arcs u -> v for symmetry (the last workgroup of k_init, while
// the others clear the state; see lbg_pull.hpp): a thread takes a node, the
// one of its first 8 neighbours with the fewest arcs, and looks for the way
// back among those, if they are at most 32.  Where few threads find such a
// neighbour (dense graphs), each wavefront looks through the two shortest
// longer lists, of at most 4096 arcs, together.  Nodes without either say
// nothing.  (A digraph of 30,000 nodes and 10^8 arcs, whose lists are all
// longer than 32: without the second part every solve went over all arcs,
// 0.49 ms against 0.41 without pull levels.)
constexpr uint32_t kSampleAlone = 32, kSampleLong = 4096;
__device__ __forceinline__ void sym_sample(const KArgs& a) {
  __shared__ uint32_t no;
  if (threadIdx.x == 0) no = 0u;
  __syncthreads();
  const uint32_t u =
      (threadIdx.x * 0x9e3779b1u + static_cast<uint32_t>(__builtin_bit_cast(unsigned long long, a.sym_x[0]) >> 8)) % a.n;
  const uint32_t s = static_cast<uint32_t>(a.offsets[u]), e = static_cast<uint32_t>(a.offsets[u + 1]);
  uint32_t vs = 0, ve = 0, best = kSampleLong + 1;
  if (s < e && e <= a.m) {
    uint32_t v[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) v[k] = s + k < e ? static_cast<uint32_t>(a.cols[s + k]) : 0xffffffffu;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      if (v[k] >= a.n || v[k] == u) continue;
      const uint32_t p = static_cast<uint32_t>(a.offsets[v[k]]), q = static_cast<uint32_t>(a.offsets[v[k] + 1]);
      if (p <= q && q <= a.m && q - p < best) {
        best = q - p;
        vs = p;
        ve = q;
      }
    }
  }
  if (best <= kSampleAlone) {
    bool back = false;
    for (uint32_t p = vs; p < ve && !back; p += 8) {
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) back = back || (p + k < ve && static_cast<uint32_t>(a.cols[p + k]) == u);
    }
    if (!back) no = 1u;
  }
  if (__syncthreads_count(best <= kSampleAlone) < kBlock / 4) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t len = best > kSampleAlone ? best : kSampleLong + 1;
    for (int r = 0; r < 2; ++r) {
      const uint32_t key = static_cast<uint32_t>(-wave_max(-static_cast<int32_t>(len << 6 | lane)));
      if (key >> 6 > kSampleLong) break;
      const int who = static_cast<int>(key & 63);
      const uint32_t wu = __shfl(u, who, 64), we = __shfl(ve, who, 64);
      bool back = false;
      for (uint32_t p = __shfl(vs, who, 64); p < we && !__any(back); p += 64 * 8) {
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
          const uint32_t i = p + k * 64 + lane;
          back = back || (i < we && static_cast<uint32_t>(a.cols[i]) == wu);
        }
      }
      if (!__any(back)) no = 1u;
      if (static_cast<int>(lane) == who) len = kSampleLong + 1;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) a.ctl->sym_no = no;
}

template <bool kSssp, bool kEdgeWl>
__global__ __launch_bounds__(kBlock) void k_init(KArgs a, int32_t src) {
  const uint32_t gid = blockIdx.x * kBlock + threadIdx.x;
  const uint32_t stride = gridDim.x * kBlock;
  // the host checked 0 <= src < n; a renaming table is the caller's array
  if (a.node_map) src = a.node_map[src];
  if (a.team) {  // also for a source outside the graph: the launches that follow read it
    if (a.far) {
      for (uint32_t k = gid; k < a.words; k += stride) a.far[k] = 0u;
      if (blockIdx.x == 0) near_far_init(a);
    } else if (gid < sizeof(TeamCtl) / 4) {
      reinterpret_cast<uint32_t*>(a.team)[gid] = 0u;
    }
    for (uint32_t k = gid; k < 2 * a.tblocks; k += stride) a.tflag[k] = 0ull;
  }
  if (static_cast<uint32_t>(src) >= a.n) {
    if (gid == 0) {
      a.ctl->error = kErrBadSrc;
      a.ctl->levels = 0u;
      // every level finds no work, and the far set, if any, no node
      a.ctl->ctr[0] = a.ctl->ctr[1] = a.ctl->ctr[2] = 0ull;
      a.ctl->next = 0u;
      a.ctl->split_at = 0u;
      a.ctl->far_seen = 0u;
    }
    return;
  }
  if (!kSssp && a.pull_min && blockIdx.x == gridDim.x - 1) sym_sample(a);
  init_state<kSssp>(a, src, gid, stride);
  if (a.hier_trace)
    for (uint32_t k = gid; k < kHierTraceLevels * kHierTraceSubs; k += stride) a.hier_trace[k] = 0u;
  const int32_t s0 = a.offsets[src];
  int32_t d0 = a.offsets[src + 1] - s0;
  if (s0 < 0 || d0 < 0 || static_cast<uint32_t>(s0) + static_cast<unsigned long long>(d0) > a.m) {
    if (gid == 0) atomicOr(&a.ctl->error, kErrBadArc);  // malformed offsets: start with no work
    d0 = 0;
  }
  if (kEdgeWl) {
    for (uint32_t k = gid; k < static_cast<uint32_t>(d0); k += stride) a.fr[0].node[k] = s0 + k;
  } else {
    constexpr uint32_t T = TileCfg<kSssp>::kEdges;
    const uint32_t tiles = (static_cast<uint32_t>(d0) + T - 1) / T;
    for (uint32_t t = gid; t < tiles && t < a.tile_cap; t += stride) a.fr[0].tile_node[t] = 0;
  }
  if (!kEdgeWl && a.child_base) {
    // split graph: the source's own piece, then its children's pieces (one
    // thread; tile marks by the thread that owns each tile)
    int32_t cb = a.child_base[src], ce = a.child_base[src + 1];
    if (cb < 0 || ce < cb || static_cast<uint32_t>(ce) > a.node_cap - a.n) {
      if (gid == 0) atomicOr(&a.ctl->error, kErrBadSplit);
      cb = ce = 0;
    }
    if (gid == 0) {
      uint32_t i = 0, p = 0;
      if (d0 > 0) {
        a.fr[0].node[0] = src;
        a.fr[0].eprefix[0] = 0u;
        a.fr[0].estart[0] = s0;
        i = 1;
        p = static_cast<uint32_t>(d0);
      }
      for (int32_t c = cb; c < ce && i < a.node_cap; ++c) {
        const int32_t cs = a.offsets[a.n + c], cl = a.offsets[a.n + c + 1] - cs;
        if (cl <= 0) {  // not a table lbg_split_graph wrote
          atomicOr(&a.ctl->error, kErrBadSplit);
          continue;
        }
        a.fr[0].node[i] = src;
        a.fr[0].eprefix[i] = p;
        a.fr[0].estart[i] = cs;
        ++i;
        p += static_cast<uint32_t>(cl);
      }
      a.ctl->ctr[0] = p > 0 ? ((static_cast<unsigned long long>(i) << 32) | p) : 0ull;
      a.ctl->ctr[1] = 0ull;
      a.ctl->ctr[2] = 0ull;
    }
    // tile t starts in the piece holding edge t * T
    constexpr uint32_t T = TileCfg<kSssp>::kEdges;
    const int32_t tot = d0 + (ce > cb ? a.offsets[a.n + ce] - a.offsets[a.n + cb] : 0);
    const uint32_t tiles = tot > 0 ? (static_cast<uint32_t>(tot) + T - 1) / T : 0u;
    for (uint32_t t = gid; t < tiles && t < a.tile_cap; t += stride) {
      const uint32_t e = t * T;
      uint32_t i = 0, p = 0;
      if (d0 > 0) {
        if (e < static_cast<uint32_t>(d0)) {
          a.fr[0].tile_node[t] = 0;
          continue;
        }
        i = 1;
        p = static_cast<uint32_t>(d0);
      }
      for (int32_t c = cb; c < ce; ++c) {
        const int32_t cl = a.offsets[a.n + c + 1] - a.offsets[a.n + c];
        if (cl <= 0) continue;
        if (e < p + static_cast<uint32_t>(cl)) break;
        ++i;
        p += static_cast<uint32_t>(cl);
      }
      a.fr[0].tile_node[t] = static_cast<int32_t>(i);
    }
    if (gid < kXcds * 16) a.ctl->xstat[gid / 16][gid % 16] = 0ull;
    return;
  }
  // the source's entry (pieces of at most a.mdt arcs for the binned strategy)
  const uint32_t pc = kEdgeWl ? 0u : split_count(static_cast<uint32_t>(d0 > 0 ? d0 : 0), a.mdt);
  for (uint32_t k = gid; k < pc; k += stride) {
    uint32_t off, len;
    split_piece(static_cast<uint32_t>(d0), pc, k, &off, &len);
    a.fr[0].node[k] = src;
    a.fr[0].eprefix[k] = off;
    a.fr[0].estart[k] = s0 + static_cast<int32_t>(off);
  }
  if (gid == 0) {
    const unsigned long long nodes = kEdgeWl ? 0ull : pc;
    a.ctl->ctr[0] = d0 > 0 ? ((nodes << 32) | static_cast<uint32_t>(d0)) : 0ull;
    a.ctl->ctr[1] = 0ull;
    a.ctl->ctr[2] = 0ull;
  }
  if (gid < kXcds * 16) a.ctl->xstat[gid / 16][gid % 16] = 0ull;
}

// SSSP epilogue: once the worklist of the next level to expand (ctl->levels:
// the last non-empty level + 1; balanced: ctl->next) is empty, and the far set
// too, copy the distances out of the packed state.  Launched after every step
// of the level loop; exits at once while work remains, so the host needs no
// extra synchronisation.
__global__ __launch_bounds__(kBlock) void k_sssp_finish(KArgs a) {
  const uint32_t L = __hip_atomic_load(a.team ? &a.ctl->next : &a.ctl->levels, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
  const unsigned long long c = __hip_atomic_load(&a.ctl->ctr[L % 3], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
  if (static_cast<uint32_t>(c) != 0u) return;
  if (a.far && a.ctl->plain == 0u && !(a.ctl->split_at == L && a.ctl->far_seen != L)) return;  // the far set may hold nodes
  if (a.sliced) {  // and the 8 slice lists
    for (int x = 0; x < kXcds; ++x)
      if (static_cast<uint32_t>(__hip_atomic_load(&a.ctl->xstat[x][4 + L % 3], __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT)) != 0u)
        return;
  }
  const uint32_t stride = gridDim.x * kBlock;
  if (a.node_map) {  // distances in original ids
    for (uint32_t v = blockIdx.x * kBlock + threadIdx.x; v < a.n; v += stride) {
      const uint32_t u = static_cast<uint32_t>(a.node_map[v]);
      a.dist[v] = u < a.n ? static_cast<uint32_t>(a.dstate[u] >> 32) : kSsspInf;
    }
    return;
  }
  for (uint32_t v = blockIdx.x * kBlock + threadIdx.x; v < a.n; v += stride)
    a.dist[v] = static_cast<uint32_t>(a.dstate[v] >> 32);
}

// ------------------------------------------------------ balanced (WD) ----
// Workload decomposition (Section III-A): the E_f edges of worklist L are cut
// into tiles of T = 64 x kItems consecutive edges, and global wavefront g
// (of W) takes tiles g, g + W, ...  Within a tile, the worklist entries that
// overlap it are staged in the wavefront's LDS (one word per entry: the arc
// index of the tile's first slot if the entry covered it, plus the entry's
// current distance for SSSP); a bitmask of entry starts with per-word
// popcount prefixes maps each edge slot to its entry in O(1).  Lane l handles
// slots l, l + 64, ..., so the lanes read consecutive arcs of the same node
// (coalesced) whatever the degree distribution; hubs simply span many tiles
// and are expanded by many wavefronts at once.
//
// The kernel is latency-bound unless each round trip carries many
// independent requests, and a workgroup-wide barrier per tile would make
// every tile wait for its slowest wavefront.  So wavefronts run their tiles
// independently (no barrier inside the loop), every phase issues all of a
// lane's kItems loads (or atomics) before consuming any, the next tile's
// start entry is fetched one tile ahead, and discoveries go to per-wave LDS
// queues whose degree reads happen in bulk at flush time.
template <bool kSssp, bool kMulti>
struct WaveLds {
  static constexpr uint32_t T = TileCfg<kSssp, kMulti>::kEdges;
  uint32_t base[T];
  uint32_t du[kSssp ? T : 1];
  int32_t delta[kMulti ? T : 1];
  int32_t lo[kMulti ? T : 1];        // first node of the query's instance
  uint32_t lenkind[kMulti ? T : 1];  // instance size | (kind << 31)
  int32_t qid[kMulti ? T : 1];
  uint32_t flag[T / 32];
  uint32_t wpre[T / 32];
  int32_t qv[kWQ];
  int32_t qq[kMulti ? kWQ : 1];
};

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// kMulti: batched solves (always the SSSP relaxation; BFS queries use unit
// weights).  Entry (q, u) relaxes arc u -> v into row(q, v) = v + delta(q).
// Capacity check of a level's packed (nodes, edges) tail; block-uniform.
template <bool kSssp, bool kMulti>
__device__ __forceinline__ bool level_fits(const KArgs& a, unsigned long long c) {
  constexpr uint32_t T = TileCfg<kSssp, kMulti>::kEdges;
  const uint32_t Ef = static_cast<uint32_t>(c);
  const uint32_t nf = static_cast<uint32_t>(c >> 32);
  return nf <= a.node_cap &&
         Ef <= (kMulti ? static_cast<unsigned long long>(a.tile_cap) * T : static_cast<unsigned long long>(a.m));
}

constexpr uint32_t kTilesPerWave = 4;

// One level of the balanced expansion by the whole grid (all threads of
// every block must call it).  c = the level's packed tail, non-empty and
// within capacity.
template <bool kSssp, bool kNarrow, bool kMulti, bool kPacked = false, bool kSplit = false, bool kFar = false>
__device__ __forceinline__ void expand_level(const KArgs& a, uint32_t L, unsigned long long c) {
  static_assert(!kMulti || kSssp, "batched solves use the SSSP relaxation");
  static_assert(!kPacked || (kSssp && !kMulti), "packed arcs: single SSSP solves");
  constexpr int kItems = TileCfg<kSssp, kMulti>::kItems;
  constexpr uint32_t T = TileCfg<kSssp, kMulti>::kEdges;
  constexpr int kPay = kMulti ? 2 : (kSssp ? 1 : 0);
  __shared__ WaveLds<kSssp, kMulti> lds[kWaves];
  __shared__ uint32_t merge[2 * kWaves];
  __shared__ unsigned long long merge_base;

  const uint32_t Ef = static_cast<uint32_t>(c);
  const uint32_t nf = static_cast<uint32_t>(c >> 32);
  const Frontier cur = a.fr[L & 1];
  Frontier nxt = a.fr[(L + 1) & 1];
  nxt.level = L + 1;
  const int nctr = (L + 1) % 3;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wid = threadIdx.x >> 6;
  WaveLds<kSssp, kMulti>& w = lds[wid];
  uint32_t* fx = a.xfilter + static_cast<size_t>(blockIdx.x % kXcds) * a.words;
  uint32_t* seen_nxt = a.seen[(L + 1) & 1];
  // A frontier node's own distance comes from the packed state
  // (authoritative); the per-arc filter reads the 2-byte copy.
  const uint32_t state_len = kMulti ? a.rows : a.n;
  uint32_t upd = 0, atom = 0, qcount = 0, skip = 0;
  // BFS scan mode (see k_bfs_compact): grid-uniform.  A scan level needs no
  // snapshot refresh: k_bfs_prep already merged `visited` into every XCD's
  // filter, and the compaction rewrites the next snapshot from the levels.
  const bool scan = !kSssp && !kMulti && !kSplit && Ef >= a.scan_min;
  if (!kSssp && !scan) refresh_seen(a, L);

  // Near-far SSSP (above): a split step when the worklist is empty.
  static_assert(!kFar || (kSssp && !kMulti && !kSplit), "near-far: single SSSP solves");
  uint32_t thr = kSsspInf;
  const bool split = kFar && Ef == 0u;
  if constexpr (kFar) {
    uint32_t delta = a.team->delta[L % 3], most = a.team->most[L % 3];
    thr = a.team->thr[L % 3];
    if (split) {
      far_raise(a.team->delta0, most, &thr, &delta);
      most = 0u;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      a.team->thr[(L + 1) % 3] = thr;
      a.team->delta[(L + 1) % 3] = delta;
      a.team->most[(L + 1) % 3] = max(most, Ef);
      a.ctl->next = L + 1;
      if (split) a.ctl->split_at = L + 1;
    }
  }

  const uint32_t ntiles = (Ef + T - 1) / T;
  // How many workgroups take part.  SSSP levels of few tiles per wavefront
  // relax too early when all of them run at once: every arc then sees the
  // distances from before the level, where half the wavefronts see those of
  // the tiles before theirs too, skip more entries and improve fewer nodes
  // twice.  From kTilesPerWave tiles for each wavefront on there is no
  // difference left, and memory needs the wavefronts.  R-MAT, 300,007 nodes:
  // 0.50 -> 0.46 ms; scale 18: 0.51 -> 0.48 ms, 25.0 -> 23.0 M arcs relaxed;
  // scale 22 unchanged (2.50 ms; 2.66 with three quarters of the wavefronts
  // throughout, 3.17 with half).  A quarter on the smallest levels gains
  // nothing more on scale 18 and loses 4 % on scale 15.  Near-far solves
  // relax few arcs twice, and lose 6 % (grid) and 1 % (uniform) with it.
  uint32_t G = gridDim.x;
  if (kSssp && !kMulti && !kFar) {
    G = min(G, max(G / 2, ntiles / (kWaves * kTilesPerWave)));
    if (blockIdx.x >= G) return;
  }
  const uint32_t W = G * kWaves;
  // Tile deal.  Tiles [0, S) go round-robin to the W wavefronts (tile g,
  // g + W, ...); single solves take the last eighth from per-XCD counters
  // (XCD x hands out S + x, S + x + 8, ...), so a wavefront that drew cheap
  // tiles (skipped entries, few winners) takes more at the end instead of
  // waiting at the workgroup's final barrier for its slowest sibling.  A
  // larger dynamic share loses: hundreds of wavefronts then queue on each
  // counter (measured on R-MAT 22: an eighth dynamic, BFS 2 % and SSSP 2.4 %
  // faster than all round-robin; a quarter 1 %; half or all, SSSP 4-11 %
  // slower).  The first round is always round-robin, so levels of at most
  // W tiles take no atomic.  The counters of level L are
  // ctl->xstat[x][8 + L % 3], cleared by launch L - 1 (or by the
  // small-frontier kernel that ran level L - 1, or by k_init).
  const bool dyn = !kMulti && G >= static_cast<uint32_t>(kXcds);
  const uint32_t S = (dyn && ntiles > W) ? max(W, (ntiles - ntiles / 8) / W * W) : ntiles;
  const uint32_t xcd = blockIdx.x % kXcds;
  unsigned long long* const dctr = &a.ctl->xstat[xcd][8 + L % 3];
  if (dyn && blockIdx.x < static_cast<uint32_t>(kXcds) && threadIdx.x == 0)
    a.ctl->xstat[blockIdx.x][8 + (L + 1) % 3] = 0ull;
  auto take = [&]() -> uint32_t {  // wave-uniform
    uint32_t k = 0;
    if (lane == 0) k = static_cast<uint32_t>(atomicAdd(dctr, 1ull));
    k = __shfl(k, 0, 64);
    return S + xcd + static_cast<uint32_t>(kXcds) * k;
  };
  uint32_t tile = blockIdx.x * kWaves + wid;
  if constexpr (kFar) {
    // Split: the far set's words, one per lane; the nodes within the
    // threshold leave it for worklist L + 1.
    if (split) {
      for (uint32_t k0 = tile * 64; k0 < a.words; k0 += W * 64) {
        const uint32_t k = k0 + lane;
        const uint32_t had = k < a.words ? *at<kNarrow>(a.far, k) & far_mask(a, k) : 0u;
        uint32_t left = had, kept = 0u;
        if (__any(had != 0u) && lane == 0) a.ctl->far_seen = L + 1;  // one value from every writer
        while (__any(left != 0u)) {
          constexpr int kB = 4;
          int32_t v[kB];
          bool near[kB];
          uint32_t P = 0;
#pragma unroll
          for (int b = 0; b < kB; ++b) {
            v[b] = left ? static_cast<int32_t>(32 * k + __builtin_ctz(left)) : -1;
            left &= left - 1u;
          }
#pragma unroll
          for (int b = 0; b < kB; ++b)
            near[b] = v[b] >= 0 && static_cast<uint32_t>(*at<kNarrow>(a.dstate, static_cast<uint32_t>(v[b])) >> 32) <= thr;
#pragma unroll
          for (int b = 0; b < kB; ++b) {
            if (v[b] >= 0 && !near[b]) kept |= 1u << (v[b] & 31);
            P += static_cast<uint32_t>(__popcll(__ballot(near[b])));
          }
          if (qcount + P > static_cast<uint32_t>(kWQ)) {
            WaveFlush<kPay, T, kNarrow, kSplit> f;
            f.flush(a, w.qv, w.qq, qcount, nxt, nctr);
            qcount = 0;
            wave_sync();
          }
#pragma unroll
          for (int b = 0; b < kB; ++b)
            wq_push<kPay, T, kNarrow, kSplit>(a, w.qv, w.qq, qcount, near[b], v[b], 0, nxt, nctr);
        }
        if (kept != had) *at<kNarrow>(a.far, k) = kept;
      }
    }
  }
  if (tile >= S) tile = S < ntiles ? take() : ntiles;
  uint32_t i0_next = tile < ntiles ? static_cast<uint32_t>(*at<kNarrow>(cur.tile_node, tile)) : 0u;
  uint32_t tnext = ntiles;
  for (; tile < ntiles; tile = tnext) {
    const uint32_t i0 = i0_next;
    // next tile: its mark is fetched now (round-robin) or once the counter
    // has answered, after staging (dynamic)
    const bool rr = tile + W < S;
    tnext = rr ? tile + W : (S < ntiles ? take() : ntiles);
    if (rr) i0_next = static_cast<uint32_t>(*at<kNarrow>(cur.tile_node, tnext));
    const uint32_t t0 = tile * T;
    const uint32_t t1 = min(t0 + T, Ef);
    if (i0 >= nf) {  // wave-uniform; cannot happen when every tile was marked
      if (lane == 0) atomicOr(&a.ctl->error, kErrBadTile);
      if (!rr && tnext < ntiles) i0_next = static_cast<uint32_t>(*at<kNarrow>(cur.tile_node, tnext));
      continue;
    }
    if (lane < T / 32) w.flag[lane] = 0u;
    wave_sync();
    // Stage the entries overlapping [t0, t1): a contiguous run starting at i0
    // of at most T entries (each holds >= 1 edge).  An entry's reads are
    // issued together.
    bool bad = false;  // malformed input (see lbg_validate_csr): flagged, arc skipped
    bool live = false;  // SSSP: this lane staged an entry that is not skipped
    for (uint32_t j = lane; j < T; j += 64) {
      const uint32_t i = i0 + j;
      bool valid = false;
      if (i < nf) {
        const uint32_t p = *at<kNarrow>(cur.eprefix, i);
        const uint32_t st = static_cast<uint32_t>(*at<kNarrow>(cur.estart, i));
        const int32_t node = kSssp ? *at<kNarrow>(cur.node, i) : 0;
        const int32_t q = kMulti ? *at<kNarrow>(cur.qid, i) : 0;
        if (p < t1) {
          valid = true;
          w.base[j] = st + t0 - p;  // arc of slot s is base + s (mod 2^32)
          int32_t delta = 0;
          uint32_t level0 = 0;
          if (kMulti) {
            const QInfo qi = a.qtab[q];
            delta = qi.delta;
            level0 = qi.level0;
            w.delta[j] = qi.delta;
            w.lo[j] = qi.row_start - qi.delta;
            w.lenkind[j] = static_cast<uint32_t>(qi.row_len) | (qi.kind ? 0x80000000u : 0u);
            w.qid[j] = q;
          }
          if (kSssp) {
            const uint32_t row = static_cast<uint32_t>(node + delta);
            if (kMulti && !(w.lenkind[j] >> 31)) {
              // BFS query: its frontier nodes are exactly its nodes at hop
              // distance L - level0
              w.du[j] = L - level0;
              live = true;
              if (row >= state_len) {
                w.du[j] = kSsspInf;
                bad = true;
              }
            } else if (row < state_len) {
              // A node that already improved during this launch is queued
              // for the next iteration with a distance at least as good, and
              // its arcs are relaxed there: skip them here (du = infinity
              // marks the entry as skipped).  The state never moves back, so
              // a stale read can only miss a skip, never invent one.
              const unsigned long long sv = *at<kNarrow>(static_cast<const unsigned long long*>(a.dstate), row);
              w.du[j] = static_cast<uint32_t>(sv) == L + 1 ? kSsspInf : static_cast<uint32_t>(sv >> 32);
              live = live || static_cast<uint32_t>(sv) != L + 1;
            } else {
              w.du[j] = kSsspInf;
              bad = true;
            }
          }
          const uint32_t s = (p > t0 ? p : t0) - t0;
          atomicOr(&w.flag[s >> 5], 1u << (s & 31));
        }
      }
      if (!__any(valid)) break;
    }
    if (!rr && tnext < ntiles) i0_next = static_cast<uint32_t>(*at<kNarrow>(cur.tile_node, tnext));
    wave_sync();
    if (kSssp && !__any(live) && !__any(bad)) {
      // every entry of the tile improved again this iteration (a hub queued
      // for the next one, typically): nothing to load, the tile ends here
      skip += (t1 - t0 + 63u - lane) / 64u;  // this lane's share of the tile's slots
      wave_sync();
      continue;
    }
    uint32_t nent;  // entries staged for this tile (wave-uniform)
    {
      const uint32_t x = lane < T / 32 ? __popc(w.flag[lane]) : 0u;
      const uint32_t inc = wave_incl_scan(x);
      if (lane < T / 32) w.wpre[lane] = inc - x;
      nent = __shfl(inc, T / 32 - 1, 64);
    }
    wave_sync();
    // a tile inside one entry (a hub's arcs): every slot maps to entry 0,
    // with no per-slot lookups (measured: SSSP 11 % faster on R-MAT 22;
    // batched solves 1 % faster with this and the skipped-tile exit)
    const bool single = nent == 1u;
    uint32_t b0 = 0, d0 = 0;
    if (single) {
      b0 = w.base[0];
      if (kSssp) d0 = w.du[0];
    }

    // Phase A: the arcs of this lane's kItems slots.
    int32_t vv[kItems];
    uint32_t ww[kItems];
    uint32_t du[kItems];
    int32_t dl[kMulti ? kItems : 1];
    int32_t qd[kMulti ? kItems : 1];
    bool inside[kMulti ? kItems : 1];
    bool bfsq[kMulti ? kItems : 1];  // batched: the slot belongs to a BFS query
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
      const uint32_t s = r * 64 + lane;
      vv[r] = -1;
      ww[r] = 0;
      du[r] = 0;
      if (kMulti) {
        dl[kMulti ? r : 0] = 0;
        qd[kMulti ? r : 0] = 0;
        inside[kMulti ? r : 0] = true;
        bfsq[kMulti ? r : 0] = false;
      }
      if (t0 + s < t1) {
        int slot = 0;
        uint32_t e, dslot = d0;
        if (single) {
          e = b0 + s;
        } else {
          const uint32_t k = s >> 5;
          const uint32_t msk = static_cast<uint32_t>((2ull << (s & 31)) - 1ull);
          slot = static_cast<int>(w.wpre[k] + __popc(w.flag[k] & msk)) - 1;
          e = slot >= 0 ? w.base[slot] + s : a.m;
          if (kSssp && slot >= 0) dslot = w.du[slot];
        }
        if (kSssp && slot >= 0 && dslot == kSsspInf) {
          ++skip;  // skipped entry (see staging)
        } else if (e < a.m) {
          if (kPacked) {
            load_arc<true, kNarrow>(a, e, &vv[r], &ww[r]);
          } else {
            vv[r] = *at<kNarrow>(a.cols, e);
          }
          if (kSssp) {
            du[r] = dslot;
            if (kMulti) {
              dl[kMulti ? r : 0] = w.delta[slot];
              qd[kMulti ? r : 0] = w.qid[slot];
              const uint32_t lk = w.lenkind[slot];
              inside[kMulti ? r : 0] =
                  static_cast<uint32_t>(vv[r] - w.lo[slot]) < (lk & 0x7fffffffu);
              bfsq[kMulti ? r : 0] = !(lk >> 31);
              ww[r] = (lk >> 31) ? *at<kNarrow>(a.weights, e) : 1u;
            } else if (!kPacked) {
              ww[r] = *at<kNarrow>(a.weights, e);
            }
          }
        } else {
          bad = true;
        }
      }
    }
    uint32_t row[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
      row[r] = static_cast<uint32_t>(vv[r] + (kMulti ? dl[kMulti ? r : 0] : 0));
      if (vv[r] >= 0 && (static_cast<uint32_t>(vv[r]) >= a.n || row[r] >= state_len ||
                         (kMulti && !inside[kMulti ? r : 0]))) {
        bad = true;  // malformed cols, or an arc leaving its query's instance
        vv[r] = -1;
      }
    }
    bool push[kItems];
    if (!kSssp) {
      // Phase B: this XCD's advisory filter, which holds the frozen visited
      // snapshot (merged in at level start) and the XCD's own claims: one
      // random read per arc; phase C: one atomic per surviving candidate.
      uint32_t x[kItems];
#pragma unroll
      for (int r = 0; r < kItems; ++r) x[r] = vv[r] >= 0 ? *at<kNarrow>(fx, static_cast<uint32_t>(vv[r]) >> 5) : ~0u;
      if (scan) {
        // Scan mode: the filter holds every node reached before this level
        // (k_bfs_prep merged the exact `visited` bitmap into it before the
        // launch), so a clear bit proves the node unreached until now and
        // it gets level L + 1 by a plain store.  Several writers of one
        // node store the same value.  No claim, no push.
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
          const uint32_t bit = 1u << (vv[r] & 31);
          if (vv[r] >= 0 && !(x[r] & bit)) {
            *at<kNarrow>(fx, static_cast<uint32_t>(vv[r]) >> 5) = x[r] | bit;  // fewer repeat stores
            *at<kNarrow>(a.levels, vv[r]) = static_cast<int32_t>(L + 1);
          }
          x[r] = ~0u;  // nothing to push
        }
      } else {
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
          const uint32_t bit = 1u << (vv[r] & 31);
          const bool cand = vv[r] >= 0 && !(x[r] & bit);
          if (cand) {
            *at<kNarrow>(fx, static_cast<uint32_t>(vv[r]) >> 5) = x[r] | bit;  // a lost bit costs one more atomic
            ++atom;
            x[r] = atomicOr(at<kNarrow>(a.visited, static_cast<uint32_t>(vv[r]) >> 5), bit);
          } else {
            x[r] = ~0u;
          }
        }
      }
#pragma unroll
      for (int r = 0; r < kItems; ++r) {
        push[r] = vv[r] >= 0 && !(x[r] & (1u << (vv[r] & 31)));
        if (push[r]) {
          *at<kNarrow>(a.levels, vv[r]) = static_cast<int32_t>(L + 1);
          uint32_t* sw = at<kNarrow>(seen_nxt, static_cast<uint32_t>(vv[r]) >> 5);
          *sw |= 1u << (vv[r] & 31);  // a lost bit only costs an atomic later
          ++upd;
        }
      }
    } else {
      // Phase B: filter distances; phase C: one 64-bit atomicMin per
      // improving arc, returning both the old distance and whether the node
      // is already queued for this iteration.  Batched BFS queries instead
      // read and claim their bit in the per-row bitmap (a BFS node is final
      // when first reached), and write the level straight to their row.
      uint32_t cd[kItems];
#pragma unroll
      for (int r = 0; r < kItems; ++r) {
        cd[r] = 0u;
        if (vv[r] >= 0) {
          if (kMulti && bfsq[kMulti ? r : 0]) cd[r] = *at<kNarrow>(static_cast<const uint32_t*>(a.visited), row[r] >> 5);
          else cd[r] = f16_bound(*at<kNarrow>(static_cast<const uint16_t*>(a.d16), row[r]));
        }
      }
      unsigned long long old[kItems];
#pragma unroll
      for (int r = 0; r < kItems; ++r) {
        const uint32_t alt = du[r] + ww[r];
        old[r] = 0ull;
        if (kMulti && bfsq[kMulti ? r : 0]) {
          const uint32_t bit = 1u << (row[r] & 31);
          if (vv[r] >= 0 && !(cd[r] & bit)) {
            ++atom;
            old[r] = atomicOr(at<kNarrow>(a.visited, row[r] >> 5), bit);
          } else {
            old[r] = bit;
          }
        } else if (vv[r] >= 0 && alt < cd[r]) {
          if (kMulti) {
            ++atom;
            old[r] = atomicMin(at<kNarrow>(a.dstate, row[r]),
                               (static_cast<unsigned long long>(alt) << 32) | (L + 1));
          } else {
            // single solves read the state coherently first (the filter is
            // a plain read and may lag other XCDs' improvements) and issue
            // the atomic only when it can still win: contended atomics on
            // popular nodes cost more than the read (measured on R-MAT 22:
            // 37 % fewer atomics, SSSP 2 % faster)
            old[r] = __hip_atomic_load(at<kNarrow>(a.dstate, row[r]), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
      if (!kMulti) {
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
          const uint32_t alt = du[r] + ww[r];
          if (vv[r] >= 0 && alt < cd[r] && alt < static_cast<uint32_t>(old[r] >> 32)) {
            ++atom;
            old[r] = atomicMin(at<kNarrow>(a.dstate, row[r]),
                               (static_cast<unsigned long long>(alt) << 32) | (L + 1));
          }
        }
      }
#pragma unroll
      for (int r = 0; r < kItems; ++r) {
        const uint32_t alt = du[r] + ww[r];
        if (kMulti && bfsq[kMulti ? r : 0]) {
          const bool won = vv[r] >= 0 && !(static_cast<uint32_t>(old[r]) & (1u << (row[r] & 31)));
          if (won) *at<kNarrow>(a.dist, row[r]) = alt;  // = L + 1, final
          upd += won ? 1u : 0u;
          push[r] = won;
        } else {
          const bool better = vv[r] >= 0 && alt < static_cast<uint32_t>(old[r] >> 32);
          if (better) *at<kNarrow>(a.d16, row[r]) = f16_of(alt);  // filter (see top of file)
          upd += better ? 1u : 0u;
          push[r] = better && static_cast<uint32_t>(old[r]) != L + 1;
          if constexpr (kFar) {
            const uint32_t was = static_cast<uint32_t>(old[r] >> 32);
            if (better && was > thr) {  // it was not queued so far
              push[r] = alt <= thr;
              far_move<kNarrow>(a, static_cast<uint32_t>(vv[r]), was, push[r]);
            }
          }
        }
      }
    }
    if (__any(bad) && lane == 0) atomicOr(&a.ctl->error, kErrBadArc);
    // Single solves push in groups of four rounds (at most 256 nodes, the
    // wave queue's size); a group that would not fit flushes the queue
    // first, so a push-heavy tile pays one reservation per 256 nodes.
    // Batched tiles (four rounds in all) push directly.
    constexpr int kGroup = kMulti ? kItems : 4;
    static_assert(kItems % kGroup == 0 && 64 * kGroup <= kWQ, "push group must fit the wave queue");
#pragma unroll
    for (int r0 = 0; r0 < kItems; r0 += kGroup) {
      if constexpr (!kMulti) {
        uint32_t P = 0;
#pragma unroll
        for (int r = r0; r < r0 + kGroup; ++r) P += static_cast<uint32_t>(__popcll(__ballot(push[r])));
        if (qcount + P > static_cast<uint32_t>(kWQ)) {
          WaveFlush<kPay, T, kNarrow, kSplit> f;
          f.flush(a, w.qv, w.qq, qcount, nxt, nctr);
          qcount = 0;
          wave_sync();
        }
      }
#pragma unroll
      for (int r = r0; r < r0 + kGroup; ++r)
        wq_push<kPay, T, kNarrow, kSplit>(a, w.qv, w.qq, qcount, push[r], vv[r], kMulti ? qd[kMulti ? r : 0] : 0,
                                          nxt, nctr);
    }
    // (single solves flush only when the next group would not fit)
    if (kMulti && qcount >= kWQ / 2) {
      WaveFlush<kPay, T, kNarrow, kSplit> f;
      f.flush(a, w.qv, w.qq, qcount, nxt, nctr);
      qcount = 0;
    }
    wave_sync();
  }

  // Final flush: one reservation for the whole workgroup.
  WaveFlush<kPay, T, kNarrow, kSplit> f;
  f.prepare(a, w.qv, w.qq, qcount);
  if (lane == 0) {
    merge[wid] = f.tot_n;
    merge[kWaves + wid] = f.tot_e;
  }
  __syncthreads();
  uint32_t pn = 0, pe = 0, tn = 0, te = 0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) {
    if (static_cast<uint32_t>(k) < wid) {
      pn += merge[k];
      pe += merge[kWaves + k];
    }
    tn += merge[k];
    te += merge[kWaves + k];
  }
  if (threadIdx.x == 0)
    merge_base = tn ? atomicAdd(&a.ctl->ctr[nctr], (static_cast<unsigned long long>(tn) << 32) | te) : 0ull;
  __syncthreads();
  f.write(a, nxt, static_cast<uint32_t>(merge_base >> 32) + pn, static_cast<uint32_t>(merge_base) + pe);
  add_stats(a, upd, atom, skip);
}

// The level is pulled (lbg_pull.hpp): it is large and the graph has been found
// symmetric.  Grid-uniform once k_bfs_sym has run.
__device__ __forceinline__ bool pulls(const KArgs& a, uint32_t Ef) {
  return a.pull_min != 0u && Ef >= a.pull_min && a.ctl->sym_run != 0u && a.ctl->sym_no == 0u;
}

// Balanced single solves: the level that launch number k of the solve finds
// is known on the device only (a team launch runs any number of them); one
// thread leaves it for the next launch and notes whether this one has work.
__device__ __forceinline__ uint32_t level_of(const KArgs& a, uint32_t k) { return a.team ? a.team->at[k & 1] : k; }
__device__ __forceinline__ void level_next(const KArgs& a, uint32_t k, uint32_t next, bool work) {
  a.team->at[(k + 1) & 1] = next;
  const unsigned long long bit = 1ull << (k & 63);
  a.ctl->worked = work ? a.ctl->worked | bit : a.ctl->worked & ~bit;
}

template <bool kSssp, bool kNarrow, bool kMulti, bool kPacked = false, bool kSplit = false, bool kFar = false>
__device__ __forceinline__ void balanced_level(const KArgs& a, uint32_t k) {
  const uint32_t L = level_of(a, k);
  if (a.team) {
    const uint32_t Ef = static_cast<uint32_t>(ld_agent(&a.ctl->ctr[L % 3]));
    const bool idle = (Ef <= a.min_arcs && !(Ef == 0u && kFar && a.min_arcs == 0u)) ||
                      (kSssp && a.far && kFar != (a.ctl->plain == 0u));  // launched before that was known
    if (blockIdx.x == 0 && threadIdx.x == 0) level_next(a, k, idle ? L : L + 1, !idle);
    if (idle) return;
  }
  const unsigned long long c = level_begin(a, L);
  if (static_cast<uint32_t>(c) == 0u && !kFar) return;
  if (!level_fits<kSssp, kMulti>(a, c)) {
    if (threadIdx.x == 0) atomicOr(&a.ctl->error, kErrNodeCap);
    return;
  }
  if (!kSssp && !kSplit && pulls(a, static_cast<uint32_t>(c))) return;  // k_bfs_pull does the level
  expand_level<kSssp, kNarrow, kMulti, kPacked, kSplit, kFar>(a, L, c);
}

template <bool kSssp, bool kNarrow, bool kMulti = false, bool kPacked = false, bool kSplit = false, bool kFar = false>
__global__ __launch_bounds__(kBlock) void k_expand_balanced(KArgs a, uint32_t k) {
  balanced_level<kSssp, kNarrow, kMulti, kPacked, kSplit, kFar>(a, k);
}

// BFS, before a level that may scan: every XCD's filter absorbs `visited`,
// which is exact (push levels set it with claim atomics, the small-frontier kernel
// too, scan levels by k_bfs_compact's whole-word stores), so in scan mode a
// clear filter bit proves the node unreached before the level and the
// expansion needs no read of the node's level (measured: BFS 2.6 % faster
// on R-MAT 22 than reading it).  Returns at once unless level L scans.
template <bool kNarrow>
__global__ __launch_bounds__(kBlock) void k_bfs_prep(KArgs a, uint32_t k) {
  const uint32_t L = level_of(a, k);
  const unsigned long long c = __hip_atomic_load(&a.ctl->ctr[L % 3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t Ef = static_cast<uint32_t>(c);
  if (Ef <= a.min_arcs || Ef < a.scan_min) return;
  if (a.pull_min)  // a pull level reads the snapshot
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < a.words; i += gridDim.x * kBlock)
      a.seen[L & 1][i] = *at<kNarrow>(a.visited, i);
  const uint32_t total = a.words * kXcds;
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < total; i += gridDim.x * kBlock) {
    const uint32_t v = *at<kNarrow>(a.visited, i % a.words);
    if (v) a.xfilter[i] |= v;
  }
}

constexpr int kCompactBlock = 1024;
// Chunk slot of node j: one pad word per kPer, so that threads reading kPer
// consecutive nodes each hit different LDS banks.
template <uint32_t kPer>
__device__ __forceinline__ uint32_t compact_slot(uint32_t j) { return j + j / kPer; }

// BFS scan levels.  A level of at least a.scan_min arcs is expanded without
// claims or pushes (expand_level, scan mode): every newly reached node gets
// level L + 1 in the levels array.  This kernel, launched behind it, then
// builds worklist L + 1 from the nodes whose level is L + 1 (the worklist of
// Section II-B, made by a scan of the node states instead of by atomic claims; at R-MAT scale 22 a big level issues ~8 M
// claim atomics, at a memory-side rate of ~25 G/s).  Each workgroup takes
// chunks of 1024 x kPer nodes: coalesced loads of the chunk's levels and
// offsets into LDS, then thread t handles nodes kPer t .. kPer (t + 1) - 1 of
// the chunk, so a block scan gives every new node with out-arcs its place in
// node order and one packed atomic reserves the chunk's entries: the next
// level reads the CSR in order.  `visited`, next level's `seen` snapshot and
// every XCD's filter are rewritten from the levels (each 32-node word by one
// thread, plain stores), so a following scan level needs no k_bfs_prep.
// What bounds it: 8 bytes per node read, and the reservations, which all hit
// one address (about 12 ns each).  kPer = 16 where that still gives a chunk to
// every CU (n >= 2^22), else 4.  Against 256 threads and 4096 nodes with a
// k_bfs_prep before every scan level: R-MAT 22, 42 -> 31 us between two big
// levels; 2048 x 2048 grid, 33 -> 17 us.
// Returns at once after a level that pushed, whose pushes already built
// worklist L + 1, after a pulled one and after a launch that had no work.  The
// host launches it behind every expansion of a solve whose levels may scan.
template <bool kNarrow, uint32_t kPer>
__global__ __launch_bounds__(kCompactBlock) void k_bfs_compact(KArgs a, uint32_t launch) {
  const uint32_t L = level_of(a, launch);
  constexpr uint32_t T = TileCfg<false>::kEdges;
  constexpr uint32_t kChunk = kCompactBlock * kPer;
  constexpr uint32_t kSlots = kChunk + kCompactBlock + 1;
  constexpr int kWv = kCompactBlock / 64;
  static_assert(kPer <= 16 && 32 % kPer == 0, "a thread's nodes are part of one bitmap word");
  __shared__ int32_t lvs[kSlots];
  __shared__ int32_t offs[kSlots];
  __shared__ uint32_t wsum[2][kWv];
  __shared__ unsigned long long base_sh;
  const unsigned long long c = __hip_atomic_load(&a.ctl->ctr[L % 3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t Ef = static_cast<uint32_t>(c);
  // push-mode level, or none was run
  if (Ef <= a.min_arcs || Ef < a.scan_min || !level_fits<false, false>(a, c) || pulls(a, Ef)) return;
  Frontier nxt = a.fr[(L + 1) & 1];
  nxt.level = L + 1;
  const int nctr = (L + 1) % 3;
  uint32_t* seen_nxt = a.seen[(L + 1) & 1];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int32_t want = static_cast<int32_t>(L + 1);
  uint32_t upd = 0;
  for (uint32_t c0 = blockIdx.x * kChunk; c0 < a.n; c0 += gridDim.x * kChunk) {
    // the chunk's levels and offsets (offsets of nodes c0 .. c0 + kChunk)
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      const uint32_t j = k * kCompactBlock + tid, v = c0 + j;
      lvs[compact_slot<kPer>(j)] = v < a.n ? *at<kNarrow>(a.levels, v) : 0;
      offs[compact_slot<kPer>(j)] = v <= a.n ? *at<kNarrow>(a.offsets, v) : 0;
    }
    if (tid == 0) {
      const uint32_t v = c0 + kChunk;
      offs[compact_slot<kPer>(kChunk)] = v <= a.n ? *at<kNarrow>(a.offsets, v) : 0;
    }
    __syncthreads();
    // this thread's kPer nodes: which are new, their degrees
    const uint32_t j0 = tid * kPer;
    uint32_t newm = 0, reached = 0, cnt = 0, deg = 0;
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      const uint32_t j = j0 + k;
      const int32_t lv = lvs[compact_slot<kPer>(j)];
      if (c0 + j < a.n && lv != static_cast<int32_t>(kBfsInf)) reached |= 1u << k;
      if (c0 + j < a.n && lv == want) {
        newm |= 1u << k;
        const uint32_t d = static_cast<uint32_t>(offs[compact_slot<kPer>(j + 1)] - offs[compact_slot<kPer>(j)]);
        cnt += d > 0u ? 1u : 0u;
        deg += d;
      }
    }
    upd += __popc(newm);
    // The chunk's 32-node words of `visited`, of next level's `seen` and of
    // every XCD's filter: the nodes of level <= L + 1, which is exactly what
    // the levels say now, so whole words are stored, no read needed.
    uint32_t word = reached << (j0 & 31);
#pragma unroll
    for (uint32_t x = 1; x < 32 / kPer; x <<= 1)
      word |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(word), static_cast<int>(x), 64));
    if ((j0 & 31) == 0u && c0 + j0 < a.n) {
      const uint32_t w = (c0 + j0) >> 5;
      *at<kNarrow>(a.visited, w) = word;
      *at<kNarrow>(seen_nxt, w) = word;
#pragma unroll
      for (int x = 0; x < kXcds; ++x) a.xfilter[static_cast<size_t>(x) * a.words + w] = word;
    }
    // block exclusive scan of (entries, arcs) in node order, one reservation
    const uint32_t ic = wave_incl_scan(cnt), ie = wave_incl_scan(deg);
    if (lane == 63) {
      wsum[0][wid] = ic;
      wsum[1][wid] = ie;
    }
    __syncthreads();
    uint32_t pc = ic - cnt, pe = ie - deg, tc = 0, te = 0;
#pragma unroll
    for (int k = 0; k < kWv; ++k) {
      if (static_cast<uint32_t>(k) < wid) {
        pc += wsum[0][k];
        pe += wsum[1][k];
      }
      tc += wsum[0][k];
      te += wsum[1][k];
    }
    if (tid == 0) base_sh = tc ? atomicAdd(&a.ctl->ctr[nctr], (static_cast<unsigned long long>(tc) << 32) | te) : 0ull;
    __syncthreads();
    const uint32_t nb = static_cast<uint32_t>(base_sh >> 32) + pc;
    uint32_t eb = static_cast<uint32_t>(base_sh) + pe;
    uint32_t i = 0;
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      const uint32_t j = j0 + k;
      if (newm & (1u << k)) {
        const int32_t s = offs[compact_slot<kPer>(j)];
        const int32_t d = offs[compact_slot<kPer>(j + 1)] - s;
        if (d > 0) {
          write_entry<0, T, kNarrow>(a, nxt, nb + i, eb, static_cast<int32_t>(c0 + j), 0, s, d);
          ++i;
          eb += static_cast<uint32_t>(d);
        }
      }
    }
    __syncthreads();  // LDS reused by the next chunk
  }
  if (a.count_stats) {
    const uint32_t su = wave_sum(upd);
    if (lane == 0 && su) atomicAdd(&a.ctl->xstat[blockIdx.x % kXcds][0], static_cast<unsigned long long>(su));
  }
}

// Graph-launched batches: one replay of a graph runs levels level_base + k
// for k = 0 .. K-1, then k_level_advance moves level_base on by K, so the
// same graph, its arguments fixed, serves every replay.
template <bool kNarrow>
__global__ __launch_bounds__(kBlock) void k_expand_batched_graph(KArgs a, uint32_t k) {
  const uint32_t L = __hip_atomic_load(&a.ctl->level_base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + k;
  balanced_level<true, kNarrow, true>(a, L);
}

__global__ void k_level_advance(Ctl* ctl, uint32_t K) {
  if (threadIdx.x == 0 && blockIdx.x == 0) ctl->level_base += K;
}

// ---------------------------------------------------------- node (BS) ----
// Node-based baseline (Section II-A): thread i of the grid-stride loop owns
// worklist entry i and walks all of its arcs; a wave runs for as long as its
// highest-degree node, which is the load imbalance the paper measures.
template <bool kSssp>
__global__ __launch_bounds__(kBlock) void k_expand_node(KArgs a, uint32_t L) {
  __shared__ int32_t qS[kWaves][kQueue];
  __shared__ int32_t qD[kWaves][kQueue];
  __shared__ int32_t qV[kSssp ? kWaves : 1][kQueue];

  const unsigned long long c = level_begin(a, L);
  const uint32_t Ef = static_cast<uint32_t>(c);
  const uint32_t nf = static_cast<uint32_t>(c >> 32);
  if (Ef == 0) return;
  if (nf > a.node_cap || Ef > a.m) {
    if (threadIdx.x == 0) atomicOr(&a.ctl->error, kErrNodeCap);
    return;
  }
  if (!kSssp) refresh_seen(a, L);
  const Frontier cur = a.fr[L & 1];
  const Frontier nxt = a.fr[(L + 1) & 1];
  const int nctr = (L + 1) % 3;
  const uint32_t tid = threadIdx.x;
  const uint32_t wid = tid >> 6;
  WaveQueue<kSssp> q{qS[wid], qD[wid], qV[kSssp ? wid : 0], 0u};
  auto flush = [&]() { q.template flush_nodes<false>(a, nxt, nctr); };
  uint32_t upd = 0, atom = 0;

  for (uint32_t base = blockIdx.x * kBlock; base < nf; base += gridDim.x * kBlock) {
    const uint32_t i = base + tid;
    int32_t s0 = 0, deg = 0;
    uint32_t du = 0;
    if (i < nf) {
      const uint32_t p = cur.eprefix[i];
      const uint32_t pn = (i + 1 < nf) ? cur.eprefix[i + 1] : Ef;
      s0 = cur.estart[i];
      deg = static_cast<int32_t>(pn - p);
      if (static_cast<uint64_t>(static_cast<uint32_t>(s0)) + static_cast<uint32_t>(deg) > a.m) {
        atomicOr(&a.ctl->error, kErrBadArc);
        deg = 0;
      }
      if (kSssp) du = static_cast<uint32_t>(a.dstate[cur.node[i]] >> 32);
    }
    const int32_t dmax = wave_max(deg);
    for (int32_t k = 0; k < dmax; ++k) {
      int32_t v = -1, s = 0, d = 0;
      bool want = false;
      if (k < deg) {
        const int32_t e = s0 + k;
        v = a.cols[e];
        want = relax<kSssp>(a, L, v, du, kSssp ? a.weights[e] : 0u, &upd, &atom, &s, &d);
      }
      q.push(want, s, d, v, flush);
    }
  }
  flush();
  add_stats(a, upd, atom);
}

// ------------------------------------------------------ degree bins ----
// Degree-binned expansion: worklist entries are nodes, or pieces of at most
// a.mdt arcs of a hub (split when pushed; Section III-B's node splitting
// applied to worklist entries instead of the graph).  Each workgroup takes
// 256 consecutive entries at a time and bins them by length: pieces longer
// than t_block are expanded one after another by the whole workgroup,
// longer than t_wave by one wavefront each, the rest by their own lane
// (the thread / wavefront / workgroup cooperation of degree-binned
// load balancing).  Lanes of a cooperating group read consecutive arcs.
constexpr uint32_t kMinMdt = 64;  // smallest split size (bounds entries per level)

template <bool kSssp>
__global__ __launch_bounds__(kBlock) void k_expand_binned(KArgs a, uint32_t L) {
  __shared__ int32_t qS[kWaves][kQueue];
  __shared__ int32_t qD[kWaves][kQueue];
  __shared__ int32_t qV[kSssp ? kWaves : 1][kQueue];
  __shared__ uint32_t bs[2][kBlock], bl[2][kBlock], bdu[2][kSssp ? kBlock : 1];
  __shared__ uint32_t bcount[2];

  const unsigned long long c = level_begin(a, L);
  const uint32_t Ef = static_cast<uint32_t>(c);
  const uint32_t nf = static_cast<uint32_t>(c >> 32);
  if (Ef == 0) return;
  if (nf > a.node_cap || Ef > a.m) {
    if (threadIdx.x == 0) atomicOr(&a.ctl->error, kErrNodeCap);
    return;
  }
  if (!kSssp) refresh_seen(a, L);
  const Frontier cur = a.fr[L & 1];
  const Frontier nxt = a.fr[(L + 1) & 1];
  const int nctr = (L + 1) % 3;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  WaveQueue<kSssp> q{qS[wid], qD[wid], qV[kSssp ? wid : 0], 0u};
  auto flush = [&]() { q.flush_split(a, nxt, nctr); };
  uint32_t upd = 0, atom = 0;

  // relax the arcs [s + k0, s + len) of one entry, k0 + stride*j per lane,
  // kBinB of a lane's arcs at a time (relax_batch); `rounds` is uniform over
  // the lanes that share the entry (wave or workgroup)
  constexpr int kBinB = kSssp ? 4 : 8;  // SSSP: fewer registers per arc in flight (measured)
  auto expand = [&](bool act, uint32_t s, uint32_t len, uint32_t du, uint32_t k0, uint32_t stride,
                    uint32_t rounds) {
    for (uint32_t j0 = 0; j0 < rounds; j0 += kBinB) {
      int32_t v[kBinB], ns[kBinB], nd[kBinB];
      uint32_t w[kBinB], dd[kBinB];
      bool want[kBinB];
#pragma unroll
      for (int b = 0; b < kBinB; ++b) {
        const uint32_t k = k0 + (j0 + b) * stride;
        v[b] = -1;
        w[b] = 0;
        dd[b] = du;
        if (act && j0 + b < rounds && k < len) {
          const uint32_t e = s + k;
          if (e < a.m) {
            v[b] = a.cols[e];
            if (kSssp) w[b] = a.weights[e];
          } else {
            atomicOr(&a.ctl->error, kErrBadArc);
          }
        }
      }
      relax_batch<kSssp, kBinB>(a, L, v, dd, w, &upd, &atom, ns, nd, want);
#pragma unroll
      for (int b = 0; b < kBinB; ++b) q.push(want[b], ns[b], nd[b], v[b], flush);
    }
  };

  for (uint32_t base = blockIdx.x * kBlock; base < nf; base += gridDim.x * kBlock) {
    if (tid < 2) bcount[tid] = 0u;
    __syncthreads();
    const uint32_t i = base + tid;
    uint32_t s = 0, len = 0, du = 0;
    if (i < nf) {
      const uint32_t p = cur.eprefix[i];
      const uint32_t pn = (i + 1 < nf) ? cur.eprefix[i + 1] : Ef;
      s = static_cast<uint32_t>(cur.estart[i]);
      len = pn - p;
      if (static_cast<unsigned long long>(s) + len > a.m) {
        atomicOr(&a.ctl->error, kErrBadArc);
        len = 0;
      }
      if (kSssp) {
        const unsigned long long sv = a.dstate[cur.node[i]];
        // already improved this iteration: relaxed with its better distance next time
        if (static_cast<uint32_t>(sv) == L + 1) len = 0;
        du = static_cast<uint32_t>(sv >> 32);
      }
    }
    // bins: 0 = workgroup, 1 = wavefront, lane otherwise
    const int bin = len > a.t_block ? 0 : (len > a.t_wave ? 1 : 2);
    if (bin < 2) {
      const uint32_t k = atomicAdd(&bcount[bin], 1u);
      bs[bin][k] = s;
      bl[bin][k] = len;
      if (kSssp) bdu[bin][k] = du;
    }
    __syncthreads();
    const uint32_t nb0 = bcount[0], nb1 = bcount[1];
    for (uint32_t k = 0; k < nb0; ++k) {  // workgroup bin, one piece at a time
      const uint32_t l = bl[0][k];
      expand(true, bs[0][k], l, kSssp ? bdu[0][k] : 0u, tid, kBlock, (l + kBlock - 1) / kBlock);
    }
    for (uint32_t k0 = 0; k0 < nb1; k0 += kWaves) {  // wavefront bin
      const uint32_t k = k0 + wid;
      const bool act = k < nb1;
      const uint32_t l = act ? bl[1][k] : 0u;
      const uint32_t r = static_cast<uint32_t>(wave_max(static_cast<int32_t>((l + 63) / 64)));
      expand(act, act ? bs[1][k] : 0u, l, (kSssp && act) ? bdu[1][k] : 0u, lane, 64, r);
    }
    {  // lane bin
      const bool act = bin == 2;
      const uint32_t r = static_cast<uint32_t>(wave_max(static_cast<int32_t>(act ? len : 0u)));
      expand(act, s, len, du, 0, 1, r);
    }
    __syncthreads();
  }
  flush();
  add_stats(a, upd, atom);
}

// -------------------------------------------------- hierarchical (HP) ----
// Hierarchical processing (Section III-C).  Sub-iteration s of a level
// relaxes window [s * mdt, (s + 1) * mdt) of the arcs of every frontier
// node still active, one thread per node; nodes with arcs beyond the window
// form the sublist of sub-iteration s + 1 (appended with one atomic per
// wavefront).  Once a sublist holds fewer than kHierWd nodes, its remaining
// arcs are expanded edge-balanced instead (the hand-over to workload
// decomposition): every block stages the sublist's remaining ranges and
// their prefix in LDS and takes a grid-strided share of the arcs.  The host
// enqueues ceil(maxDegree / mdt) sub-iterations per level; later ones find
// an empty sublist and return.  Sublist counters rotate over three slots:
// sub-iteration s reads sub_cnt[s % 3], appends to sub_cnt[(s + 1) % 3] and
// clears sub_cnt[(s + 2) % 3]; k_hier_reset clears slot 1 before a level.
constexpr uint32_t kHierWd = 1024;

__global__ void k_hier_reset(Ctl* ctl) {
  if (threadIdx.x == 0 && blockIdx.x == 0) ctl->sub_cnt[1] = 0u;
}

template <bool kSssp>
__global__ __launch_bounds__(kBlock) void k_expand_hier(KArgs a, uint32_t L, uint32_t sub, uint32_t mdt) {
  __shared__ int32_t qS[kWaves][kQueue];
  __shared__ int32_t qD[kWaves][kQueue];
  __shared__ int32_t qV[kSssp ? kWaves : 1][kQueue];
  __shared__ uint32_t ws_start[kHierWd], ws_pre[kHierWd], ws_du[kSssp ? kHierWd : 1];
  __shared__ uint32_t wsum[kWaves];

  unsigned long long c;
  if (sub == 0) {
    c = level_begin(a, L);
  } else {
    c = __hip_atomic_load(&a.ctl->ctr[L % 3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const uint32_t Ef = static_cast<uint32_t>(c);
  const uint32_t nf = static_cast<uint32_t>(c >> 32);
  if (Ef == 0) return;
  if (nf > a.node_cap || Ef > a.m) {
    if (threadIdx.x == 0 && sub == 0) atomicOr(&a.ctl->error, kErrNodeCap);
    return;
  }
  const uint32_t cnt = sub == 0 ? nf
                                : __hip_atomic_load(&a.ctl->sub_cnt[sub % 3], __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.ctl->sub_cnt[(sub + 2) % 3] = 0u;
    if (a.hier_trace && cnt && L < kHierTraceLevels && sub < kHierTraceSubs)
      a.hier_trace[L * kHierTraceSubs + sub] = cnt;
  }
  if (cnt == 0) return;
  if (!kSssp && sub == 0) refresh_seen(a, L);
  const Frontier cur = a.fr[L & 1];
  const Frontier nxt = a.fr[(L + 1) & 1];
  const int32_t* in = sub == 0 ? nullptr : a.sub[(sub - 1) & 1];
  int32_t* out = a.sub[sub & 1];
  const int nctr = (L + 1) % 3;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  WaveQueue<kSssp> q{qS[wid], qD[wid], qV[kSssp ? wid : 0], 0u};
  auto flush = [&]() { q.template flush_nodes<false>(a, nxt, nctr); };
  uint32_t upd = 0, atom = 0, skip = 0;
  const unsigned long long w0 = static_cast<unsigned long long>(sub) * mdt;

  // entry e of the level: first arc, degree and (SSSP) current distance;
  // deg = 0 when it was improved again this iteration (relaxed next time:
  // its arcs from this sub-iteration's window on count as skipped, by the
  // one thread that stages the entry for the grid: count_skip)
  auto entry = [&](uint32_t e, uint32_t* st, uint32_t* deg, uint32_t* du, bool count_skip) {
    const uint32_t p = cur.eprefix[e];
    const uint32_t pn = (e + 1 < nf) ? cur.eprefix[e + 1] : Ef;
    *st = static_cast<uint32_t>(cur.estart[e]);
    *deg = pn - p;
    if (static_cast<unsigned long long>(*st) + *deg > a.m) {
      atomicOr(&a.ctl->error, kErrBadArc);
      *deg = 0;
    }
    *du = 0;
    if (kSssp) {
      const unsigned long long sv = a.dstate[cur.node[e]];
      if (static_cast<uint32_t>(sv) == L + 1) {
        if (count_skip) skip += *deg > w0 ? static_cast<uint32_t>(*deg - w0) : 0u;
        *deg = 0;
      }
      *du = static_cast<uint32_t>(sv >> 32);
    }
  };
  auto relax_push = [&](bool act, uint32_t arc, uint32_t du) {
    int32_t v = -1, ns = 0, nd = 0;
    bool want = false;
    if (act) {
      v = a.cols[arc];
      want = relax<kSssp>(a, L, v, du, kSssp ? a.weights[arc] : 0u, &upd, &atom, &ns, &nd);
    }
    q.push(want, ns, nd, v, flush);
  };

  if (cnt >= kHierWd) {
    // one thread per active node: this sub-iteration's window of its arcs
    for (uint32_t base = blockIdx.x * kBlock; base < cnt; base += gridDim.x * kBlock) {
      const uint32_t i = base + tid;
      uint32_t st = 0, deg = 0, du = 0;
      if (i < cnt) entry(sub == 0 ? i : static_cast<uint32_t>(in[i]), &st, &deg, &du, true);
      const unsigned long long lo = w0 < deg ? w0 : deg;
      const unsigned long long hi = (w0 + mdt) < deg ? (w0 + mdt) : deg;
      const uint32_t len = static_cast<uint32_t>(hi - lo);
      const uint32_t rounds = static_cast<uint32_t>(wave_max(static_cast<int32_t>(len)));
      // the window's arcs, kHierB of this thread's at a time (relax_batch)
      constexpr int kHierB = kSssp ? 4 : 8;
      for (uint32_t k0 = 0; k0 < rounds; k0 += kHierB) {
        int32_t v[kHierB], ns[kHierB], nd[kHierB];
        uint32_t w[kHierB], dd[kHierB];
        bool want[kHierB];
#pragma unroll
        for (int b = 0; b < kHierB; ++b) {
          v[b] = -1;
          w[b] = 0;
          dd[b] = du;
          if (k0 + b < len) {
            const uint32_t arc = st + static_cast<uint32_t>(lo) + k0 + b;
            v[b] = a.cols[arc];
            if (kSssp) w[b] = a.weights[arc];
          }
        }
        relax_batch<kSssp, kHierB>(a, L, v, dd, w, &upd, &atom, ns, nd, want);
#pragma unroll
        for (int b = 0; b < kHierB; ++b) q.push(want[b], ns[b], nd[b], v[b], flush);
      }
      // arcs beyond the window: the node stays active
      const bool more = i < cnt && deg > w0 + mdt;
      const uint64_t mask = __ballot(more);
      if (mask) {
        uint32_t b = 0;
        if (lane == 0) b = atomicAdd(&a.ctl->sub_cnt[(sub + 1) % 3], static_cast<uint32_t>(__popcll(mask)));
        b = __shfl(b, 0, 64);
        if (more) {
          const uint32_t k = b + lane_rank(mask);
          if (k < a.node_cap) out[k] = static_cast<int32_t>(sub == 0 ? i : static_cast<uint32_t>(in[i]));
          else atomicOr(&a.ctl->error, kErrNodeCap);
        }
      }
    }
  } else {
    // hand-over: all remaining arcs of the (< kHierWd) active nodes, balanced
    // (every workgroup stages every entry; workgroup 0 counts the skips)
    uint32_t st = 0, deg = 0, du = 0;
    for (uint32_t j = tid; j < kHierWd; j += kBlock) {
      uint32_t rem = 0, s0 = 0, d0 = 0;
      if (j < cnt) {
        entry(sub == 0 ? j : static_cast<uint32_t>(in[j]), &st, &deg, &du, blockIdx.x == 0);
        rem = deg > w0 ? static_cast<uint32_t>(deg - w0) : 0u;
        s0 = st + static_cast<uint32_t>(deg > w0 ? w0 : deg);
        d0 = du;
      }
      ws_start[j] = s0;
      ws_pre[j] = rem;  // lengths for now, prefix below
      if (kSssp) ws_du[j] = d0;
    }
    __syncthreads();
    // exclusive prefix of the kHierWd lengths (4 per thread)
    uint32_t v[kHierWd / kBlock], tsum = 0;
#pragma unroll
    for (uint32_t r = 0; r < kHierWd / kBlock; ++r) {
      v[r] = ws_pre[tid * (kHierWd / kBlock) + r];
      tsum += v[r];
    }
    const uint32_t inc = wave_incl_scan(tsum);
    if (lane == 63) wsum[wid] = inc;
    __syncthreads();
    uint32_t before = inc - tsum, total = 0;
    for (uint32_t w = 0; w < kWaves; ++w) {
      if (w < wid) before += wsum[w];
      total += wsum[w];
    }
#pragma unroll
    for (uint32_t r = 0; r < kHierWd / kBlock; ++r) {
      ws_pre[tid * (kHierWd / kBlock) + r] = before;
      before += v[r];
    }
    __syncthreads();
    const uint32_t ne = cnt;  // entries with a range (zero lengths are skipped by the search)
    const uint32_t stride = gridDim.x * kBlock;
    const uint32_t rounds = (total + stride - 1) / stride;
    for (uint32_t r = 0; r < rounds; ++r) {
      const uint32_t e = r * stride + blockIdx.x * kBlock + tid;
      bool act = e < total;
      uint32_t arc = 0, d = 0;
      if (act) {
        uint32_t lo = 0, hi = ne;  // last entry with prefix <= e
        while (hi - lo > 1) {
          const uint32_t mid = (lo + hi) >> 1;
          if (ws_pre[mid] <= e) lo = mid;
          else hi = mid;
        }
        arc = ws_start[lo] + (e - ws_pre[lo]);
        d = kSssp ? ws_du[lo] : 0u;
      }
      relax_push(act, arc, d);
    }
  }
  flush();
  add_stats(a, upd, atom, skip);
}

// ---------------------------------------------------------- edge (EP) ----
// Edge-based baseline (Section II-B): the worklist holds arc ids; thread i of
// the grid-stride loop relaxes arc wl[i] (SSSP reads its source from the COO
// array); a node whose value improved pushes all of its arcs, reserved with
// one atomic per wave batch (work chunking).
//
// kChunk = false is the ablation without work chunking (Section IV-D): an
// improved node reserves each of its arcs with its own atomic on the tail.
template <bool kSssp, bool kChunk>
__global__ __launch_bounds__(kBlock) void k_expand_edge(KArgs a, uint32_t L) {
  __shared__ int32_t qS[kWaves][kQueue];
  __shared__ int32_t qD[kWaves][kQueue];

  const unsigned long long c = level_begin(a, L);
  const uint32_t cnt = static_cast<uint32_t>(c);
  if (cnt == 0) return;
  if (cnt > a.edge_cap) {
    if (threadIdx.x == 0) atomicOr(&a.ctl->error, kErrEdgeCap);
    return;
  }
  if (!kSssp) refresh_seen(a, L);
  const int32_t* wl = a.fr[L & 1].node;
  int32_t* nwl = a.fr[(L + 1) & 1].node;
  const int nctr = (L + 1) % 3;
  const uint32_t tid = threadIdx.x;
  const uint32_t wid = tid >> 6;
  WaveQueue<false> q{qS[wid], qD[wid], nullptr, 0u};
  auto flush = [&]() { q.flush_edges(a, nwl, nctr); };
  uint32_t upd = 0, atom = 0;

  for (uint32_t base = blockIdx.x * kBlock; base < cnt; base += gridDim.x * kBlock) {
    const uint32_t i = base + tid;
    int32_t s = 0, d = 0;
    bool want = false;
    if (i < cnt) {
      const int32_t e = wl[i];
      const int32_t v = static_cast<uint32_t>(e) < a.m ? a.cols[e] : -1;
      uint32_t du = 0, w = 0;
      if (kSssp) {
        du = static_cast<uint32_t>(a.dstate[a.coo_src[e]] >> 32);
        w = a.weights[e];
      }
      want = relax<kSssp>(a, L, v, du, w, &upd, &atom, &s, &d);
    }
    if (kChunk) {
      q.push(want, s, d, 0, flush);
    } else if (want) {
      for (int32_t t = 0; t < d; ++t) {
        const uint32_t p = static_cast<uint32_t>(atomicAdd(&a.ctl->ctr[nctr], 1ull));
        if (p < a.edge_cap) nwl[p] = s + t;
        else atomicOr(&a.ctl->error, kErrEdgeCap);
      }
    }
  }
  flush();
  add_stats(a, upd, atom);
}

// Batched rows.  SSSP rows keep the packed state; BFS rows keep one bit per
// row in the row bitmap (`visited`) and their level in the output row.  Fill
// and finish kernels run a 2-D grid: y walks the queries, x the kRowChunk
// element chunks of a query's row, so a large instance is spread over many
// workgroups.  Bitmap words that a chunk shares with a neighbouring chunk or
// row range are cleared with an atomic AND.
constexpr uint32_t kRowChunk = 4096;

// Queries that one workgroup solves alone (lbg_solo.hpp), by the LDS words
// their state takes: classes 1 and 2, BFS with a bit per node; 3 and 4, SSSP
// with a word per node.  Class 0: the shared worklist.
constexpr uint32_t kSoloWords[5] = {0u, 8192u, 32768u, 8192u, 32768u};
__device__ __forceinline__ bool query_arcs(const KArgs& a, const QInfo& qi, uint32_t* arcs) {
  const int32_t lo = qi.row_start - qi.delta;
  const int32_t s = a.offsets[lo], e = a.offsets[lo + qi.row_len];
  *arcs = static_cast<uint32_t>(e - s);
  return s >= 0 && e >= s && static_cast<uint32_t>(e) <= a.m;
}
__device__ __forceinline__ int solo_class(const KArgs& a, const QInfo& qi) {
  const uint32_t len = static_cast<uint32_t>(qi.row_len);
  const uint32_t words = qi.kind ? len : (len + 31) / 32;
  if (a.solo == 0u || words > kSoloWords[2]) return 0;
  const uint32_t limit = a.ctl->solo_limit;
  uint32_t arcs;
  if (limit == 0u || !query_arcs(a, qi, &arcs) || arcs > limit) return 0;
  return (qi.kind ? 3 : 1) + (words > kSoloWords[1] ? 1 : 0);
}

// One workgroup gets through 0.6 to 1.2 G arcs/s, the chip through about 200
// when it has several for every CU: batches of 2^29 arcs and more take their
// small queries that way (2,048 queries over 2.6 G arcs: the 1,024 BFS queries
// 20 -> 6.8 ms), except those with more than a 256th of the batch, which would
// hold it up.  Smaller batches are done sooner in the shared worklist; shared
// against alone, in ms: 2^25.2 arcs 1.53 / 2.38, 2^27.3 5.38 / 7.03, 2^28.2
// 11.6 / 13.1, 2^29.7 25.2 / 23.5, 2^31.1 65.3 / 53.9.  The arcs are those of
// the batch's instances (one pass over the query table, 1,024 threads); the
// caller's bound on them only says whether it is worth asking.
constexpr unsigned long long kSoloBatch = 1ull << 29;
__global__ __launch_bounds__(1024) void k_solo_limit(KArgs a) {
  __shared__ unsigned long long total;
  if (threadIdx.x == 0) total = 0ull;
  __syncthreads();
  unsigned long long sum = 0;
  for (uint32_t q = threadIdx.x; q < a.num_queries; q += 1024) {
    uint32_t arcs;
    if (query_arcs(a, a.qtab[q], &arcs)) sum += arcs;
  }
  atomicAdd(&total, sum);
  __syncthreads();
  if (threadIdx.x == 0)
    a.ctl->solo_limit =
        total < kSoloBatch ? 0u : static_cast<uint32_t>(min(total / 256ull, static_cast<unsigned long long>(0x7fffffffu)));
}

__device__ __forceinline__ void fill_chunk(const KArgs& a, const QInfo& qi, uint32_t c0) {
  const uint32_t r0 = static_cast<uint32_t>(qi.row_start) + c0;
  const uint32_t r1 = static_cast<uint32_t>(qi.row_start) + min(static_cast<uint32_t>(qi.row_len), c0 + kRowChunk);
  for (uint32_t idx = r0 + threadIdx.x; idx < r1; idx += kBlock) {
    if (qi.kind) {
      a.dstate[idx] = static_cast<unsigned long long>(kSsspInf) << 32;
      a.d16[idx] = static_cast<uint16_t>(kF16None);
    }
    a.dist[idx] = kSsspInf;
  }
  if (!qi.kind) {
    const uint32_t w0 = r0 >> 5, w1 = (r1 - 1) >> 5;
    for (uint32_t w = w0 + threadIdx.x; w <= w1; w += kBlock) {
      const uint32_t lo = w == w0 ? (r0 & 31) : 0u;
      const uint32_t hi = w == w1 ? ((r1 - 1) & 31) : 31u;
      const uint32_t m = (hi == 31u ? ~0u : ((2u << hi) - 1u)) & ~((1u << lo) - 1u);
      if (m == ~0u) a.visited[w] = 0u;
      else atomicAnd(&a.visited[w], ~m);
    }
  }
}

__device__ __forceinline__ void finish_chunk(const KArgs& a, const QInfo& qi, uint32_t c0) {
  const uint32_t r0 = static_cast<uint32_t>(qi.row_start) + c0;
  const uint32_t r1 = static_cast<uint32_t>(qi.row_start) + min(static_cast<uint32_t>(qi.row_len), c0 + kRowChunk);
  for (uint32_t idx = r0 + threadIdx.x; idx < r1; idx += kBlock) {
    if (qi.kind) a.dist[idx] = static_cast<uint32_t>(a.dstate[idx] >> 32);
    else if (a.dist[idx] == kSsspInf) a.dist[idx] = kBfsInf;
  }
}

__device__ __forceinline__ void seed_row(const KArgs& a, const QInfo& qi) {
  const uint32_t row = static_cast<uint32_t>(qi.src + qi.delta);
  if (qi.kind) {
    a.dstate[row] = 0ull;
    a.d16[row] = 0;
  } else atomicOr(&a.visited[row >> 5], 1u << (row & 31));
  a.dist[row] = 0u;
}

__global__ __launch_bounds__(kBlock) void k_batch_fill(KArgs a) {
  for (uint32_t q = blockIdx.y; q < a.num_queries; q += gridDim.y) {
    const QInfo qi = a.qtab[q];
    if (solo_class(a, qi)) continue;
    for (uint32_t c0 = blockIdx.x * kRowChunk; c0 < static_cast<uint32_t>(qi.row_len); c0 += gridDim.x * kRowChunk)
      fill_chunk(a, qi, c0);
  }
  if (blockIdx.x == 0 && blockIdx.y == 0) {
    if (threadIdx.x == 0) {
      a.ctl->ctr[0] = a.ctl->ctr[1] = a.ctl->ctr[2] = 0ull;
      a.ctl->error = 0u;
      a.ctl->levels = 0u;
      a.ctl->level_base = 0u;
      a.ctl->solo_levels = 0u;
      a.ctl->frontier_entries = 0ull;
      a.ctl->edges_scanned = 0ull;
    }
    for (uint32_t k = threadIdx.x; k < kXcds * 16; k += kBlock) a.ctl->xstat[k / 16][k % 16] = 0ull;
  }
}

// Each query's source gets distance 0 and (query, source) enters worklist 0.
template <bool kNarrow>
__global__ __launch_bounds__(kBlock) void k_batch_seed(KArgs a) {
  const uint32_t q = blockIdx.x * kBlock + threadIdx.x;
  bool act = q < a.num_queries;
  int32_t v = 0;
  if (act) {
    const QInfo qi = a.qtab[q];
    v = qi.src;
    act = solo_class(a, qi) == 0;
    if (act) seed_row(a, qi);
  }
  Frontier f0 = a.fr[0];
  f0.level = 0;
  wave_append<2, kMultiTile, kNarrow>(a, act, v, static_cast<int32_t>(q), f0, 0);
}

// ------------------------------------------------------------------ engine --
// Continuous batching: queries join a running batch between levels.  Rows of
// the admitted queries start at infinity ...
__global__ __launch_bounds__(kBlock) void k_engine_fill(KArgs a, const QInfo* stage, QInfo* qtab,
                                                        int count) {
  for (int k = blockIdx.y; k < count; k += gridDim.y) {
    const QInfo qi = stage[k];
    if (blockIdx.x == 0 && threadIdx.x == 0) qtab[qi.slot] = qi;  // read there by later kernels
    for (uint32_t c0 = blockIdx.x * kRowChunk; c0 < static_cast<uint32_t>(qi.row_len); c0 += gridDim.x * kRowChunk)
      fill_chunk(a, qi, c0);
  }
}

// ... then each source gets distance 0 and joins worklist L, the next one to
// be expanded (appending to it exactly like a push of the previous level).
template <bool kNarrow>
__global__ __launch_bounds__(kBlock) void k_engine_seed(KArgs a, const QInfo* stage, int count,
                                                        uint32_t L) {
  const int k = blockIdx.x * kBlock + threadIdx.x;
  const bool act = k < count;
  int32_t v = 0, q = 0;
  if (act) {
    const QInfo qi = stage[k];
    q = qi.slot;
    v = qi.src;
    seed_row(a, qi);
    a.qlast[q] = L;  // even a source without out-arcs is live until level L ends
  }
  Frontier f = a.fr[L & 1];
  f.level = L;
  wave_append<2, kMultiTile, kNarrow>(a, act, v, q, f, static_cast<int>(L % 3));
}

// After a step's levels: rows of queries that no worklist from level L on holds
// are written out (as k_batch_finish), and the control block and every slot's
// last level go to pinned host memory.  The rows, the two read-backs and the
// list of finished slots used to be four copies and two waits of the host,
// most of what a step of small queries took (48 requests in 24 slots: 1.72 ->
// 1.47 ms).  k_engine_idle then marks the finished slots, so that the
// next step does not write their rows again.
__global__ __launch_bounds__(kBlock) void k_engine_finish(KArgs a, uint32_t L, uint32_t* host_last, Ctl* host) {
  if (blockIdx.x == 0 && blockIdx.y == 0) {
    constexpr uint32_t kN = sizeof(Ctl) / sizeof(unsigned long long);
    for (uint32_t k = threadIdx.x; k < kN; k += kBlock)
      reinterpret_cast<unsigned long long*>(host)[k] = reinterpret_cast<const unsigned long long*>(a.ctl)[k];
    for (uint32_t q = threadIdx.x; q < a.num_queries; q += kBlock) host_last[q] = a.qlast[q];
  }
  if (a.ctl->error) return;
  for (uint32_t q = blockIdx.y; q < a.num_queries; q += gridDim.y) {
    if (a.qlast[q] >= L) continue;  // running, or not in use
    const QInfo qi = a.qtab[q];
    for (uint32_t c0 = blockIdx.x * kRowChunk; c0 < static_cast<uint32_t>(qi.row_len); c0 += gridDim.x * kRowChunk)
      finish_chunk(a, qi, c0);
  }
}
__global__ __launch_bounds__(kBlock) void k_engine_idle(KArgs a, uint32_t L) {
  for (uint32_t q = threadIdx.x; q < a.num_queries; q += kBlock)
    if (a.qlast[q] < L) a.qlast[q] = kQIdle;
}

// Once worklist L is empty, each row is written out: SSSP rows as distances,
// BFS rows as int32 levels (INT32_MAX for unreached).  L = UINT32_MAX: the
// level is ctl->level_base (graph-launched batches).
__global__ __launch_bounds__(kBlock) void k_batch_finish(KArgs a, uint32_t L) {
  if (L == 0xffffffffu) L = __hip_atomic_load(&a.ctl->level_base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned long long c = __hip_atomic_load(&a.ctl->ctr[L % 3], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
  if (static_cast<uint32_t>(c) != 0u) return;
  for (uint32_t q = blockIdx.y; q < a.num_queries; q += gridDim.y) {
    const QInfo qi = a.qtab[q];
    if (solo_class(a, qi)) continue;
    for (uint32_t c0 = blockIdx.x * kRowChunk; c0 < static_cast<uint32_t>(qi.row_len); c0 += gridDim.x * kRowChunk)
      finish_chunk(a, qi, c0);
  }
}

// ------------------------------------------------------ MDT histogram --
// Out-degree histogram for the MDT rule of Section III-B: maximum degree,
// then counts of 10 bins of width maxDegree/10 numbered from 1 (bin of
// degree d: max(1, ceil(10 d / maxDegree))), summed per workgroup in LDS and
// added to per-XCD lines (xstat[x][bin - 1]).
constexpr int kMdtBins = 10;

__global__ __launch_bounds__(kBlock) void k_deg_clear(Ctl* ctl) {
  if (threadIdx.x == 0) ctl->deg_max = 0u;
  for (int k = threadIdx.x; k < kXcds * 16; k += kBlock) ctl->xstat[k / 16][k % 16] = 0ull;
}

__global__ __launch_bounds__(kBlock) void k_deg_max(const int32_t* offsets, uint32_t n, Ctl* ctl) {
  uint32_t mx = 0;
  for (uint32_t v = blockIdx.x * kBlock + threadIdx.x; v < n; v += gridDim.x * kBlock)
    mx = max(mx, static_cast<uint32_t>(offsets[v + 1] - offsets[v]));
  mx = static_cast<uint32_t>(wave_max(static_cast<int32_t>(mx)));
  if (lane_id() == 0 && mx) atomicMax(&ctl->deg_max, mx);
}

__global__ __launch_bounds__(kBlock) void k_deg_hist(const int32_t* offsets, uint32_t n, Ctl* ctl) {
  __shared__ uint32_t h[kMdtBins];
  if (threadIdx.x < kMdtBins) h[threadIdx.x] = 0u;
  __syncthreads();
  const unsigned long long mx = ctl->deg_max;
  for (uint32_t v = blockIdx.x * kBlock + threadIdx.x; v < n; v += gridDim.x * kBlock) {
    const unsigned long long d = static_cast<uint32_t>(offsets[v + 1] - offsets[v]);
    unsigned long long b = mx ? (d * kMdtBins + mx - 1) / mx : 1ull;
    if (b < 1) b = 1;
    if (b > kMdtBins) b = kMdtBins;
    atomicAdd(&h[b - 1], 1u);
  }
  __syncthreads();
  if (threadIdx.x < kMdtBins && h[threadIdx.x])
    atomicAdd(&ctl->xstat[blockIdx.x % kXcds][threadIdx.x], static_cast<unsigned long long>(h[threadIdx.x]));
}

// ------------------------------------------------------- CSR validation --
__global__ __launch_bounds__(kBlock) void k_validate(const int32_t* offsets, const int32_t* cols,
                                                     uint32_t n, uint32_t m, Ctl* ctl) {
  const uint32_t gid = blockIdx.x * kBlock + threadIdx.x;
  const uint32_t stride = gridDim.x * kBlock;
  uint32_t flags = 0;
  if (gid == 0) {
    if (offsets[0] != 0) flags |= 1u;
    if (offsets[n] != static_cast<int32_t>(m)) flags |= 4u;
  }
  for (uint32_t u = gid; u < n; u += stride)
    if (offsets[u + 1] < offsets[u]) flags |= 2u;
  for (uint32_t e = gid; e < m; e += stride)
    if (cols[e] < 0 || static_cast<uint32_t>(cols[e]) >= n) flags |= 8u;
  if (flags) atomicOr(&ctl->csr_flags, flags);
}

// ------------------------------------------------------- packed arcs --
// Largest weight (into ctl->deg_max), then the packed words
// (cols[e] << wbits) | weights[e].
__global__ __launch_bounds__(kBlock) void k_weight_max(const uint32_t* weights, uint32_t m, Ctl* ctl) {
  uint32_t mx = 0u;
  for (uint32_t e = blockIdx.x * kBlock + threadIdx.x; e < m; e += gridDim.x * kBlock) mx = max(mx, weights[e]);
  mx = static_cast<uint32_t>(wave_max(static_cast<int32_t>(mx ^ 0x80000000u))) ^ 0x80000000u;  // unsigned max
  if (lane_id() == 0 && mx) atomicMax(&ctl->deg_max, mx);
}

// Source node of every arc (the COO array the edge-based strategy reads,
// Section II-B): wavefront w of the grid writes the arcs of nodes w, w + W,
// ..., 64 consecutive positions per store, so hubs cost many stores of one
// wavefront but every store is coalesced.  Offsets outside [0, m] are
// clamped (lbg_validate_csr first on untrusted input).
__global__ __launch_bounds__(kBlock) void k_coo_sources(const int32_t* offsets, uint32_t n, uint32_t m,
                                                        int32_t* coo) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t W = gridDim.x * kWaves;
  for (uint32_t u = blockIdx.x * kWaves + (threadIdx.x >> 6); u < n; u += W) {
    const int32_t s0 = offsets[u], s1 = offsets[u + 1];
    const uint32_t b = static_cast<uint32_t>(s0 < 0 ? 0 : s0), e = min(static_cast<uint32_t>(s1 < 0 ? 0 : s1), m);
    for (uint32_t k = b + lane; k < e; k += 64) coo[k] = static_cast<int32_t>(u);
  }
}

__global__ __launch_bounds__(kBlock) void k_pack_arcs(const int32_t* cols, const uint32_t* weights, uint32_t m,
                                                      uint32_t wbits, uint32_t* arcs) {
  for (uint32_t e = blockIdx.x * kBlock + threadIdx.x; e < m; e += gridDim.x * kBlock)
    arcs[e] = (static_cast<uint32_t>(cols[e]) << wbits) | weights[e];
}

}  // namespace lbg
