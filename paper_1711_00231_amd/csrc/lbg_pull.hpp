// Pull levels of balanced BFS on symmetric graphs.
//
// On a skewed graph the one or two largest levels hold nearly all arcs, and
// nearly all of those arcs point at nodes reached before: R-MAT scale 22
// expands 125 M arcs in two levels to find 2.4 M nodes, one random read of
// the filter each (about 170 G arcs/s).  If every arc u -> v has its reverse,
// an unreached node can look for a reached one among its own arcs instead and
// stop at the first (Beamer, Asanovic, Patterson 2012): any reached neighbour
// of a node that is unreached after level L has level L.  Most find one among
// their first few arcs.
//
// The caller's CSR is any directed graph, so symmetry is established in the
// solve, and only when a level is about to be pulled:
//  * k_init samples arcs to nodes of few arcs; one without its reverse settles
//    the matter (almost all directed graphs stop here);
//  * k_bfs_sym then reads every arc once, in order (a streaming pass, 4 bytes
//    per arc), and compares the products of lbg_sym.hpp at two random points.
//    A graph that does not pass is expanded as before.
// R-MAT 22: 0.98 -> 0.47 ms for the solve, of which the pass over 513 MB of
// arcs takes about 185 us (2.8 TB/s; 163 - 176 us when it summed a 64-bit hash,
// which a family of directed graphs could make zero) and the two pulled levels
// about 74 + 35 us, where expansion and compaction took 265 + 582 us; R-MAT 24:
// 4.28 -> 1.41 ms.  A graph that is symmetric but for a few arcs pays for the
// pass and has no pulled level (R-MAT 22 less three arcs: 1.07 -> 1.21 ms).
#pragma once

#include <type_traits>

#include "lbg_kernels.hpp"
#include "lbg_sym.hpp"

namespace lbg {

constexpr int kPullBlock = 512;
constexpr uint32_t kPullPer = 8;  // nodes per thread and chunk
constexpr uint32_t kPullChunk = kPullBlock * kPullPer;
constexpr uint32_t kPullAlone = 32;  // arcs a lane tries before its wavefront helps
constexpr uint32_t kSymItems = 16;   // arcs per lane of a tile of k_bfs_sym
constexpr uint32_t kSymTile = 64 * kSymItems;

// The products of a workgroup's threads, in thread 0.  Begins and ends with
// the use of `sums`: two calls need a barrier in between.
__device__ __forceinline__ void sym_block(SymProducts& s, double (&sums)[kWaves][2 * kSymPoints]) {
  const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  double up[kSymPoints], down[kSymPoints];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const int l = static_cast<int>(lane ^ d);
#pragma unroll
    for (int i = 0; i < kSymPoints; ++i) {
      up[i] = __builtin_bit_cast(double, bcast64(__builtin_bit_cast(unsigned long long, s.up[i]), l));
      down[i] = __builtin_bit_cast(double, bcast64(__builtin_bit_cast(unsigned long long, s.down[i]), l));
    }
    sym_join(s, up, down);
  }
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < kSymPoints; ++i) {
      sums[wid][2 * i] = s.up[i];
      sums[wid][2 * i + 1] = s.down[i];
    }
  }
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < kWaves; ++w) {
      for (int i = 0; i < kSymPoints; ++i) {
        up[i] = sums[w][2 * i];
        down[i] = sums[w][2 * i + 1];
      }
      sym_join(s, up, down);
    }
}

// Launched before the solve's one-level launches; does its pass once, before
// the first level that is large enough to be pulled.  What bounds it: reading
// cols in order.  Each wavefront takes one contiguous range of arcs, so it
// looks its first node up once and then walks offsets and arcs together;
// the arcs of 64 x 16 slots are mapped to nodes through an LDS bitmask of
// node starts (one word per 64 slots, so a wavefront-wide uniform read).
template <bool kNarrow>
__global__ __launch_bounds__(kBlock) void k_bfs_sym(KArgs a, uint32_t launch) {
  __shared__ unsigned long long flag_s[kWaves][kSymItems];
  __shared__ uint32_t node_s[kWaves][kSymTile + 1];
  __shared__ double sums[kWaves][2 * kSymPoints];
  __shared__ uint32_t last;
  const uint32_t L = level_of(a, launch);
  const uint32_t Ef = static_cast<uint32_t>(ld_agent(&a.ctl->ctr[L % 3]));
  if (Ef < a.pull_min || Ef <= a.min_arcs || a.ctl->sym_no != 0u) return;
  const uint32_t run = a.ctl->sym_run;
  if (run != 0u && run != launch + 1u) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) a.ctl->sym_run = launch + 1u;
  const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  unsigned long long* flag = flag_s[wid];
  uint32_t* nodes = node_s[wid];
  // whole tiles per wavefront
  const unsigned long long tiles = (static_cast<unsigned long long>(a.m) + kSymTile - 1) / kSymTile;
  const unsigned long long W = static_cast<unsigned long long>(gridDim.x) * kWaves;
  const unsigned long long g = static_cast<unsigned long long>(blockIdx.x) * kWaves + wid;
  const uint32_t t0 = static_cast<uint32_t>(tiles * g / W), t1 = static_cast<uint32_t>(tiles * (g + 1) / W);
  SymProducts prod;
  int32_t swapped = 0;
  sym_start(prod);
  const double x[kSymPoints] = {a.sym_x[0], a.sym_x[1]};
  bool bad = false;
  if (t0 < t1) {
    // the node that holds the range's first arc: the last with offset <= e
    uint32_t lo = 0, hi = a.n;  // offsets[lo] <= e < offsets[hi] (or hi = n)
    {
      const uint32_t e = t0 * kSymTile;
      while (hi - lo > 1) {
        const uint32_t step = (hi - lo + 63) / 64;
        const uint32_t i = lo + lane * step;
        const bool le = i < hi && static_cast<uint32_t>(*at<kNarrow>(a.offsets, i)) <= e;
        const uint32_t ranks = static_cast<uint32_t>(__popcll(__ballot(le)));
        if (ranks == 0u) break;  // malformed offsets
        lo += (ranks - 1) * step;
        hi = min(hi, lo + step);
      }
    }
    uint32_t next = lo + 1;  // next node to place
    if (lane == 0) nodes[0] = lo;
    for (uint32_t t = t0; t < t1; ++t) {
      const uint32_t e0 = t * kSymTile, e1 = min(e0 + kSymTile, a.m);
      if (lane < kSymItems) flag[lane] = 0ull;
      wave_sync();
      // the nodes that start in this tile, in order, behind the one that holds
      // its first arc unless another starts there
      uint32_t found = 0;
      for (;;) {
        const uint32_t i = next + lane;
        const uint32_t s = i < a.n ? static_cast<uint32_t>(*at<kNarrow>(a.offsets, i)) : 0xffffffffu;
        const uint32_t f = i < a.n ? static_cast<uint32_t>(*at<kNarrow>(a.offsets, i + 1)) : 0xffffffffu;
        const bool in = s < e1;  // offsets do not decrease: a prefix of the lanes
        const bool put = in && s >= e0 && f > s;
        const uint64_t puts = __ballot(put);
        if (put) {
          atomicOr(&flag[(s - e0) >> 6], 1ull << ((s - e0) & 63));
          const uint32_t k = found + lane_rank(puts);
          if (k < kSymTile) nodes[1 + k] = i;  // as many as there are slots, at most
        }
        found += static_cast<uint32_t>(__popcll(puts));
        const uint32_t k = static_cast<uint32_t>(__popcll(__ballot(in)));
        next += k;
        if (k < 64u) break;
      }
      wave_sync();
      const unsigned long long words = flag[lane % kSymItems];
      uint32_t before = 0;  // nodes that start before the word
      // all but the last tile are full, and need no bounds
      auto arcs = [&](auto full) {
        constexpr bool kFull = decltype(full)::value;
        const int32_t* cols = at<kNarrow>(a.cols, e0 + lane);
        uint32_t uu[kSymItems], vv[kSymItems];
#pragma unroll
        for (uint32_t r = 0; r < kSymItems; ++r)
          vv[r] = kFull || e0 + r * 64 + lane < e1 ? static_cast<uint32_t>(cols[r * 64]) : 0u;
#pragma unroll
        for (uint32_t r = 0; r < kSymItems; ++r) {
          const uint32_t w0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(words), r));
          const uint32_t w1 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(words >> 32), r));
          // starts up to this lane's slot: the word's first bit, and those
          // below the lane among the others
          uu[r] = nodes[__builtin_amdgcn_mbcnt_hi(w1 >> 1, __builtin_amdgcn_mbcnt_lo(w0 >> 1 | w1 << 31,
                                                                                    before + (w0 & 1u)))];
          before += static_cast<uint32_t>(__popc(w0) + __popc(w1));
        }
#pragma unroll
        for (uint32_t r = 0; r < kSymItems; ++r) {
          const uint32_t u = uu[r], v = vv[r];
          const bool in = kFull || e0 + r * 64 + lane < e1;
          bad = bad || (in && v >= a.n);  // its product is of no use then
          if (in && u != v) {
            const int32_t side = static_cast<int32_t>(v - u);  // negative: v < u
            sym_take(prod, (side ^ swapped) < 0, min(u, v), max(u, v), x);
            swapped = side;
          }
        }
      };
      if (e1 - e0 == kSymTile) arcs(std::true_type{});
      else arcs(std::false_type{});
      const uint32_t cur = nodes[before];
      wave_sync();
      if (lane == 0) nodes[0] = cur;
    }
  }
  if (__any(bad) && lane == 0) a.ctl->sym_no = 1u;
  sym_finish(prod, swapped < 0);
  sym_block(prod, sums);
  unsigned long long* const part = reinterpret_cast<unsigned long long*>(a.fr[1].node);
  if (threadIdx.x == 0) {
    unsigned long long* mine = part + 2 * kSymPoints * static_cast<size_t>(blockIdx.x);
#pragma unroll
    for (int i = 0; i < kSymPoints; ++i) {
      st_agent(&mine[2 * i], __builtin_bit_cast(unsigned long long, prod.up[i]));
      st_agent(&mine[2 * i + 1], __builtin_bit_cast(unsigned long long, prod.down[i]));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    last = atomicAdd(&a.ctl->xstat[0][11], 1ull) == gridDim.x - 1 ? 1u : 0u;
  }
  __syncthreads();
  if (!last) return;
  sym_start(prod);
  for (uint32_t b = threadIdx.x; b < gridDim.x; b += kBlock) {
    const unsigned long long* w = part + 2 * kSymPoints * static_cast<size_t>(b);
    double up[kSymPoints], down[kSymPoints];
#pragma unroll
    for (int i = 0; i < kSymPoints; ++i) {
      up[i] = __builtin_bit_cast(double, ld_agent(&w[2 * i]));
      down[i] = __builtin_bit_cast(double, ld_agent(&w[2 * i + 1]));
    }
    sym_join(prod, up, down);
  }
  sym_block(prod, sums);
  if (threadIdx.x == 0) {
    bool same = true;
    for (int i = 0; i < kSymPoints; ++i) same = same && sym_equal(prod.up[i], prod.down[i]);
    if (!same) a.ctl->sym_no = 1u;
  }
}

// One pulled level, after k_expand_balanced has accounted for it: every
// unreached node with a reached neighbour gets level L + 1 and joins worklist
// L + 1.  Reached means the frozen snapshot seen[L & 1], so nodes found here
// do not count; the next snapshot, `visited` and every XCD's filter are
// written as whole words.  What bounds it: the dependent reads of a node's
// offsets, arcs and their snapshot words (random 4-byte reads that hit L2).
template <bool kNarrow>
__global__ __launch_bounds__(kPullBlock) void k_bfs_pull(KArgs a, uint32_t launch) {
  constexpr uint32_t T = TileCfg<false>::kEdges;
  constexpr int kWv = kPullBlock / 64;
  __shared__ uint32_t wsum[2][kWv];
  __shared__ unsigned long long base_sh;
  const uint32_t L = level_of(a, launch);
  const unsigned long long c = ld_agent(&a.ctl->ctr[L % 3]);
  const uint32_t Ef = static_cast<uint32_t>(c);
  if (Ef <= a.min_arcs || !level_fits<false, false>(a, c) || !pulls(a, Ef)) return;
  Frontier nxt = a.fr[(L + 1) & 1];
  nxt.level = L + 1;
  const int nctr = (L + 1) % 3;
  const uint32_t* seen = a.seen[L & 1];
  uint32_t* seen_nxt = a.seen[(L + 1) & 1];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  // the balanced kernel's tile counters of level L + 1 (see expand_level)
  if (blockIdx.x == 0 && tid < static_cast<uint32_t>(kXcds)) a.ctl->xstat[tid][8 + (L + 1) % 3] = 0ull;
  uint32_t upd = 0;
  bool bad = false;
  for (uint32_t c0 = blockIdx.x * kPullChunk; c0 < a.n; c0 += gridDim.x * kPullChunk) {
    uint32_t s[kPullPer], e[kPullPer], word[kPullPer];
#pragma unroll
    for (uint32_t i = 0; i < kPullPer; ++i) {
      const uint32_t v = c0 + i * kPullBlock + tid;
      word[i] = v < a.n ? *at<kNarrow>(seen, v >> 5) : ~0u;
    }
#pragma unroll
    for (uint32_t i = 0; i < kPullPer; ++i) {
      const uint32_t v = c0 + i * kPullBlock + tid;
      s[i] = 0u;
      e[i] = 0u;
      if (!((word[i] >> (v & 31)) & 1u)) {
        s[i] = static_cast<uint32_t>(*at<kNarrow>(a.offsets, v));
        e[i] = static_cast<uint32_t>(*at<kNarrow>(a.offsets, v + 1));
        if (s[i] > e[i] || e[i] > a.m) {
          bad = true;
          e[i] = s[i] = 0u;
        }
      }
    }
    uint32_t found = 0, cnt = 0, deg = 0;  // bit i: node i is new
#pragma unroll
    for (uint32_t i = 0; i < kPullPer; ++i) {
      uint32_t p = s[i];
      const uint32_t stop = min(e[i], s[i] + kPullAlone);
      bool hit = false;
      while (p < stop && !hit) {
        uint32_t col[4];
        bool ok[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          ok[b] = p + b < stop;
          col[b] = ok[b] ? static_cast<uint32_t>(*at<kNarrow>(a.cols, p + b)) : 0u;
          if (col[b] >= a.n) {
            bad = true;
            ok[b] = false;
            col[b] = 0u;
          }
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const uint32_t w = *at<kNarrow>(seen, col[b] >> 5);
          hit = hit || (ok[b] && ((w >> (col[b] & 31)) & 1u));
        }
        p += 4;
      }
      // long lists: the wavefront reads them together
      for (uint64_t more = __ballot(!hit && p < e[i]); more; more &= more - 1ull) {
        const int who = __builtin_ctzll(more);
        const uint32_t q1 = __shfl(e[i], who, 64);
        bool any = false;
        for (uint32_t q = __shfl(p, who, 64) + lane; !any && q - lane < q1; q += 64) {
          bool here = false;
          if (q < q1) {
            const uint32_t col = static_cast<uint32_t>(*at<kNarrow>(a.cols, q));
            if (col < a.n) here = (*at<kNarrow>(seen, col >> 5) >> (col & 31)) & 1u;
            else bad = true;
          }
          any = __any(here);
        }
        if (static_cast<int>(lane) == who) hit = any;
      }
      const uint32_t v = c0 + i * kPullBlock + tid;
      if (hit) {
        *at<kNarrow>(a.levels, v) = static_cast<int32_t>(L + 1);
        found |= 1u << i;
        ++cnt;
        deg += e[i] - s[i];
      }
      const uint64_t hits = __ballot(hit);
      const uint32_t now = word[i] | static_cast<uint32_t>(hits >> (lane & 32));
      if ((lane & 31) == 0u && v < a.n) {
        const uint32_t w = v >> 5;
        *at<kNarrow>(a.visited, w) = now;
        *at<kNarrow>(seen_nxt, w) = now;
#pragma unroll
        for (int x = 0; x < kXcds; ++x) a.xfilter[static_cast<size_t>(x) * a.words + w] = now;
      }
    }
    upd += cnt;
    // the chunk's new nodes: one reservation
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
    uint32_t nb = static_cast<uint32_t>(base_sh >> 32) + pc, eb = static_cast<uint32_t>(base_sh) + pe;
#pragma unroll
    for (uint32_t i = 0; i < kPullPer; ++i) {
      if (found & (1u << i)) {
        write_entry<0, T, kNarrow>(a, nxt, nb, eb, 0, 0, static_cast<int32_t>(s[i]), static_cast<int32_t>(e[i] - s[i]));
        ++nb;
        eb += e[i] - s[i];
      }
    }
  }
  if (__any(bad) && lane == 0) atomicOr(&a.ctl->error, kErrBadArc);
  if (a.count_stats) {
    const uint32_t su = wave_sum(upd);
    if (lane == 0 && su) atomicAdd(&a.ctl->xstat[blockIdx.x % kXcds][0], static_cast<unsigned long long>(su));
    // none of the worklist's arcs were loaded
    if (blockIdx.x == 0 && tid == 0) atomicAdd(&a.ctl->xstat[0][7], static_cast<unsigned long long>(Ef));
  }
}

}  // namespace lbg
