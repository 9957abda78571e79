// Batched queries on small instances, each solved by one workgroup.
//
// In the shared worklist a batch's node state is spread over all rows (8 bytes
// per SSSP row, 1.6 GB for 2,048 queries over 322 M arcs), so every filter
// read and atomic goes to memory: 47 G arcs/s for SSSP, 64 for BFS.  The
// state of one query on a small instance fits a CU's LDS: one bit per node
// for BFS, one distance per node for SSSP, where a random read or atomic
// costs a tenth of one in L2 and a hundredth of a memory-side atomic (2,300
// G/s for the chip against 256 and 27, measured).  A workgroup takes a query
// from source to result: levels are separated by its own barriers, nodes to
// expand are listed in the query's row of the packed-state array, and nothing
// is shared with other workgroups.
//
// What bounds it: the latency of a level's dependent reads (list, offsets,
// arcs) on one CU, and the arcs themselves, read in order.  So a query on an
// instance with many more arcs than the others' share would run long after
// the rest is done: those with more than Ctl::solo_limit stay in the shared
// worklist.
#pragma once

#include "lbg_kernels.hpp"

namespace lbg {

constexpr int kSoloBlock = 1024;
constexpr int kSoloWaves = kSoloBlock / 64;
constexpr int kSoloU = 8;               // windows of 64 arcs a wavefront loads together
constexpr uint32_t kSoloSpan = 4096;    // arcs mapped to nodes at a time (64 windows)
constexpr uint32_t kSoloHub = 2048;     // from this many arcs the whole workgroup expands a node
constexpr uint32_t kSoloHubs = 64;

template <bool kSssp, uint32_t kWords>
struct SoloLds {
  uint32_t state[kWords];                      // BFS: visited bits; SSSP: distances
  uint32_t queued[kSssp ? kWords / 32 : 1];    // SSSP: node is in a list
  unsigned long long flag[kSoloWaves][kSoloSpan / 64];  // bit s: a node's arcs start at slot s
  uint32_t base[kSoloWaves][64], du[kSssp ? kSoloWaves : 1][64];
  uint32_t hub_s[kSoloHubs], hub_d[kSoloHubs], hub_du[kSssp ? kSoloHubs : 1];
  uint32_t head, next, hubs, query;
};

// Expands one query (all threads of the workgroup).
template <bool kSssp, uint32_t kWords, bool kNarrow>
__device__ __forceinline__ void solo_solve(const KArgs& a, SoloLds<kSssp, kWords>& sm, const QInfo& qi) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const uint32_t len = static_cast<uint32_t>(qi.row_len), lo = static_cast<uint32_t>(qi.row_start - qi.delta);
  uint32_t* const out = a.dist + qi.row_start;
  uint32_t* cur = reinterpret_cast<uint32_t*>(a.dstate + qi.row_start);  // row_len entries each
  uint32_t* nxt = cur + len;
  const uint32_t x0 = static_cast<uint32_t>(qi.src) - lo;
  if (kSssp) {
    for (uint32_t i = tid; i < len; i += kSoloBlock) sm.state[i] = kSsspInf;
    for (uint32_t i = tid; i < (len + 31) / 32; i += kSoloBlock) sm.queued[i] = 0u;
  } else {
    for (uint32_t i = tid; i < (len + 31) / 32; i += kSoloBlock) sm.state[i] = 0u;
    for (uint32_t i = tid; i < len; i += kSoloBlock) out[i] = kBfsInf;
  }
  __syncthreads();
  if (tid == 0) {
    cur[0] = x0;
    if (kSssp) {
      sm.state[x0] = 0u;
    } else {
      sm.state[x0 >> 5] = 1u << (x0 & 31);
      out[x0] = 0u;
    }
    sm.head = sm.next = sm.hubs = 0u;
  }
  __syncthreads();
  uint32_t cnt = 1, upd = 0, level = 0;
  unsigned long long tot_f = 0, tot_e = 0;
  bool bad = false;

  // The arcs e[u] (0xffffffff: none) of one wavefront, relaxed with the
  // distances d[u].
  auto relax = [&](const uint32_t (&e)[kSoloU], const uint32_t (&d)[kSoloU]) {
    uint32_t x[kSoloU], w[kSoloU];
#pragma unroll
    for (int u = 0; u < kSoloU; ++u) {
      x[u] = 0xffffffffu;
      w[u] = 0;
      if (e[u] != 0xffffffffu) {
        x[u] = static_cast<uint32_t>(*at<kNarrow>(a.cols, e[u])) - lo;
        if (kSssp) w[u] = *at<kNarrow>(a.weights, e[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < kSoloU; ++u) {
      bool push = false;
      if (e[u] != 0xffffffffu) {
        if (x[u] >= len) {
          bad = true;  // malformed cols, or an arc leaving its query's instance
        } else if (kSssp) {
          const uint32_t alt = d[u] + w[u];
          if (alt < sm.state[x[u]] && alt < atomicMin(&sm.state[x[u]], alt)) {
            ++upd;
            const uint32_t bit = 1u << (x[u] & 31);
            push = !(atomicOr(&sm.queued[x[u] >> 5], bit) & bit);
          }
        } else {
          const uint32_t bit = 1u << (x[u] & 31);
          push = !(atomicOr(&sm.state[x[u] >> 5], bit) & bit);
          if (push) {
            ++upd;
            out[x[u]] = level + 1;
          }
        }
      }
      const uint64_t mask = __ballot(push);
      if (mask) {
        uint32_t k = 0;
        if (lane == 0) k = atomicAdd(&sm.next, static_cast<uint32_t>(__popcll(mask)));
        k = __shfl(k, 0, 64) + lane_rank(mask);
        if (push) nxt[k] = x[u];  // a node is listed once: k < len
      }
    }
  };

  while (cnt) {
    // wavefronts take 64 nodes at a time
    for (;;) {
      uint32_t g = 0;
      if (lane == 0) g = atomicAdd(&sm.head, 64u);
      g = __shfl(g, 0, 64);
      if (g >= cnt) break;
      uint32_t s = 0, d = 0, du = 0;
      if (g + lane < cnt) {
        const uint32_t x = cur[g + lane];
        s = static_cast<uint32_t>(*at<kNarrow>(a.offsets, lo + x));
        const uint32_t f = static_cast<uint32_t>(*at<kNarrow>(a.offsets, lo + x + 1));
        if (f >= s && f <= a.m) d = f - s;
        else bad = true;
        if (kSssp) {
          // out of the list first: an improvement from here on lists it again
          atomicAnd(&sm.queued[x >> 5], ~(1u << (x & 31)));
          asm volatile("" ::: "memory");
          du = sm.state[x];
        }
        ++tot_f;
        tot_e += d;
        if (d >= kSoloHub) {
          const uint32_t h = atomicAdd(&sm.hubs, 1u);
          if (h < kSoloHubs) {
            sm.hub_s[h] = s;
            sm.hub_d[h] = d;
            if (kSssp) sm.hub_du[h] = du;
            d = 0;
          }
        }
      }
      const uint32_t pre = wave_incl_scan(d) - d;
      const uint32_t total = __shfl(pre + d, 63, 64);
      // nodes with arcs, in order
      const uint64_t some = __ballot(d > 0u);
      if (d > 0u) {
        const uint32_t r = lane_rank(some);
        sm.base[wid][r] = s - pre;
        if (kSssp) sm.du[wid][r] = du;
      }
      uint32_t before = 0;  // nodes that start before the span
      for (uint32_t b0 = 0; b0 < total; b0 += kSoloSpan) {
        const uint32_t windows = min((total - b0 + 63) / 64, kSoloSpan / 64);
        sm.flag[wid][lane] = 0ull;
        wave_sync();
        if (d > 0u && pre >= b0 && pre - b0 < kSoloSpan)
          atomicOr(&sm.flag[wid][(pre - b0) >> 6], 1ull << (pre & 63));
        wave_sync();
        for (uint32_t w0 = 0; w0 < windows; w0 += kSoloU) {
          uint32_t e[kSoloU], dd[kSoloU];
#pragma unroll
          for (int u = 0; u < kSoloU; ++u) {
            const uint32_t slot = b0 + (w0 + u) * 64 + lane;
            e[u] = 0xffffffffu;
            dd[u] = 0;
            if (w0 + u < windows) {  // wavefront-uniform
              const unsigned long long word = sm.flag[wid][w0 + u];
              const uint32_t i = before + __popcll(word & (~0ull >> (63 - lane))) - 1u;
              before += __popcll(word);
              if (slot < total) {
                e[u] = sm.base[wid][i] + slot;
                if (kSssp) dd[u] = sm.du[wid][i];
              }
            }
          }
          relax(e, dd);
        }
        wave_sync();
      }
    }
    __syncthreads();
    // nodes with many arcs: every wavefront takes its share
    const uint32_t hubs = min(sm.hubs, kSoloHubs);
    for (uint32_t h = 0; h < hubs; ++h) {
      const uint32_t s = sm.hub_s[h], d = sm.hub_d[h], du = kSssp ? sm.hub_du[h] : 0u;
      for (uint32_t c = wid * 64 * kSoloU; c < d; c += kSoloBlock * kSoloU) {
        uint32_t e[kSoloU], dd[kSoloU];
#pragma unroll
        for (int u = 0; u < kSoloU; ++u) {
          const uint32_t slot = c + u * 64 + lane;
          e[u] = slot < d ? s + slot : 0xffffffffu;
          dd[u] = du;
        }
        relax(e, dd);
      }
    }
    __syncthreads();
    cnt = min(sm.next, len);
    uint32_t* t = cur;
    cur = nxt;
    nxt = t;
    ++level;
    __syncthreads();
    if (tid == 0) sm.head = sm.next = sm.hubs = 0u;
    __syncthreads();
  }
  if (kSssp)
    for (uint32_t i = tid; i < len; i += kSoloBlock) out[i] = sm.state[i];
  if (__any(bad) && lane == 0) atomicOr(&a.ctl->error, kErrBadArc);
  if (a.count_stats) {
    const uint32_t su = wave_sum(upd), sf = wave_sum(static_cast<uint32_t>(tot_f));
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) tot_e += bcast64(tot_e, static_cast<int>(lane ^ k));
    if (lane == 0) {
      unsigned long long* x = a.ctl->xstat[blockIdx.x % kXcds];
      if (su) atomicAdd(&x[0], static_cast<unsigned long long>(su));
      if (sf) atomicAdd(&x[13], static_cast<unsigned long long>(sf));
      if (tot_e) atomicAdd(&x[14], tot_e);
    }
    if (tid == 0) atomicMax(&a.ctl->solo_levels, level);
  }
}

// Solves the queries of one class (solo_class) of the batch's table, which is
// sorted by size so that the longest start first; workgroups take them from a
// counter.
template <int kClass, bool kNarrow>
__global__ __launch_bounds__(kSoloBlock) void k_solo(KArgs a) {
  constexpr bool kSssp = kClass >= 3;
  constexpr uint32_t kWords = kSoloWords[kClass];
  __shared__ SoloLds<kSssp, kWords> sm;
  if (a.ctl->solo_limit == 0u) return;
  for (;;) {
    if (threadIdx.x == 0) sm.query = static_cast<uint32_t>(atomicAdd(&a.ctl->xstat[kClass][12], 1ull));
    __syncthreads();
    const uint32_t q = sm.query;
    if (q >= a.num_queries) return;
    const QInfo qi = a.qtab[q];
    if (solo_class(a, qi) == kClass) solo_solve<kSssp, kWords, kNarrow>(a, sm, qi);
    __syncthreads();
  }
}

}  // namespace lbg
