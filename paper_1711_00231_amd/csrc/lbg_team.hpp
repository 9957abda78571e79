// Small frontiers (a8): a level loop on the device by a team of workgroups.
//
// High-diameter graphs spend thousands of levels with a few thousand arcs
// each, and small graphs spend all of theirs that way; there a level's cost
// is its chain of dependent memory round trips plus whatever separates it
// from the next level.  k_expand_team keeps up to kTeamMax workgroups
// resident and runs level after level with one flag exchange between them.
//
// What bounds it: latency.  A level is the flag exchange (about 2.5 us for
// 64 or 128 workgroups on all eight XCDs, measured; 4.6 us for 256), one
// read of the level's entries, the arcs, one atomic per arc with the target's
// offsets fetched alongside it, and the stores of the pushed entries.
// Everything workgroups exchange goes through agent-scope atomic loads and
// stores, ordered by waiting for the stores before the flag is raised; the
// agent-scope fences that plain data would need write back and invalidate
// whole L2s and cost about 30 us per level (measured), which is as slow as
// one launch per level.  Against one workgroup with the frontier in its LDS
// (levels of at most 16 K arcs) and one-level launches for the rest: a solve
// of a 16 K-node uniform graph went from 194 to 92 us (BFS) and from 311 to
// 179 us (SSSP), BFS of the 2048 x 2048 grid with shortcuts from 1.71 to
// 1.24 ms.
//
// Membership: a workgroup joins by an atomic on join[]; the first one closes
// the team when every workgroup of the grid has joined or after kTeamWait,
// and only the workgroups that joined before take part.  So the members are
// all running, and nobody ever waits for a workgroup that has not been
// scheduled.  A wait gives up after kTeamPatience (kErrTeam).
#pragma once

#include "lbg_kernels.hpp"

namespace lbg {

constexpr int kTeamBlock = 512;
constexpr int kTeamWaves = kTeamBlock / 64;
constexpr int kTeamU = kTeamSlots / kTeamBlock;
// Up to this many arcs a level is all latency: every arc issues its atomic,
// and its target's offsets, at once.  Beyond, the state is read first and
// only arcs that can still win issue them (one more round trip, but the
// memory side takes about 27 G atomics/s for the whole chip).
constexpr uint32_t kTeamEager = 32768;
constexpr unsigned long long kTeamWait = 1000;               // 10 us of the 100 MHz clock
constexpr unsigned long long kTeamPatience = 1000000000ull;  // 10 s

constexpr uint32_t kTeamClosed = 0x80000000u;

template <typename T>
__device__ __forceinline__ T ld_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Joins launch seq's team (one thread).  Returns the workgroup's number and
// sets *size, or returns kTeamMax when it is not a member.
__device__ __forceinline__ uint32_t team_join(const KArgs& a, uint32_t seq, uint32_t* size) {
  TeamCtl* t = a.team;
  uint32_t* join = &t->join[seq & 3];
  const uint32_t me = __hip_atomic_fetch_add(join, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  *size = 0u;
  if (me & kTeamClosed) return kTeamMax;
  const unsigned long long t0 = wall_clock64();
  if (me == 0u) {
    t->join[(seq + 2) & 3] = 0u;
    t->size[(seq + 2) & 3] = 0u;
    while (ld_agent(join) < gridDim.x && wall_clock64() - t0 < kTeamWait) __builtin_amdgcn_s_sleep(1);
    const uint32_t p = __hip_atomic_fetch_or(join, kTeamClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    st_agent(&t->size[seq & 3], p);
    *size = p;
    return 0u;
  }
  for (;;) {
    const uint32_t p = ld_agent(&t->size[seq & 3]);
    if (p) {
      *size = p;
      return me;
    }
    if (wall_clock64() - t0 > kTeamPatience) {
      atomicOr(&a.ctl->error, kErrTeam);
      return kTeamMax;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

template <bool kSssp>
struct TeamLds {
  uint32_t segn[kTeamMax + 1];  // entries of the level before segment q
  uint32_t sege[kTeamMax + 1];  // arcs of the level before segment q
  uint32_t base[2 * kTeamSlots];                 // arc of slot s of entry i is base[i] + s
  int32_t node[kSssp ? 2 * kTeamSlots : 1];      // entry i's node
  uint32_t flag[kTeamSlots / 32];                // bit s: an entry starts at slot s
  uint32_t lead;                                 // the entry that holds slot 0
  uint32_t ppre[kTeamSlots];                     // pushes: arcs of the pushes before,
  int32_t pst[kTeamSlots];                       //   first arc,
  int32_t pnode[kSssp ? kTeamSlots : 1];         //   node
  unsigned long long push;                       // (entries << 32) | arcs pushed so far
  uint32_t me, size, ok;
  uint32_t over;                                 // some workgroup's pushes outgrew its segment
};

// Exchange number e: wave 0 raises this workgroup's flag, waits for every
// member's and leaves the prefix sums of their payloads in segn / sege:
// (entries << 21 | arcs) or, kArcsOnly, arcs alone (segn is kept); over says
// whether a workgroup has more than seg entries.  Must be reached by the
// whole workgroup after its stores have been waited for and a barrier; ends
// with one.
template <bool kSssp, bool kArcsOnly>
__device__ __forceinline__ bool team_exchange(const KArgs& a, TeamLds<kSssp>& sm, uint32_t e, uint32_t me,
                                              uint32_t size, uint32_t seg, unsigned long long payload) {
  if (threadIdx.x < 64) {
    const uint32_t lane = threadIdx.x;
    unsigned long long* f = a.tflag + (e & 1) * a.tblocks;
    if (lane == 0) st_agent(&f[me], (static_cast<unsigned long long>(e) << 34) | payload);
    const unsigned long long t0 = wall_clock64();
    unsigned long long v[2];
    bool ok = false;
    for (uint32_t spin = 1; !ok; ++spin) {
      bool here = true;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t q = h * 64 + lane;
        v[h] = q < size ? ld_agent(&f[q]) : 0ull;
        here = here && (q >= size || static_cast<uint32_t>(v[h] >> 34) == (e & 0x3fffffffu));
      }
      ok = __all(here);
      if (!ok && (spin & 1023u) == 0u && wall_clock64() - t0 > kTeamPatience) break;
    }
    uint32_t cn = 0, ce = 0;
    bool over = false;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t q = h * 64 + lane;
      const uint32_t xe = kArcsOnly ? static_cast<uint32_t>(v[h]) : static_cast<uint32_t>(v[h]) & 0x1fffffu;
      const uint32_t ie = wave_incl_scan(xe);
      sm.sege[q + 1] = ce + ie;
      ce += __shfl(ie, 63, 64);
      if (!kArcsOnly) {
        const uint32_t xn = static_cast<uint32_t>(v[h] >> 21) & 0x1fffu;
        over = over || xn > seg;
        const uint32_t in = wave_incl_scan(xn);
        sm.segn[q + 1] = cn + in;
        cn += __shfl(in, 63, 64);
      }
    }
    over = __any(over);
    if (lane == 0) {
      if (!kArcsOnly) sm.over = over ? 1u : 0u;
      sm.sege[0] = 0u;
      if (!kArcsOnly) sm.segn[0] = 0u;
      sm.ok = ok ? 1u : 0u;
      if (!ok) atomicOr(&a.ctl->error, kErrTeam);
    }
  }
  __syncthreads();
  return sm.ok != 0u;
}

// Levels L0, L0 + 1, ... until the worklist is empty, max_levels levels have
// run or a level has more than `limit` arcs; then the next level is written
// in the one-level kernels' worklist format and the host continues from
// ctl->levels.  Level L0 comes in that format (at most `limit` arcs and
// kTeamE entries, or nothing is done); later levels live as one segment of
// entries per workgroup, segment q of level L at q * seg of the arrays of
// buffer (L + 1) & 1 (estart, node; eprefix counts from the segment's start),
// with the segments' sizes exchanged in the flags.  A level's arcs are cut
// evenly: workgroup w takes arcs [w C, (w + 1) C), so a hub is shared by many
// workgroups and none pushes more than C <= kTeamSlots entries; they are kept
// in LDS as well.  The arrays hold n entries in all, so with fewer than
// kTeamE nodes a workgroup's pushes may outgrow its segment; then the level
// is written in the one-level format from the LDS copies, once the counts
// are known (one more exchange).
template <bool kSssp, bool kNarrow, bool kPacked = false>
__global__ __launch_bounds__(kTeamBlock) void k_expand_team(KArgs a, uint32_t L0, uint32_t seq, uint32_t limit,
                                                            uint32_t max_levels) {
  static_assert(!kPacked || kSssp, "packed arcs: SSSP");
  static_assert(kTeamMax == 128 && kTeamSlots == 64 * 32, "two flags per lane, one flag word per lane");
  constexpr uint32_t T = TileCfg<kSssp>::kEdges;
  constexpr int kPay = kSssp ? 1 : 0;
  __shared__ TeamLds<kSssp> sm;
  __shared__ uint32_t red[2][kTeamWaves];
  const uint32_t tid = threadIdx.x, lane = tid & 63;

  const unsigned long long c0 = ld_agent(&a.ctl->ctr[L0 % 3]);
  uint32_t nf = static_cast<uint32_t>(c0 >> 32), E = static_cast<uint32_t>(c0);
  if (E == 0u || nf == 0u || E > min(limit, kTeamE) || nf > a.node_cap) return;  // grid-uniform
  if (tid == 0) sm.me = team_join(a, seq, &sm.size);
  __syncthreads();
  const uint32_t me = sm.me, P = min(sm.size, kTeamMax);
  if (me >= P) return;
  limit = min(limit, P * kTeamSlots);
  const uint32_t seg = min(kTeamSlots, a.node_cap / gridDim.x);  // entries of a segment
  if (E > limit) return;  // a small team: the host goes on with one-level launches

  uint32_t e = a.team->epoch;
  // the first level: pseudo-segments of equal entry counts
  bool contiguous = true;
  uint32_t stride = (nf + P - 1) / P;
  if (tid <= P) {
    const uint32_t i = min(tid * stride, nf);
    sm.segn[tid] = i;
    sm.sege[tid] = i < nf ? ld_agent(at<kNarrow>(a.fr[L0 & 1].eprefix, i)) : E;
  }
  if (tid < kTeamSlots / 32) sm.flag[tid] = 0u;
  if (tid == 0) sm.push = 0ull;
  __syncthreads();

  uint32_t upd = 0, atom = 0;
  unsigned long long tot_f = 0, tot_e = 0;
  bool bad = false, alive = true;
  uint32_t L = L0;
  for (;;) {
    const Frontier cur = a.fr[contiguous ? (L & 1) : ((L + 1) & 1)];
    const Frontier nxt = a.fr[L & 1];
    const uint32_t C = (E + P - 1) / P;
    const uint32_t lo = min(me * C, E), hi = min(lo + C, E);
    tot_f += nf;
    tot_e += E;
    // Stage the entries that overlap [lo, hi).
    if (lo < hi) {
      uint32_t q1 = 0, q2 = 0;  // the segments that do: [q1, q2)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t q = h * 64 + lane;
        q1 += static_cast<uint32_t>(__popcll(__ballot(q < P && sm.sege[q < P ? q + 1 : 0] <= lo)));
        q2 += static_cast<uint32_t>(__popcll(__ballot(q < P && sm.sege[q] < hi)));
      }
      const uint32_t first = sm.segn[q1], last = sm.segn[q2];
      for (uint32_t i = first + tid; i < last; i += kTeamBlock) {
        uint32_t q = q1, top = q2;  // segn[q] <= i < segn[top]
        while (top - q > 1) {
          const uint32_t mid = (q + top) / 2;
          if (sm.segn[mid] <= i) q = mid;
          else top = mid;
        }
        const uint32_t at_ = q * stride + (i - sm.segn[q]);
        const uint32_t off = contiguous ? 0u : sm.sege[q];
        const bool more = i + 1 < sm.segn[q + 1];
        const uint32_t p = off + ld_agent(at<kNarrow>(cur.eprefix, at_));
        const uint32_t pn = more ? off + ld_agent(at<kNarrow>(cur.eprefix, at_ + 1)) : sm.sege[q + 1];
        const uint32_t st = static_cast<uint32_t>(ld_agent(at<kNarrow>(cur.estart, at_)));
        const int32_t u = kSssp ? ld_agent(at<kNarrow>(cur.node, at_)) : 0;
        if (p < hi && pn > lo) {
          const uint32_t k = i - first;
          if (k < 2 * kTeamSlots) {
            const uint32_t s = (p > lo ? p : lo) - lo;
            sm.base[k] = st + lo - p;
            if (kSssp) sm.node[k] = u;
            if (s == 0u) sm.lead = k;
            atomicOr(&sm.flag[s >> 5], 1u << (s & 31));
          } else {
            bad = true;
          }
        }
      }
    }
    __syncthreads();
    if (contiguous) {
      // pushes reuse this level's arrays: everyone has to have read them
      ++e;
      alive = team_exchange<kSssp, false>(a, sm, e, me, P, seg, 0ull);
      if (!alive) break;
    }
    if (lo < hi) {
      const uint32_t fw = sm.flag[lane];
      const uint32_t pre = wave_incl_scan(__popc(fw)) - __popc(fw);
      const uint32_t lead = sm.lead, len = hi - lo;
      const bool eager = E <= kTeamEager;
      int32_t vv[kTeamU];
      uint32_t ww[kTeamU], du[kTeamU];
#pragma unroll
      for (int r = 0; r < kTeamU; ++r) {
        const uint32_t s = r * kTeamBlock + tid;
        vv[r] = -1;
        ww[r] = 0;
        du[r] = 0;
        if (r * kTeamBlock < len) {  // workgroup-uniform
          const uint32_t k = s >> 5;
          const uint32_t before = __shfl(pre, k, 64);
          const uint32_t bits = __shfl(fw, k, 64) & static_cast<uint32_t>((2ull << (s & 31)) - 1ull);
          if (s < len) {
            const uint32_t i = lead + before + __popc(bits) - 1u;
            const uint32_t arc = i < 2 * kTeamSlots ? sm.base[i] + s : a.m;
            if (arc < a.m) {
              if (kPacked) {
                load_arc<true, kNarrow>(a, arc, &vv[r], &ww[r]);
              } else {
                vv[r] = *at<kNarrow>(a.cols, arc);
                if (kSssp) ww[r] = *at<kNarrow>(a.weights, arc);
              }
              if (kSssp) {
                // the node's distance, settled for this level by the exchange
                const uint32_t u = static_cast<uint32_t>(sm.node[i]);
                if (u < a.n) {
                  du[r] = static_cast<uint32_t>(ld_agent(at<kNarrow>(a.dstate, u)) >> 32);
                } else {
                  bad = true;
                  vv[r] = -1;
                }
              }
            } else {
              bad = true;
            }
          }
        }
      }
      bool win[kTeamU];
      int32_t s0[kTeamU], s1[kTeamU];
#pragma unroll
      for (int r = 0; r < kTeamU; ++r) {
        if (vv[r] >= 0 && static_cast<uint32_t>(vv[r]) >= a.n) {  // malformed cols (see lbg_validate_csr)
          bad = true;
          vv[r] = -1;
        }
        win[r] = vv[r] >= 0;
        s0[r] = 0;
        s1[r] = 0;
      }
      if (!eager) {
        unsigned long long x[kTeamU];
#pragma unroll
        for (int r = 0; r < kTeamU; ++r) {
          x[r] = 0ull;
          if (win[r])
            x[r] = kSssp ? ld_agent(at<kNarrow>(a.dstate, static_cast<uint32_t>(vv[r])))
                         : ld_agent(at<kNarrow>(a.visited, static_cast<uint32_t>(vv[r]) >> 5));
        }
#pragma unroll
        for (int r = 0; r < kTeamU; ++r)
          win[r] = win[r] && (kSssp ? du[r] + ww[r] < static_cast<uint32_t>(x[r] >> 32)
                                    : !((x[r] >> (vv[r] & 31)) & 1ull));
      }
#pragma unroll
      for (int r = 0; r < kTeamU; ++r) {
        if (win[r] && eager) {
          s0[r] = *at<kNarrow>(a.offsets, vv[r]);
          s1[r] = *at<kNarrow>(a.offsets, vv[r] + 1);
        }
      }
      unsigned long long old[kTeamU];
#pragma unroll
      for (int r = 0; r < kTeamU; ++r) {
        old[r] = 0ull;
        if (win[r]) {
          ++atom;
          if (kSssp)
            old[r] = atomicMin(at<kNarrow>(a.dstate, static_cast<uint32_t>(vv[r])),
                               (static_cast<unsigned long long>(du[r] + ww[r]) << 32) | (L + 1));
          else
            old[r] = atomicOr(at<kNarrow>(a.visited, static_cast<uint32_t>(vv[r]) >> 5), 1u << (vv[r] & 31));
        }
      }
#pragma unroll
      for (int r = 0; r < kTeamU; ++r) {
        if (!win[r]) continue;
        if (!kSssp) {
          win[r] = !((old[r] >> (vv[r] & 31)) & 1ull);
          if (win[r]) {
            *at<kNarrow>(a.levels, vv[r]) = static_cast<int32_t>(L + 1);
            ++upd;
          }
        } else {
          const uint32_t alt = du[r] + ww[r];
          win[r] = alt < static_cast<uint32_t>(old[r] >> 32);
          if (win[r]) {
            *at<kNarrow>(a.d16, vv[r]) = f16_of(alt);  // filter of the one-level launches
            ++upd;
            win[r] = static_cast<uint32_t>(old[r]) != L + 1;  // not yet queued this level
          }
        }
        if (win[r] && !eager) {
          s0[r] = *at<kNarrow>(a.offsets, vv[r]);
          s1[r] = *at<kNarrow>(a.offsets, vv[r] + 1);
        }
      }
      // Push: one LDS atomic per wavefront and round places the winners that
      // have out-arcs and their arcs in this workgroup's segment.
#pragma unroll
      for (int r = 0; r < kTeamU; ++r) {
        if (r * kTeamBlock >= len) continue;
        const int32_t d = s1[r] - s0[r];
        const bool put = win[r] && d > 0;  // a node without out-arcs has nothing to expand
        const uint64_t mask = __ballot(put);
        if (mask == 0) continue;
        const uint32_t inc = wave_incl_scan(put ? static_cast<uint32_t>(d) : 0u);
        unsigned long long b = 0;
        if (lane == 63)
          b = atomicAdd(&sm.push, (static_cast<unsigned long long>(__popcll(mask)) << 32) | inc);
        b = bcast64(b, 63);
        if (put) {
          const uint32_t k = static_cast<uint32_t>(b >> 32) + lane_rank(mask);
          const uint32_t p = static_cast<uint32_t>(b) + inc - static_cast<uint32_t>(d);
          if (k < kTeamSlots) {
            sm.ppre[k] = p;
            sm.pst[k] = s0[r];
            if (kSssp) sm.pnode[k] = vv[r];
          } else {
            bad = true;
          }
          if (k < seg) {
            const uint32_t to = me * seg + k;
            st_agent(at<kNarrow>(nxt.eprefix, to), p);
            st_agent(at<kNarrow>(nxt.estart, to), s0[r]);
            if (kSssp) st_agent(at<kNarrow>(nxt.node, to), vv[r]);
          }
        }
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the entries are out before the flag is raised
    __syncthreads();
    const unsigned long long pushed = sm.push;
    if (tid < kTeamSlots / 32) sm.flag[tid] = 0u;
    ++e;
    alive = team_exchange<kSssp, false>(
        a, sm, e, me, P, seg,
        (min(pushed >> 32, 0x1fffull) << 21) | min(pushed & 0xffffffffull, 0x1fffffull));
    if (!alive) break;
    if (tid == 0) sm.push = 0ull;  // everyone has read it; the next pushes follow a barrier
    contiguous = false;
    stride = seg;
    ++L;
    nf = sm.segn[P];
    E = sm.sege[P];
    if (E == 0u) break;
    const bool leave = E > limit || L - L0 >= max_levels;
    if (!leave && !sm.over) continue;
    // Level L in the one-level format, to go on there (exact arc counts
    // first, then entries, prefixes and marks) or here.
    if (leave) {
      __syncthreads();  // the prefixes are read before the next exchange writes them
      ++e;
      alive = team_exchange<kSssp, true>(a, sm, e, me, P, seg, pushed & 0xffffffffull);
      if (!alive) break;
      E = sm.sege[P];
    }
    const Frontier out = a.fr[L & 1];
    const uint32_t cnt = static_cast<uint32_t>(pushed >> 32), nb = sm.segn[me], eb = sm.sege[me];
    for (uint32_t k = tid; k < min(cnt, kTeamSlots); k += kTeamBlock) {
      const uint32_t p = sm.ppre[k];
      if (leave) {
        const uint32_t pn = k + 1 < cnt ? sm.ppre[k + 1] : static_cast<uint32_t>(pushed);
        write_entry<kPay, T, kNarrow>(a, out, nb + k, eb + p, kSssp ? sm.pnode[k] : 0, 0, sm.pst[k],
                                      static_cast<int32_t>(pn - p));
      } else if (nb + k < a.node_cap) {
        st_agent(at<kNarrow>(out.eprefix, nb + k), eb + p);
        st_agent(at<kNarrow>(out.estart, nb + k), sm.pst[k]);
        if (kSssp) st_agent(at<kNarrow>(out.node, nb + k), sm.pnode[k]);
      } else {
        bad = true;
      }
    }
    if (leave) break;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    ++e;
    alive = team_exchange<kSssp, false>(a, sm, e, me, P, seg, 0ull);
    if (!alive) break;
    contiguous = true;
    stride = (nf + P - 1) / P;
    if (tid <= P) {
      const uint32_t i = min(tid * stride, nf);
      sm.segn[tid] = i;
      sm.sege[tid] = i < nf ? ld_agent(at<kNarrow>(out.eprefix, i)) : E;
    }
    __syncthreads();
  }
  if (__any(bad) && lane == 0) atomicOr(&a.ctl->error, kErrBadArc);
  // Bookkeeping of every level run here, then the tail of level L (the next
  // to expand) and a cleared counter for the level after it.
  if (me == 0u && tid == 0 && alive) {
    a.team->epoch = e;
    a.ctl->levels = L;
    a.ctl->frontier_entries += tot_f;
    a.ctl->edges_scanned += tot_e;
    a.ctl->p_frontier_entries += tot_f;
    a.ctl->p_edges_scanned += tot_e;
    st_agent(&a.ctl->ctr[L % 3], E ? (static_cast<unsigned long long>(nf) << 32) | E : 0ull);
    st_agent(&a.ctl->ctr[(L + 1) % 3], 0ull);
  }
  // the balanced kernel's tile counters of level L (see expand_level)
  if (me == 0u && tid < static_cast<uint32_t>(kXcds)) a.ctl->xstat[tid][8 + L % 3] = 0ull;
  if (a.count_stats) {
    const uint32_t su = wave_sum(upd), sa = wave_sum(atom);
    if (lane == 0) {
      red[0][tid >> 6] = su;
      red[1][tid >> 6] = sa;
    }
    __syncthreads();
    if (tid == 0) {
      unsigned long long tu = 0, ta = 0;
      for (int w = 0; w < kTeamWaves; ++w) {
        tu += red[0][w];
        ta += red[1][w];
      }
      const int x = blockIdx.x % kXcds;
      if (tu) atomicAdd(&a.ctl->xstat[x][2], tu);
      if (ta) atomicAdd(&a.ctl->xstat[x][3], ta);
    }
  }
}

}  // namespace lbg
