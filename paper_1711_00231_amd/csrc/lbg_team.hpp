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
// of a 16 K-node uniform graph went from 198 to 87 us (BFS) and from 318 to
// 194 us (SSSP), BFS of the 2048 x 2048 grid with shortcuts from 1.73 to
// 0.87 ms, without them from 53 to 13.7 ms (2,500 to 3,700 levels).
//
// Membership: a workgroup joins by an atomic on join[]; the first one closes
// the team when every workgroup of the grid has joined or after kTeamWait,
// and only the workgroups that joined before take part.  So the members are
// all running, and nobody ever waits for a workgroup that has not been
// scheduled.  A wait gives up after kTeamPatience (kErrTeam), and the launches
// behind it do nothing.  One solve at a time has a team of several workgroups
// (TeamPlace in lbg.hip); the others launch this kernel with one.
#pragma once

#include "lbg_kernels.hpp"

namespace lbg {

constexpr int kTeamBlock = 1024;
constexpr int kTeamWaves = kTeamBlock / 64;
constexpr int kTeamU = 2;                             // slots per thread of a pass over the arcs
constexpr uint32_t kTeamPass = kTeamU * kTeamBlock;
// Up to this many arcs a level is all latency: every arc issues its atomic,
// and its target's offsets, at once.  Beyond, the state is read first and
// only arcs that can still win issue them (one more round trip, but the
// memory side takes about 27 G atomics/s for the whole chip).
constexpr uint32_t kTeamEager = 16384;
// Arcs a workgroup may hold whatever the others do.  Cutting a level again
// costs an exchange and a pass through memory (5 us), 8 us for SSSP.
constexpr uint32_t kTeamOwnBfs = 512, kTeamOwnSssp = 1024;
constexpr uint32_t kTeamRounds = 16;   // SSSP rounds between exchanges while the frontier is small,
constexpr uint32_t kTeamCalm = 512;    //   at most so many arcs per workgroup
constexpr uint32_t kTeamAhead = 1024;  // BFS levels a workgroup runs while it holds the whole frontier
constexpr unsigned long long kTeamWait = 1000;               // 10 us of the 100 MHz clock
constexpr unsigned long long kTeamPatience = 1000000000ull;  // 10 s

constexpr uint32_t kTeamArcs = 0xfffffu;  // largest arc count of a flag (more than any level run here)
constexpr uint32_t kTeamClosed = 0x80000000u;

// The words that launch seq + 2 will use; by one thread of every launch,
// whether it runs a level or not.
__device__ __forceinline__ void team_clear(const KArgs& a, uint32_t seq) {
  a.team->join[(seq + 2) & 3] = 0u;
  a.team->size[(seq + 2) & 3] = 0u;
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
    team_clear(a, seq);
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
struct TeamList {  // the entries one workgroup holds, in arc order
  uint32_t pre[kTeamSlots];                  // arcs of the entries before
  int32_t st[kTeamSlots];                    // first arc
  int32_t node[kSssp ? kTeamSlots : 1];      // node
  uint32_t du[kSssp ? kTeamSlots : 1];       // the distance it was pushed with
};

template <bool kSssp>
struct TeamLds {
  TeamList<kSssp> list[2];      // this level's entries, the next one's
  uint32_t segn[kTeamMax + 1];  // entries before workgroup q's
  uint32_t sege[kTeamMax + 1];  // arcs before workgroup q's
  unsigned long long flag[kTeamSlots / 64];  // bit s: an entry starts at slot s
  unsigned long long push;      // (entries << 32) | arcs pushed so far
  uint32_t me, size, ok;
  uint32_t found;               // split: this workgroup found nodes in the far set
  uint32_t any_found;           //   or some other one did
  uint32_t most;                // arcs of the workgroup with the most
};

// Exchange number e: wave 0 raises this workgroup's flag, waits for every
// member's and leaves the prefix sums of their payloads in segn / sege:
// (found << 33 | entries << 20 | arcs) or, kArcsOnly, arcs alone (segn is
// kept).  Must be reached by the whole workgroup, with a barrier between it
// and what it publishes or overwrites; ends with one.
template <bool kSssp, bool kArcsOnly>
__device__ __forceinline__ bool team_exchange(const KArgs& a, TeamLds<kSssp>& sm, uint32_t e, uint32_t me,
                                              uint32_t size, unsigned long long payload) {
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
      if (!ok && spin > 64u) __builtin_amdgcn_s_sleep(2);
      if (!ok && (spin & 1023u) == 0u && wall_clock64() - t0 > kTeamPatience) break;
    }
    uint32_t cn = 0, ce = 0, most = 0;
    bool found = false;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t q = h * 64 + lane;
      const uint32_t xe = kArcsOnly ? static_cast<uint32_t>(v[h]) : static_cast<uint32_t>(v[h]) & kTeamArcs;
      const uint32_t ie = wave_incl_scan(xe);
      sm.sege[q + 1] = ce + ie;
      ce += __shfl(ie, 63, 64);
      if (!kArcsOnly) {
        const uint32_t xn = static_cast<uint32_t>(v[h] >> 20) & 0x1fffu;
        const uint32_t in = wave_incl_scan(xn);
        sm.segn[q + 1] = cn + in;
        cn += __shfl(in, 63, 64);
        found = found || ((v[h] >> 33) & 1ull);
        most = max(most, xe);
      }
    }
    if (!kArcsOnly) {
      found = __any(found);
      most = static_cast<uint32_t>(wave_max(static_cast<int32_t>(most)));
    }
    if (lane == 0) {
      sm.sege[0] = 0u;
      if (!kArcsOnly) {
        sm.segn[0] = 0u;
        sm.any_found = found ? 1u : 0u;
        sm.most = most;
      }
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
// ctl->next.  Level L0 comes in that format (at most
// `limit` arcs, or nothing is done) and is cut into equal shares of arcs, so
// a hub is shared by many workgroups.  From then on a workgroup expands the
// nodes it pushed itself, from its LDS: no entry passes through memory, and
// the arcs of a level are loaded while the flags are exchanged.  Where that
// leaves a workgroup with more than kTeamOwn* arcs and twice the mean (or
// more than it can hold), the level is written out and cut again.
//
// BFS exchanges flags before every level (levels are hop counts), except where
// one workgroup holds the whole frontier: it runs level after level, up to
// kTeamAhead of them, until it has nothing left or more than kTeamOwnBfs arcs,
// and leaves the level it has reached for the others (a path of 20,000 nodes:
// 61 -> 37 ms; 53 with the frontier in one workgroup's LDS and no team).  SSSP
// runs kTeamRounds rounds between exchanges: distances only fall, so the order
// of relaxations is free (and L counts exchanges).  Since a node may improve
// again after a workgroup has expanded it, every improvement is pushed, with
// its distance, and an entry whose node has a smaller one by then is passed
// over.
template <bool kSssp, bool kNarrow, bool kPacked = false>
__global__ __launch_bounds__(kTeamBlock) void k_expand_team(KArgs a, uint32_t launch, uint32_t seq, uint32_t limit,
                                                            uint32_t max_levels) {
  static_assert(!kPacked || kSssp, "packed arcs: SSSP");
  static_assert(kTeamMax == 128 && kTeamSlots == 64 * 64, "two flags per lane, one word of entry starts per lane");
  constexpr uint32_t T = TileCfg<kSssp>::kEdges;
  constexpr int kPay = kSssp ? 1 : 0;
  __shared__ TeamLds<kSssp> sm;
  __shared__ uint32_t red[2][kTeamWaves];
  const uint32_t tid = threadIdx.x, lane = tid & 63;

  const uint32_t failed = ld_agent(&a.ctl->error);
  const uint32_t L0 = level_of(a, launch);
  const unsigned long long c0 = ld_agent(&a.ctl->ctr[L0 % 3]);
  if (failed) return;  // in an earlier launch: what it left is not to be built on
  uint32_t nf = static_cast<uint32_t>(c0 >> 32), E = static_cast<uint32_t>(c0);
  const bool far = kSssp && a.far && a.ctl->plain == 0u;
  if ((E == 0u && !far) || E > min(limit, kTeamE) || nf > a.node_cap) {
    // Nothing for a team to do, if nobody has joined one: a workgroup that
    // starts late (other streams hold the CUs) may find the counter as a team
    // that has come and gone left it, and that team has set the next level.
    // The counter is read before join (the branch needs it), and a team
    // changes it only after its members joined.
    if (blockIdx.x == 0 && tid == 0 &&
        __hip_atomic_fetch_or(&a.team->join[seq & 3], kTeamClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) {
      team_clear(a, seq);
      level_next(a, launch, L0, false);
    }
    return;
  }
  if (tid == 0) {
    sm.me = team_join(a, seq, &sm.size);
    sm.push = 0ull;
    sm.found = 0u;
  }
  if (tid < kTeamSlots / 64) sm.flag[tid] = 0ull;
  __syncthreads();
  const uint32_t me = sm.me, P = min(sm.size, kTeamMax);
  if (me >= P) return;
  limit = min(limit, P * kTeamSlots);
  if (E > limit) {  // a small team: the host goes on with one-level launches
    if (me == 0u && tid == 0) level_next(a, launch, L0, false);
    return;
  }

  uint32_t e = a.team->epoch;
  // near-far state (see far_raise); every member keeps the same
  uint32_t thr = kSsspInf, delta = 0, delta0 = 0, most = 0;
  if (far) {
    thr = a.team->thr[L0 % 3];
    delta = a.team->delta[L0 % 3];
    most = a.team->most[L0 % 3];
    delta0 = a.team->delta0;
  }
  uint32_t upd = 0, atom = 0, levels = 0;
  unsigned long long tot_f = 0, tot_e = 0;  // this workgroup's share
  bool bad = false, alive = true, done = false;
  uint32_t cur = 0;            // the list of this level
  uint32_t cnt = 0, arcs = 0;  // its size
  uint32_t L = L0;

  bool staged = E > 0u;                  // the lists are an equal cut of level L: nothing to ask the others
  bool known = false;                    // the others' counts are known
  uint32_t rounds = 1;                   // until the next exchange
  bool ahead = false;                    // BFS: one workgroup runs ahead,
  bool leads = false;                    //   this one
  uint32_t part = 0;                     // stage() took an entry whose first arc is another workgroup's

  // Adds (per wavefront, convergent) the lanes with `put` to list `to`.  SSSP
  // lists a node once for every improvement, with all of its arcs each time,
  // so their sum is bounded by no graph size.  An entry counts kMostArcs at
  // most: with one such the level has more than `limit` and leaves the team,
  // and the nodes' arcs are looked up again then; 4096 of them are below 2^32.
  constexpr uint32_t kMostArcs = kTeamE + 1;
  auto put_all = [&](uint32_t to, bool put, int32_t v, int32_t s0, int32_t d, uint32_t du) {
    const uint64_t mask = __ballot(put);
    if (mask == 0) return;
    const uint32_t inc = wave_incl_scan(put ? static_cast<uint32_t>(d) : 0u);
    unsigned long long b = 0;
    if (lane == 63) b = atomicAdd(&sm.push, (static_cast<unsigned long long>(__popcll(mask)) << 32) | inc);
    b = bcast64(b, 63);
    if (put) {
      const uint32_t k = static_cast<uint32_t>(b >> 32) + lane_rank(mask);
      if (k < kTeamSlots) {
        sm.list[to].pre[k] = static_cast<uint32_t>(b) + inc - static_cast<uint32_t>(d);
        sm.list[to].st[k] = s0;
        if (kSssp) {
          sm.list[to].node[k] = v;
          sm.list[to].du[k] = du;
        }
      } else {
        bad = true;
      }
    }
  };
  // The list put_all filled becomes this level's.  Barriers on both sides.
  auto turn = [&]() {
    __syncthreads();
    const unsigned long long p = sm.push;
    cur ^= 1u;
    cnt = min(static_cast<uint32_t>(p >> 32), kTeamSlots);
    arcs = static_cast<uint32_t>(p);
    __syncthreads();
    if (tid == 0) sm.push = 0ull;
  };
  // This workgroup's share of level L from the one-level worklist format
  // (E arcs, nf entries, in buffer L & 1).
  auto stage = [&]() {
    const Frontier f = a.fr[L & 1];
    const uint32_t C = (E + P - 1) / P;
    const uint32_t lo = min(me * C, E), hi = min(lo + C, E);
    // the entry that holds arc lo: by halving steps of the whole workgroup
    uint32_t i0 = 0, i1 = nf;  // eprefix[i0] <= lo, eprefix[i1] > lo
    while (lo < hi && i1 - i0 > 1) {
      const uint32_t step = (i1 - i0 + kTeamBlock - 1) / kTeamBlock;
      const uint32_t i = i0 + tid * step;
      const bool le = i < i1 && ld_agent(at<kNarrow>(f.eprefix, i)) <= lo;
      const uint32_t ranks = static_cast<uint32_t>(__syncthreads_count(le));
      if (ranks == 0u) {  // not a worklist
        bad = true;
        break;
      }
      i0 += (ranks - 1) * step;
      i1 = min(i1, i0 + step);
    }
    cnt = 0;
    arcs = hi - lo;
    part = lo < hi && ld_agent(at<kNarrow>(f.eprefix, i0)) < lo ? 1u : 0u;
    if (lo < hi) {
      for (uint32_t k0 = 0;; k0 += kTeamBlock) {  // at least one arc of every entry taken lies in [lo, hi)
        const uint32_t i = i0 + k0 + tid;
        bool mine = false;
        if (i < nf && k0 + tid < kTeamSlots) {
          const uint32_t p = ld_agent(at<kNarrow>(f.eprefix, i));
          const uint32_t st = static_cast<uint32_t>(ld_agent(at<kNarrow>(f.estart, i)));
          if (p < hi) {
            mine = true;
            sm.list[cur].pre[k0 + tid] = p > lo ? p - lo : 0u;
            sm.list[cur].st[k0 + tid] = static_cast<int32_t>(p > lo ? st : st + (lo - p));
            if (kSssp) {
              const uint32_t u = static_cast<uint32_t>(ld_agent(at<kNarrow>(f.node, i)));
              sm.list[cur].node[k0 + tid] = static_cast<int32_t>(u);
              sm.list[cur].du[k0 + tid] = u < a.n ? static_cast<uint32_t>(ld_agent(at<kNarrow>(a.dstate, u)) >> 32) : 0u;
            }
          }
        }
        const uint32_t got = static_cast<uint32_t>(__syncthreads_count(mine));
        cnt += got;
        if (got < static_cast<uint32_t>(kTeamBlock)) break;
      }
    }
  };
  // Level L, held in the members' lists, to the one-level format: kLast for
  // the next kernel (with tile marks), else for stage().
  auto spill = [&](bool last) {
    const Frontier out = a.fr[L & 1];
    const uint32_t nb = sm.segn[me], eb = sm.sege[me];
    for (uint32_t k0 = 0; k0 < cnt; k0 += kTeamBlock) {  // convergent
      const uint32_t k = k0 + tid;
      const bool act = k < cnt;
      const uint32_t p = act ? sm.list[cur].pre[k] : 0u;
      const int32_t v = kSssp && act ? sm.list[cur].node[k] : 0, st = act ? sm.list[cur].st[k] : 0;
      if (last) {
        const uint32_t pn = k + 1 < cnt ? sm.list[cur].pre[k + 1] : arcs;
        write_entry_wave<kPay, T, kNarrow>(a, out, act, nb + k, eb + p, v, st, static_cast<int32_t>(pn - p));
      } else if (!act) {
        continue;
      } else if (nb + k < a.node_cap) {
        st_agent(at<kNarrow>(out.eprefix, nb + k), eb + p);
        st_agent(at<kNarrow>(out.estart, nb + k), st);
        if (kSssp) st_agent(at<kNarrow>(out.node, nb + k), v);
      } else {
        bad = true;
      }
    }
  };
  auto payload = [&]() {
    return (static_cast<unsigned long long>(cnt) << 20) | min(arcs, kTeamArcs);
  };

  uint32_t len = 0;            // its arcs, if they fit the slots
  int32_t vv[kTeamU];
  uint32_t ww[kTeamU], du[kTeamU];
  // The arcs of slots [from, from + kTeamPass) of this workgroup's entries.
  auto load = [&](uint32_t from) {
    const unsigned long long fw = sm.flag[lane];
    const uint32_t pre = wave_incl_scan(__popcll(fw)) - __popcll(fw);
#pragma unroll
    for (int r = 0; r < kTeamU; ++r) {
      const uint32_t s = from + r * kTeamBlock + tid;
      vv[r] = -1;
      ww[r] = 0;
      du[r] = 0;
      if (from + r * kTeamBlock < len) {  // workgroup-uniform
        // a wavefront's 64 slots are one word's
        const uint32_t before = __shfl(pre, s >> 6, 64);
        const unsigned long long bits = bcast64(fw, s >> 6) & (~0ull >> (63 - lane));
        if (s < len) {
          const uint32_t i = before + __popcll(bits) - 1u;  // slot 0 starts entry 0
          const uint32_t arc =
              i < kTeamSlots ? static_cast<uint32_t>(sm.list[cur].st[i]) + (s - sm.list[cur].pre[i]) : a.m;
          if (arc < a.m) {
            if (kPacked) {
              load_arc<true, kNarrow>(a, arc, &vv[r], &ww[r]);
            } else {
              vv[r] = *at<kNarrow>(a.cols, arc);
              if (kSssp) ww[r] = *at<kNarrow>(a.weights, arc);
            }
            if (kSssp) {
              const uint32_t u = static_cast<uint32_t>(sm.list[cur].node[i]);
              du[r] = sm.list[cur].du[i];
              if (u >= a.n) {
                bad = true;
                vv[r] = -1;
              } else if (static_cast<uint32_t>(ld_agent(at<kNarrow>(a.dstate, u)) >> 32) < du[r]) {
                vv[r] = -1;  // improved since: pushed again by whoever did
              }
            }
          } else {
            bad = true;
          }
        }
      }
    }
  };
  // Relaxes them; the nodes to expand next go to the other list.
  auto relax = [&](uint32_t from) {
    const bool eager = E <= kTeamEager;
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
                             static_cast<unsigned long long>(du[r] + ww[r]) << 32);
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
        const uint32_t was = static_cast<uint32_t>(old[r] >> 32);
        win[r] = alt < was;
        if (win[r]) {
          *at<kNarrow>(a.d16, vv[r]) = f16_of(alt);  // filter of the one-level launches
          ++upd;
          if (was > thr) {  // near-far only: it was not queued so far
            win[r] = alt <= thr;
            far_move<kNarrow>(a, static_cast<uint32_t>(vv[r]), was, win[r]);
          }
        }
      }
      if (win[r] && !eager) {
        s0[r] = *at<kNarrow>(a.offsets, vv[r]);
        s1[r] = *at<kNarrow>(a.offsets, vv[r] + 1);
      }
    }
#pragma unroll
    for (int r = 0; r < kTeamU; ++r) {
      if (from + r * kTeamBlock >= len) continue;
      const int32_t d = s1[r] - s0[r];
      // a node without out-arcs has nothing to expand
      put_all(cur ^ 1u, win[r] && d > 0, vv[r], s0[r], kSssp ? min(d, static_cast<int32_t>(kMostArcs)) : d,
              du[r] + ww[r]);
    }
  };

  if (E > 0u) stage();
  for (;;) {
    const bool fits = arcs <= kTeamSlots;
    len = fits ? arcs : 0u;
    if (fits)
      for (uint32_t k = tid; k < cnt; k += kTeamBlock) {
        const uint32_t s = sm.list[cur].pre[k];
        if (kSssp || s < kTeamSlots) atomicOr(&sm.flag[s >> 6], 1ull << (s & 63));  // BFS: malformed offsets
      }
    __syncthreads();
    load(0u);
    if (known || (!staged && (rounds == 0u || !fits || (leads && (arcs == 0u || arcs > kTeamOwnBfs))))) {
      if (!known) {
        ++e;
        if (leads && tid == 0) {  // the thread that raises the flag
          st_agent(&a.team->level[e & 1], L);
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        alive = team_exchange<kSssp, false>(a, sm, e, me, P, payload());
        if (!alive) break;
        if (kSssp) ++L;
        if (ahead) {
          const uint32_t now = ld_agent(&a.team->level[e & 1]);
          levels += now - L;
          L = now;
        }
      }
      known = false;
      nf = sm.segn[P];
      // several rounds until the next exchange only while the frontier is
      // small and steady: else some workgroups' lists grow while others idle
      rounds = kSssp && sm.sege[P] <= P * kTeamCalm && sm.sege[P] <= 2 * E ? kTeamRounds : 1u;
      E = sm.sege[P];
      ahead = !kSssp && sm.most == E && E <= kTeamOwnBfs;
      leads = ahead && arcs > 0u;
      if (leads) rounds = kTeamAhead;
      if (E == 0u) {
        if (!far) {
          done = true;
          break;
        }
        // Split the far set (see near_far_init): this workgroup's share of
        // its words; nodes beyond what it can push stay in it.
        if (tid < kTeamSlots / 64) sm.flag[tid] = 0ull;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // moves in and out of the far set
        __syncthreads();
        ++e;
        alive = team_exchange<kSssp, false>(a, sm, e, me, P, 0ull);
        if (!alive) break;
        if constexpr (kSssp) {
          far_raise(delta0, most, &thr, &delta);
          most = 0u;
          const uint32_t share = (a.words + P - 1) / P;
          const uint32_t k1 = min((me + 1) * share, a.words);
          for (uint32_t k0 = me * share; k0 < k1; k0 += kTeamBlock) {
            const uint32_t k = k0 + tid;
            const uint32_t had = k < k1 ? ld_agent(at<kNarrow>(a.far, k)) & far_mask(a, k) : 0u;
            if (had) sm.found = 1u;
            uint32_t left = had, kept = 0u;
            while (__any(left != 0u)) {
              constexpr int kB = 4;
              int32_t v[kB], s0[kB], s1[kB];
              uint32_t d[kB];
#pragma unroll
              for (int b = 0; b < kB; ++b) {
                v[b] = left ? static_cast<int32_t>(32 * k + __builtin_ctz(left)) : -1;
                left &= left - 1u;
              }
#pragma unroll
              for (int b = 0; b < kB; ++b) {
                d[b] = kSsspInf;
                s0[b] = 0;
                s1[b] = 0;
                if (v[b] >= 0) {
                  d[b] = static_cast<uint32_t>(ld_agent(at<kNarrow>(a.dstate, static_cast<uint32_t>(v[b]))) >> 32);
                  s0[b] = *at<kNarrow>(a.offsets, v[b]);
                  s1[b] = *at<kNarrow>(a.offsets, v[b] + 1);
                }
              }
#pragma unroll
              for (int b = 0; b < kB; ++b) {
                // room for this push and one in flight of every wavefront
                const bool room = __any((sm.push >> 32) + kTeamBlock <= kTeamSlots);
                const bool go = v[b] >= 0 && d[b] <= thr && room;
                if (v[b] >= 0 && !go) kept |= 1u << (v[b] & 31);
                put_all(cur ^ 1u, go && s1[b] > s0[b], v[b], s0[b],
                        min(s1[b] - s0[b], static_cast<int32_t>(kMostArcs)), d[b]);
              }
            }
            if (kept != had) st_agent(at<kNarrow>(a.far, k), kept);
          }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        turn();
        const bool found = sm.found != 0u;
        ++e;
        alive = team_exchange<kSssp, false>(a, sm, e, me, P, payload() | (found ? 1ull << 33 : 0ull));
        if (!alive) break;
        if (tid == 0) sm.found = 0u;
        ++L;
        nf = sm.segn[P];
        E = sm.sege[P];
        if (E == 0u && !sm.any_found) {
          done = true;
          break;
        }
        known = true;
        continue;
      }
      const bool leave = E > limit || L - L0 >= max_levels;
      if (leave || sm.most > max(kSssp ? kTeamOwnSssp : kTeamOwnBfs, 2 * ((E + P - 1) / P)) || sm.most > kTeamSlots) {
        // load() has read the flags in every wavefront; after a split no
        // exchange, with its barrier, lies in between
        __syncthreads();
        if (tid < kTeamSlots / 64) sm.flag[tid] = 0ull;
        if (kSssp && (leave || nf > a.node_cap)) {
          // only the entry with its node's distance: one per node, so the
          // worklist holds them
          __syncthreads();
          for (uint32_t k0 = 0; k0 < cnt; k0 += kTeamBlock) {
            const uint32_t k = k0 + tid;
            int32_t v = 0, s0 = 0, d = 0;
            uint32_t x = 0;
            bool keep = false;
            if (k < cnt) {
              v = sm.list[cur].node[k];
              x = sm.list[cur].du[k];
              s0 = sm.list[cur].st[k];
              if (static_cast<uint32_t>(v) < a.n) {
                d = *at<kNarrow>(a.offsets, v + 1) - s0;
                keep = static_cast<uint32_t>(ld_agent(at<kNarrow>(a.dstate, static_cast<uint32_t>(v))) >> 32) == x;
              }
            }
            put_all(cur ^ 1u, keep, v, s0, d, x);
          }
          turn();
          ++e;
          alive = team_exchange<kSssp, false>(a, sm, e, me, P, payload());
          if (!alive) break;
          nf = sm.segn[P];
        }
        __syncthreads();  // the prefixes are read before the next exchange writes them
        if (leave || sm.most >= kTeamArcs) {
          bad = bad || arcs > a.m;  // each node once from here on
          ++e;
          alive = team_exchange<kSssp, true>(a, sm, e, me, P, arcs);
          if (!alive) break;
        }
        E = sm.sege[P];
        spill(leave || E > limit);
        if (leave || E > limit) break;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        ++e;
        alive = team_exchange<kSssp, false>(a, sm, e, me, P, 0ull);
        if (!alive) break;
        if (E > 0u) stage();
        else cnt = arcs = 0u;
        staged = true;
        rounds = 1u;
        continue;
      }
    }
    staged = false;
    most = max(most, E);
    tot_f += tid == 0 ? cnt - part : 0u;
    part = 0u;
    tot_e += tid == 0 ? arcs : 0u;
    --rounds;
    if (len) relax(0u);  // workgroup-uniform
    for (uint32_t from = kTeamPass; from < len; from += kTeamPass) {
      load(from);
      relax(from);
    }
    turn();
    if (tid < kTeamSlots / 64) sm.flag[tid] = 0ull;
    __syncthreads();
    if (!kSssp) ++L;
    ++levels;
  }
  if (__any(bad) && lane == 0) atomicOr(&a.ctl->error, kErrBadArc);
  // Bookkeeping of every level run here, then the tail of level L (the next
  // to expand) and a cleared counter for the level after it.
  if (me == 0u && tid == 0 && alive) {
    a.team->epoch = e;
    a.ctl->levels += levels;
    a.ctl->next = L;
    level_next(a, launch, L, true);
    if (far) {
      a.team->thr[L % 3] = thr;
      a.team->delta[L % 3] = delta;
      a.team->most[L % 3] = most;
      if (done) a.ctl->split_at = L;
    }
    st_agent(&a.ctl->ctr[L % 3], E ? (static_cast<unsigned long long>(nf) << 32) | E : 0ull);
    st_agent(&a.ctl->ctr[(L + 1) % 3], 0ull);
  }
  // the balanced kernel's tile counters of level L (see expand_level)
  if (me == 0u && tid < static_cast<uint32_t>(kXcds)) a.ctl->xstat[tid][8 + L % 3] = 0ull;
  if (tid == 0) {
    if (tot_f) {
      atomicAdd(&a.ctl->frontier_entries, tot_f);
      atomicAdd(&a.ctl->p_frontier_entries, tot_f);
    }
    if (tot_e) {
      atomicAdd(&a.ctl->edges_scanned, tot_e);
      atomicAdd(&a.ctl->p_edges_scanned, tot_e);
    }
  }
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
