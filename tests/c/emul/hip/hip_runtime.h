// Runs device code on the host, for tests: compiled with this folder before
// the ROCm headers, a kernel's source is an ordinary C++ function, called once
// per thread.  A workgroup is an operating-system thread (so __shared__ is
// static thread_local); its threads are fibers, which switch where a
// wavefront exchanges values or a barrier is reached; workgroups hand one
// baton around where they wait for each other.  So a run is deterministic:
// within a workgroup the wavefront `emu::first_wave` runs until the next
// barrier, then the one after it, ...; within a wavefront lane 0 runs to the next
// exchange, then lane 1.  Each such order is one the GPU may produce, and
// "one wavefront as far ahead as the barriers let it" shows missing barriers.
//
// Wave-wide operations must be reached by all 64 lanes that have not left the
// kernel (as the kernels' comments require); another kind met by some of them
// aborts, as does a wait that lasts too long.
#pragma once
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <condition_variable>
#include <functional>
#include <mutex>
#include <thread>
#include <type_traits>
#include <vector>

#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(x)
#define __shared__ static thread_local
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_SYSTEM 0
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, order)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, order)
#define __hip_atomic_fetch_or(p, v, order, scope) __atomic_fetch_or(p, v, order)
#define __builtin_amdgcn_fence(order, scope)
#define __builtin_amdgcn_wave_barrier() emu::wave_exchange('b', 0)
#define __builtin_amdgcn_readlane(v, l) __shfl(v, l, 64)
#define __builtin_amdgcn_s_sleep(n) emu::spin()
#define __builtin_amdgcn_mbcnt_lo(m, c) ((c) + __builtin_popcount((m) & emu::below_lo()))
#define __builtin_amdgcn_mbcnt_hi(m, c) ((c) + __builtin_popcount((m) & emu::below_hi()))

// the one instruction that the kernels name
asm(".macro s_waitcnt args:vararg\n.endm");

// Saves the callee's registers and the stack pointer, goes on with another stack (x86-64).
extern "C" void emu_switch(void** save, void* to);
asm(R"(
.text
emu_switch:
  push %rbp
  push %rbx
  push %r12
  push %r13
  push %r14
  push %r15
  mov %rsp, (%rdi)
  mov %rsi, %rsp
  pop %r15
  pop %r14
  pop %r13
  pop %r12
  pop %rbx
  pop %rbp
  ret
)");

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

namespace emu {

[[noreturn]] inline void die(const char* what) {
  fprintf(stderr, "emulation: %s\n", what);
  fflush(stderr);
  _Exit(70);
}

constexpr size_t kStack = 96 << 10;
enum State { kReady, kWave, kBlockWait, kLeft };

struct Fiber {
  void* sp = nullptr;
  char* stack = nullptr;
  uint32_t tid;
  State state = kReady;
};

struct Wave {
  uint64_t buf[2][64];
  uint64_t in[2];     // lanes that took part
  uint32_t gen = 0;   // exchanges so far
  uint32_t arrived = 0, live = 0;
  char kind = 0;
};

struct Group {
  std::vector<Fiber> fibers;
  std::vector<Wave> waves;
  void* main = nullptr;
  uint32_t cur = 0;            // running fiber
  uint32_t live = 0, at_barrier = 0, barrier_gen = 0;
  uint32_t count[2] = {0, 0};  // of __syncthreads_count, by generation
  bool spinning = false;
  std::function<void()> body;
};

inline thread_local Group* group = nullptr;
inline thread_local dim3 block_idx, grid_dim, block_dim;

// The baton: one workgroup runs at a time, in turn.
inline std::mutex mu;
inline std::condition_variable cv;
inline uint32_t turn = 0;
inline std::vector<char> running;
inline unsigned long long clock_ticks = 0;
inline uint32_t first_wave = 0;  // a workgroup's wavefronts run in the order first_wave, first_wave + 1, ..., cyclically
inline unsigned long long kTooLong = 2000000ull;

inline void pass_baton(bool leaving) {
  std::unique_lock<std::mutex> lk(mu);
  const uint32_t me = block_idx.x, n = static_cast<uint32_t>(running.size());
  if (leaving) running[me] = 0;
  uint32_t next = me;
  for (uint32_t k = 1; k <= n; ++k)
    if (running[(me + k) % n]) {
      next = (me + k) % n;
      break;
    }
  turn = next;
  cv.notify_all();
  if (!leaving) cv.wait(lk, [&] { return turn == me; });
}

// Stacks are kept for the next launch.
inline std::vector<char*> stacks;
inline char* stack_new() {
  std::lock_guard<std::mutex> lk(mu);
  if (stacks.empty()) return new char[kStack];
  char* s = stacks.back();
  stacks.pop_back();
  return s;
}
inline void stack_free(char* s) {
  std::lock_guard<std::mutex> lk(mu);
  stacks.push_back(s);
}

inline Fiber& self() { return group->fibers[group->cur]; }
inline uint32_t lane() { return self().tid & 63; }
inline uint32_t below_lo() { return lane() >= 32 ? ~0u : (1u << lane()) - 1u; }
inline uint32_t below_hi() { return lane() >= 32 ? (1u << (lane() - 32)) - 1u : 0u; }

inline void yield() {
  Group* g = group;
  emu_switch(&g->fibers[g->cur].sp, g->main);
}

inline void spin() {
  if (++clock_ticks > kTooLong) die("a wait does not end");
  group->spinning = true;
  yield();
}

// All live lanes of the wavefront give a value; afterwards value(l) is lane
// l's, in `mask` of those that gave one.
struct Got {
  const uint64_t* v;
  uint64_t mask;
};
inline Got wave_exchange(char kind, uint64_t x) {
  Fiber& f = self();
  Wave& w = group->waves[f.tid >> 6];
  const uint32_t gen = w.gen, p = gen & 1;
  if (w.arrived == 0) {
    w.kind = kind;
    w.in[p] = 0;
  } else if (w.kind != kind) {
    die("lanes of a wavefront meet at different exchanges");
  }
  w.buf[p][f.tid & 63] = x;
  w.in[p] |= 1ull << (f.tid & 63);
  if (++w.arrived == w.live) {
    w.arrived = 0;
    ++w.gen;
    for (uint32_t t = (f.tid & ~63u); t < (f.tid | 63u) + 1 && t < group->fibers.size(); ++t)
      if (group->fibers[t].state == kWave) group->fibers[t].state = kReady;
    yield();  // lane 0 goes first
  } else {
    f.state = kWave;
    while (w.gen == gen) yield();
  }
  return Got{w.buf[p], w.in[p]};
}

inline uint32_t barrier(uint32_t add) {
  Group* g = group;
  const uint32_t gen = g->barrier_gen;
  g->count[gen & 1] += add;
  if (++g->at_barrier == g->live) {
    g->at_barrier = 0;
    ++g->barrier_gen;
    g->count[(gen + 1) & 1] = 0;
    for (Fiber& f : g->fibers)
      if (f.state == kBlockWait) f.state = kReady;
  }
  // everyone stops here once, so that the scheduler's order starts anew
  if (g->barrier_gen == gen) {
    self().state = kBlockWait;
    while (g->barrier_gen == gen) yield();
  } else {
    yield();
  }
  return g->count[gen & 1];
}

inline void entry() {
  group->body();
  Group* g = group;
  Fiber& f = self();
  f.state = kLeft;
  Wave& w = g->waves[f.tid >> 6];
  --w.live;
  --g->live;
  if (w.live && w.arrived == w.live) die("lanes left while others exchange");  // none of the kernels does
  if (g->live && g->at_barrier == g->live) {
    const uint32_t gen = g->barrier_gen;
    g->at_barrier = 0;
    ++g->barrier_gen;
    g->count[(gen + 1) & 1] = 0;
    for (Fiber& o : g->fibers)
      if (o.state == kBlockWait) o.state = kReady;
  }
  emu_switch(&f.sp, g->main);
}

inline void run_group(uint32_t threads, const std::function<void()>& body) {
  Group g;
  group = &g;
  g.body = body;
  g.fibers = std::vector<Fiber>(threads);
  g.waves.resize((threads + 63) / 64);
  g.live = threads;
  for (uint32_t t = 0; t < threads; ++t) {
    Fiber& f = g.fibers[t];
    f.tid = t;
    f.stack = stack_new();
    ++g.waves[t >> 6].live;
    // entry's address above six registers; the stack is 8 off 16 there, as after a call
    void** top = reinterpret_cast<void**>((reinterpret_cast<uintptr_t>(f.stack) + kStack) / 16 * 16) - 1;
    *--top = reinterpret_cast<void*>(entry);
    for (int r = 0; r < 6; ++r) *--top = nullptr;
    f.sp = top;
  }
  const uint32_t nw = static_cast<uint32_t>(g.waves.size());
  while (g.live) {
    // the first wavefront, in order, that has a lane to run
    bool ran = false;
    for (uint32_t k = 0; k < nw && !ran; ++k) {
      const uint32_t w = (first_wave + k) % nw;
      for (uint32_t t = w * 64; t < w * 64 + 64 && t < threads; ++t) {
        if (g.fibers[t].state != kReady) continue;
        g.cur = t;
        g.spinning = false;
        emu_switch(&g.main, g.fibers[t].sp);
        ran = true;
        if (g.spinning) pass_baton(false);
      }
    }
    if (!ran) die("deadlock in a workgroup");
  }
  for (Fiber& f : g.fibers) stack_free(f.stack);
  group = nullptr;
}

// Runs a grid of one-dimensional workgroups.
inline void launch(uint32_t blocks, uint32_t threads, const std::function<void()>& kernel) {
  running.assign(blocks, 1);
  turn = 0;
  std::vector<std::thread> ts;
  for (uint32_t b = 0; b < blocks; ++b)
    ts.emplace_back([=] {
      block_idx = dim3(b);
      grid_dim = dim3(blocks);
      block_dim = dim3(threads);
      {
        std::unique_lock<std::mutex> lk(mu);
        cv.wait(lk, [&] { return turn == b; });
      }
      run_group(threads, kernel);
      pass_baton(true);
    });
  for (std::thread& t : ts) t.join();
}

struct Tid {
  struct X {
    operator uint32_t() const { return self().tid; }
  } x;
};
inline Tid thread_idx;

}  // namespace emu

#define threadIdx emu::thread_idx
#define blockIdx emu::block_idx
#define gridDim emu::grid_dim
#define blockDim emu::block_dim

template <typename T>
using emu_id = typename std::type_identity<T>::type;
template <typename T> T atomicAdd(T* p, emu_id<T> v) { return __atomic_fetch_add(p, v, __ATOMIC_RELAXED); }
template <typename T> T atomicOr(T* p, emu_id<T> v) { return __atomic_fetch_or(p, v, __ATOMIC_RELAXED); }
template <typename T> T atomicAnd(T* p, emu_id<T> v) { return __atomic_fetch_and(p, v, __ATOMIC_RELAXED); }
template <typename T> T atomicMin(T* p, emu_id<T> v) {
  T o = __atomic_load_n(p, __ATOMIC_RELAXED);
  while (v < o && !__atomic_compare_exchange_n(p, &o, v, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED)) {}
  return o;
}
template <typename T> T atomicMax(T* p, emu_id<T> v) {
  T o = __atomic_load_n(p, __ATOMIC_RELAXED);
  while (v > o && !__atomic_compare_exchange_n(p, &o, v, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED)) {}
  return o;
}
template <typename A, typename B> auto min(A a, B b) -> std::common_type_t<A, B> { return a < b ? a : b; }
template <typename A, typename B> auto max(A a, B b) -> std::common_type_t<A, B> { return a > b ? a : b; }

inline uint32_t __lane_id() { return emu::lane(); }
inline int __popc(uint32_t x) { return __builtin_popcount(x); }
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
inline unsigned long long wall_clock64() {
  if (++emu::clock_ticks > emu::kTooLong) emu::die("a wait does not end");
  return emu::clock_ticks;
}

inline unsigned long long __ballot(bool p) {
  const emu::Got g = emu::wave_exchange('v', p);
  unsigned long long m = 0;
  for (int l = 0; l < 64; ++l)
    if (((g.mask >> l) & 1) && g.v[l]) m |= 1ull << l;
  return m;
}
inline bool __any(bool p) { return __ballot(p) != 0; }
inline bool __all(bool p) {  // the kernels use it to wait for other workgroups only
  const emu::Got g = emu::wave_exchange('a', p);
  bool r = true;
  for (int l = 0; l < 64; ++l)
    if ((g.mask >> l) & 1) r = r && g.v[l];
  if (!r && emu::lane() == 0) emu::spin();
  return r;
}
template <typename T>
T emu_from(const emu::Got& g, uint32_t l) {
  static_assert(sizeof(T) == 4, "32-bit shuffles");
  return static_cast<T>(static_cast<uint32_t>(g.v[(g.mask >> (l & 63)) & 1 ? l & 63 : emu::lane()]));
}
template <typename T> T __shfl(T v, int src, int) {
  return emu_from<T>(emu::wave_exchange('s', static_cast<uint32_t>(v)), static_cast<uint32_t>(src));
}
template <typename T> T __shfl_up(T v, int d, int) {
  const emu::Got g = emu::wave_exchange('u', static_cast<uint32_t>(v));
  return emu_from<T>(g, emu::lane() >= static_cast<uint32_t>(d) ? emu::lane() - d : emu::lane());
}
template <typename T> T __shfl_xor(T v, int d, int) {
  return emu_from<T>(emu::wave_exchange('x', static_cast<uint32_t>(v)), emu::lane() ^ static_cast<uint32_t>(d));
}
inline void __syncthreads() { emu::barrier(0); }
inline int __syncthreads_count(bool p) { return static_cast<int>(emu::barrier(p ? 1u : 0u)); }
