// Solves by the balanced strategy's kernels, run on the host (see
// hip/hip_runtime.h): k_init, k_expand_team, the one-level kernels and
// k_sssp_finish as solve() in lbg.hip launches them, with every array ending
// at an unmapped page, so that an access beyond one ends the run by a signal.
//
// usage: team_run GRAPH OUT key=value...   (tests/test_team_emulation_cpu.py)
//   GRAPH  int32 n, m, then n + 1 offsets, m columns, m weights
//   OUT    int64 error, levels, next, arcs and entries of the next worklist,
//          team launches, one-level launches with work, 1 if nothing was deferred,
//          then the n results
//   sssp=0|1 src=.. far=0|1 limit=.. blocks=.. grid=..
//   extra=K    K more arcs to node 0, weight 0, after the graph's own: the
//              last node's (their arrays are zero pages)
//   renamed=K  the source's id in a renaming table (node_map[src] = K)
//   fill=B     byte that the workspace and the output hold before the solve
//   join=J     words 0 .. 3 of the team's control block (its join counters)
//   alone=1    one-level launches only, as after a submission without progress
//   error=E    an error that the launches after k_init find
//   stop=1     end after the first team launch
//   first=W    the wavefront of a workgroup that runs first
#include <sys/mman.h>
#include <unistd.h>

#include <map>
#include <string>

#include "lbg_kernels.hpp"
#include "lbg_team.hpp"

using namespace lbg;

template <typename T>
T* array(size_t count, int fill = -1) {
  const size_t page = 4096, bytes = count * sizeof(T), size = (bytes + page - 1) / page * page;
  char* p = static_cast<char*>(mmap(nullptr, size + 2 * page, PROT_READ | PROT_WRITE,
                                    MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
  if (p == MAP_FAILED) emu::die("mmap");
  mprotect(p, page, PROT_NONE);
  mprotect(p + page + size, page, PROT_NONE);
  if (fill >= 0) memset(p + page, fill, size);
  return reinterpret_cast<T*>(p + page + (size - bytes) / alignof(T) * alignof(T));
}

int main(int argc, char** argv) {
  std::map<std::string, long long> opt;
  for (int i = 3; i < argc; ++i) {
    const std::string s = argv[i];
    opt[s.substr(0, s.find('='))] = atoll(s.c_str() + s.find('=') + 1);
  }
  auto get = [&](const char* k, long long d) { return opt.count(k) ? opt[k] : d; };
  FILE* f = fopen(argv[1], "rb");
  int32_t nm[2];
  if (!f || fread(nm, 4, 2, f) != 2) emu::die("graph");
  const uint32_t n = static_cast<uint32_t>(nm[0]), m0 = static_cast<uint32_t>(nm[1]);
  const uint32_t m = m0 + static_cast<uint32_t>(get("extra", 0));
  int32_t* offsets = array<int32_t>(n + 1);
  int32_t* cols = array<int32_t>(m);
  uint32_t* weights = array<uint32_t>(m);
  if (fread(offsets, 4, n + 1, f) != n + 1 || fread(cols, 4, m0, f) != m0 || fread(weights, 4, m0, f) != m0)
    emu::die("graph");
  fclose(f);
  offsets[n] = static_cast<int32_t>(m);

  const bool sssp = get("sssp", 1), alone = get("alone", 0);
  const int32_t src = static_cast<int32_t>(get("src", 0));
  const int fill = static_cast<int>(get("fill", 0));
  emu::first_wave = static_cast<uint32_t>(get("first", 0));

  KArgs a{};
  a.offsets = offsets;
  a.cols = cols;
  a.weights = weights;
  a.n = n;
  a.m = m;
  a.words = (n + 31) / 32;
  a.node_cap = n;
  a.tile_cap = (m + kMinTile - 1) / kMinTile + 2;
  a.scan_min = 0xffffffffu;
  a.count_stats = 1;
  // one block, as in a workspace: the control words follow the control block
  char* ctl = array<char>(1280, fill);
  a.ctl = reinterpret_cast<Ctl*>(ctl);
  a.team = reinterpret_cast<TeamCtl*>(ctl + sizeof(Ctl));
  if (opt.count("join"))
    for (uint32_t& j : a.team->join) j = static_cast<uint32_t>(get("join", 0));
  a.tblocks = static_cast<uint32_t>(get("blocks", std::min<uint32_t>(std::max(1u, n / kTeamNodes), kTeamMax)));
  uint32_t* out = array<uint32_t>(n, fill);
  for (int b = 0; b < 2; ++b) {
    a.fr[b].node = array<int32_t>(a.node_cap, fill);
    a.fr[b].eprefix = array<uint32_t>(a.node_cap, fill);
    a.fr[b].estart = array<int32_t>(a.node_cap, fill);
    a.fr[b].tile_node = array<int32_t>(a.tile_cap, fill);
  }
  if (sssp) {
    a.dist = out;
    a.dstate = array<unsigned long long>(n, fill);
    a.d16 = array<uint16_t>(n, fill);
  } else {
    a.levels = reinterpret_cast<int32_t*>(out);
    a.visited = array<uint32_t>(a.words, fill);
    a.seen[0] = array<uint32_t>(a.words, fill);
    a.seen[1] = array<uint32_t>(a.words, fill);
    a.xfilter = array<uint32_t>(a.words * kXcds, fill);
  }
  a.tflag = array<unsigned long long>(2 * a.tblocks, fill);
  if (sssp && get("far", 0)) a.far = array<uint32_t>(a.words, fill);
  int32_t* map = nullptr;
  if (opt.count("renamed")) {
    map = array<int32_t>(n);
    for (uint32_t v = 0; v < n; ++v) map[v] = static_cast<int32_t>(v);
    map[src] = static_cast<int32_t>(get("renamed", 0));
    a.node_map = map;
  }

  const uint32_t limit = static_cast<uint32_t>(get("limit", a.tblocks * kTeamSlots));
  const uint32_t grid = static_cast<uint32_t>(get("grid", 8));
  uint32_t k = 0, seq = 0, ones = 0, L = 0, L_prev = 0;
  const uint32_t cap = 2 * (n + 2) + 64;
  auto team = [&] {
    const uint32_t kk = k++, s = seq++, left = cap + 1 - L;
    emu::launch(a.tblocks, kTeamBlock, [=] {
      if (sssp) k_expand_team<true, true>(a, kk, s, limit, left);
      else k_expand_team<false, true>(a, kk, s, limit, left);
    });
  };
  auto one = [&] {
    const uint32_t kk = k++;
    emu::launch(grid, kBlock, [=] {
      if (!sssp) k_expand_balanced<false, true>(a, kk);
      else if (a.far) k_expand_balanced<true, true, false, false, false, true>(a, kk);
      else k_expand_balanced<true, true>(a, kk);
    });
    if ((a.ctl->worked >> (kk & 63)) & 1) ++ones;
  };
  emu::launch(2, kBlock, [=] {
    if (sssp) k_init<true, false>(a, src);
    else k_init<false, false>(a, src);
  });
  if (opt.count("error")) a.ctl->error = static_cast<unsigned>(get("error", 0));
  for (int step = 0; step < 2000; ++step) {
    a.min_arcs = alone ? 0u : limit;
    if (!alone) team();
    if (get("stop", 0) || opt.count("error")) break;
    if (a.ctl->plain && step) a.far = nullptr;  // known once a submission has ended
    for (int i = 0; i < 3; ++i) one();
    if (!alone) team();
    if (sssp) emu::launch(2, kBlock, [=] { k_sssp_finish(a); });
    if (a.ctl->error) break;
    L = a.ctl->next;
    const bool empty = static_cast<uint32_t>(a.ctl->ctr[L % 3]) == 0u;
    if (empty && (!a.far || (a.ctl->split_at == L && a.ctl->far_seen != L))) break;
    if (L > cap) emu::die("too many levels");
    if (L == L_prev && step) emu::die("no progress");
    L_prev = L;
  }
  const unsigned long long c = a.ctl->ctr[a.ctl->next % 3];
  const int64_t head[8] = {a.ctl->error, a.ctl->levels, a.ctl->next, static_cast<uint32_t>(c),
                           static_cast<int64_t>(c >> 32), seq, ones,
                           a.tblocks && sssp ? a.ctl->plain : 0};
  f = fopen(argv[2], "wb");
  if (!f) emu::die("output");
  fwrite(head, 8, 8, f);
  fwrite(out, 4, n, f);
  const Frontier& fr = a.fr[a.ctl->next & 1];
  const uint32_t e = static_cast<uint32_t>(std::min<unsigned long long>(c >> 32, n));
  // every tile of the next worklist names the entry that holds its first arc
  const uint32_t T = sssp ? TileCfg<true>::kEdges : TileCfg<false>::kEdges;
  for (uint32_t t = 0; get("stop", 0) && static_cast<uint64_t>(t) * T < static_cast<uint32_t>(c); ++t) {
    const uint32_t i = static_cast<uint32_t>(fr.tile_node[t]);
    if (i >= e || fr.eprefix[i] > t * T || (i + 1 < e && fr.eprefix[i + 1] <= t * T)) emu::die("tile marks");
  }
  fwrite(fr.eprefix, 4, e, f);
  fwrite(fr.estart, 4, e, f);
  fclose(f);
  fflush(nullptr);
  _exit(0);
}
