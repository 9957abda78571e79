// k_bfs_sym on the host (see hip/hip_runtime.h), or with BLOCKS = 0 the sample
// of arcs that k_init takes.
// usage: sym_run GRAPH BLOCKS X0 X1: prints 1 when the graph passes.
//   GRAPH  int32 n, m, then n + 1 offsets, m columns
#include <string>

#include "lbg_pull.hpp"

using namespace lbg;

int main(int argc, char** argv) {
  FILE* f = fopen(argv[1], "rb");
  int32_t nm[2];
  if (argc < 5 || !f || fread(nm, 4, 2, f) != 2) emu::die("graph");
  std::vector<int32_t> offsets(nm[0] + 1), cols(nm[1]);
  if (fread(offsets.data(), 4, offsets.size(), f) != offsets.size() ||
      fread(cols.data(), 4, cols.size(), f) != cols.size())
    emu::die("graph");
  fclose(f);
  const uint32_t blocks = static_cast<uint32_t>(atoi(argv[2]));
  Ctl ctl{};
  std::vector<unsigned long long> part(2 * kSymPoints * blocks, 0xa5a5a5a5a5a5a5a5ull);
  KArgs a{};
  a.offsets = offsets.data();
  a.cols = cols.data();
  a.n = static_cast<uint32_t>(nm[0]);
  a.m = static_cast<uint32_t>(nm[1]);
  a.ctl = &ctl;
  a.pull_min = 1;
  a.fr[1].node = reinterpret_cast<int32_t*>(part.data());
  for (int i = 0; i < kSymPoints; ++i) a.sym_x[i] = static_cast<double>((1ull << 52) + std::stoull(argv[3 + i]));
  if (blocks == 0) {
    const size_t words = (a.n + 31) / 32;
    std::vector<int32_t> levels(a.n), node(a.n), estart(a.n), tile(a.m / kMinTile + 2);
    std::vector<uint32_t> visited(words), seen0(words), seen1(words), filter(kXcds * words), eprefix(a.n);
    a.levels = levels.data();
    a.visited = visited.data();
    a.seen[0] = seen0.data();
    a.seen[1] = seen1.data();
    a.xfilter = filter.data();
    a.words = static_cast<uint32_t>(words);
    a.fr[0] = Frontier{};
    a.fr[0].node = node.data();
    a.fr[0].eprefix = eprefix.data();
    a.fr[0].estart = estart.data();
    a.fr[0].tile_node = tile.data();
    a.tile_cap = a.m / kMinTile + 2;
    ctl.sym_no = 7u;
    emu::launch(2, kBlock, [=] { k_init<false, false>(a, 0); });
    printf("%d\n", ctl.sym_no == 0 ? 1 : 0);
    return ctl.sym_no > 1;
  }
  ctl.ctr[0] = (1ull << 32) | a.m;
  for (int launch = 0; launch < 2; ++launch)  // the second one, in another place, is not to do it again
    emu::launch(blocks, kBlock, [=] { k_bfs_sym<true>(a, 3 * launch); });
  printf("%d\n", ctl.sym_run == 1 && ctl.sym_no == 0 ? 1 : 0);
  if (ctl.sym_run != 1 || ctl.xstat[0][11] != blocks) emu::die("not run once");
  return 0;
}
