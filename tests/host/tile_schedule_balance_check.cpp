// Host check of a tiling's schedule (schedule_tiles): the nodes of any two
// XCDs differ by at most two of the largest tile.
// Usage: tile_schedule_balance_check N ring tile_rows sweep_bands budget
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "mesh.hpp"

using namespace atlasnabla;

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const int N = std::atoi(argv[1]), ring = std::atoi(argv[2]), H = std::atoi(argv[3]), R = std::atoi(argv[4]);
  HostMesh m;
  build_host_mesh(N, 6371220.0, m);
  OpTables t;
  build_op_tables(m, t);
  HaloTiles ht;
  build_halo_tiles(m, t, ring, H, R, 264, 96, std::atoll(argv[5]), ht);
  std::vector<int32_t> sched;
  schedule_tiles(m, ht, ht.info, H, sched);
  long long nodes[8] = {};
  for (size_t k = 0; k + 4 <= sched.size(); k += 4) nodes[k / 4 % 8] += sched[k + 3];
  const long long lo = *std::min_element(nodes, nodes + 8), hi = *std::max_element(nodes, nodes + 8);
  std::printf("O%d ring %d: %lld tiles of at most %d nodes, XCDs of %lld to %lld nodes\n", N, ring,
              (long long)ht.ntiles, ht.max_nodes, lo, hi);
  const bool bad = hi - lo > 2 * ht.max_nodes;
  std::printf(bad ? "FAILED\n" : "OK\n");
  return bad ? 1 : 0;
}
