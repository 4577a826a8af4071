// Host check of a tiling's schedule (schedule_tiles): every tile is listed
// exactly once, with its own words, and the list comes in rounds of eight.
// Usage: tile_schedule_check N ring tile_rows sweep_bands budget
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
  build_halo_tiles(m, t, ring, H, R, 548, 96, std::atoll(argv[5]), ht);
  std::vector<int32_t> sched;
  schedule_tiles(m, ht, ht.info, H, sched);
  int bad = sched.size() % 32 != 0;
  std::vector<std::vector<int32_t>> a, b;
  for (size_t k = 0; k + 4 <= sched.size(); k += 4)
    if (sched[k + 3]) a.push_back({sched.begin() + k, sched.begin() + k + 4});
  for (int64_t k = 0; k < ht.ntiles; ++k) b.push_back({ht.info.begin() + 4 * k, ht.info.begin() + 4 * k + 4});
  std::sort(a.begin(), a.end());
  std::sort(b.begin(), b.end());
  if (a != b) ++bad;
  std::printf("O%d ring %d: %zu entries for %lld tiles\n%s\n", N, ring, sched.size() / 4, (long long)ht.ntiles,
              bad ? "FAILED" : "OK");
  return bad ? 1 : 0;
}
