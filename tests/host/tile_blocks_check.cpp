// Host check of the blocks of a tiling (group_blocks): every tile keeps its
// nodes, the blocks lead its stretch of the order, and the column of every
// stencil entry of a block's node b lies where the kernel looks for it: at
// the first node's position of that row plus b, in LDS and in the mesh.
// Usage: tile_blocks_check N ring tile_rows sweep_bands block_nodes budget
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "mesh.hpp"

using namespace atlasnabla;

int main(int argc, char** argv) {
  if (argc != 7) return 2;
  const int N = std::atoi(argv[1]), ring = std::atoi(argv[2]), H = std::atoi(argv[3]), R = std::atoi(argv[4]),
            NB = std::atoi(argv[5]);
  HostMesh m;
  build_host_mesh(N, 6371220.0, m);
  OpTables t;
  build_op_tables(m, t);
  HaloTiles ht;
  build_halo_tiles(m, t, ring, H, R, 548, 96, std::atoll(argv[6]), ht);
  const std::vector<int32_t> before = ht.order;
  std::vector<int32_t> nblk;
  group_blocks(t, NB, ht, nblk);
  int bad = 0;
  long long in_blocks = 0;
  for (int64_t tl = 0; tl < ht.ntiles; ++tl) {
    const int pos0 = ht.info[4 * tl + 1], n = ht.info[4 * tl + 3];
    std::vector<int32_t> a(before.begin() + pos0, before.begin() + pos0 + n),
        b(ht.order.begin() + pos0, ht.order.begin() + pos0 + n);
    if (nblk[tl] * NB > n) ++bad;
    std::sort(a.begin(), a.end());
    std::vector<int32_t> c = b;
    std::sort(c.begin(), c.end());
    if (a != c) ++bad;
    for (int q = 0; q < nblk[tl]; ++q) {
      in_blocks += NB;
      const uint16_t* l0 = &ht.loc[(size_t)ht.stride * b[q * NB]];
      const int self0 = l0[ht.stride - 1] & kMaxTileCols;
      // row positions of the first node, and each entry's row and offset
      const int up = l0[0], lo = l0[4], uu = ring == 2 ? l0[6] : 0, ll = ring == 2 ? l0[15] : 0;
      for (int k = 0; k < NB; ++k) {
        const int32_t i = b[q * NB + k];
        if (i != b[q * NB] + k) ++bad;
        const uint16_t* l = &ht.loc[(size_t)ht.stride * i];
        const int want[18] = {up, up + 1, self0 - 1, self0 + 1, lo, lo + 1,
                              uu, uu + 1, uu + 2, up - 1, up + 2, self0 - 2, self0 + 2,
                              lo - 1, lo + 2, ll, ll + 1, ll + 2};
        const int ne = ring == 1 ? 6 : 18;
        if ((l[ht.stride - 1] >> kLocCountShift) != ne || (l[ht.stride - 1] & kMaxTileCols) != self0 + k) ++bad;
        for (int s = 0; s < ne; ++s)
          if (l[s] != want[s] + k) ++bad;
      }
    }
  }
  std::printf("O%d ring %d: %lld tiles, %lld of %lld nodes in blocks of %d\n", N, ring, (long long)ht.ntiles, in_blocks,
              (long long)m.V, NB);
  // most nodes are regular, and tiles of this budget several nodes wide
  if (NB > 0 && N >= 32 && std::atoll(argv[6]) >= 40000 && in_blocks * 2 < (long long)m.V) ++bad;
  std::printf(bad ? "FAILED\n" : "OK\n");
  return bad ? 1 : 0;
}
