// Host check of the LDS a one-tile launch asks for: every level that a step of
// a block or of a lone node reads, lanes past the column's end included, lies
// inside it.  Follows the evaluation in kernels.hip: blocks step over at most
// two 64-level slices (one in the FP64 two-ring and the BF16 pairs, which have
// no blocks on longer steps), the nodes outside the blocks over one; kernels
// without blocks over the launch's slices, their nodes of other degrees over
// one.  A remainder of 1..32 levels is read without running past it.  In the
// batched kernel the FP64 divergence and gradient adjoint have no blocks, the
// FP64 pair only on one slice, FP32 scalar inputs only on one and two.
// Usage: tile_tail_check N nlev one|batched
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "launch.hpp"
#include "mesh.hpp"

using namespace atlasnabla;

int main(int argc, char** argv) {
  if (argc != 4) return 2;
  const bool batched = argv[3][0] == 'b';
  const int N = std::atoi(argv[1]), L = std::atoi(argv[2]);
  HostMesh m;
  build_host_mesh(N, 6371220.0, m);
  OpTables t;
  build_op_tables(m, t);
  const int ops[] = {OP_GRAD, OP_DIV, OP_GRADT, OP_DIVT, OP_LAP, OP_CURL, OP_CURLT, OP_GRADLAP, OP_DIVCURL, OP_DIVGRADT};
  int bad = 0;
  for (int dtype = 0; dtype < (batched ? 2 : 3); ++dtype)
    for (int op : ops)
      for (int k = 0; k < 8; ++k) {
        const int slices = k & 3;
        Shape ask;
        ask.slices_per_iter = slices;
        ask.tile_kb = k < 4 ? 0 : 160;   // the default, and whole columns up to some hundred levels
        const Shape sh = resolve_shape(op, dtype, L, m.V, ask);
        if (batched && op >= OP_LAP && op != OP_DIVGRADT) continue;
        if (sh.lds_tiles != 3 || !uses_tiles(op, dtype, L, sh)) continue;
        const TileGeom g = tile_geom(op, dtype, L, sh);
        if (g.KL < 1) continue;
        HaloTiles ht;
        build_halo_tiles(m, t, g.ring, sh.band_rows, sh.run_nodes, g.col_bytes, g.row_bytes, g.budget, ht);
        std::vector<int32_t> nblk;
        group_blocks(t, g.block, ht, nblk);
        const bool bf = dtype == DT_BF16, dual = kernel_op(op) == OP_DIVCURL, two = g.ring == 2;
        const int cin = dual || kernel_op(op) == OP_DIV || kernel_op(op) == OP_GRADT ? 2 : 1;
        const int64_t el = (dtype == DT_F64 ? 8 : bf ? 2 : 4) * cin;
        const int U = tile_slices(g.KL, sh);
        int64_t tile_lds = 0;
        for (int64_t tl = 0; tl < ht.ntiles; ++tl)
          tile_lds = std::max(tile_lds, ht.info[4 * tl + 2] * g.col_bytes + ht.info[4 * tl + 3] * g.row_bytes);
        const int64_t lds = tile_lds + (bf ? 16 : 0) + tile_tail_bytes(op, dtype, g.KL, L, U, batched ? TileForm::kBatched : TileForm::kOneTile);
        if (lds > 160 * 1024) ++bad;
        const bool in_batched = dtype == DT_F64 ? cin == 1 || (dual && U == 1) : cin == 2 || U < 3;
        const bool blocks = g.block > 0 && !(bf && dual && U > 1) && (!batched || in_batched);
        const int bu = (dtype == DT_F64 && two) || (bf && dual) ? 1 : 2;
        int64_t worst = 0, over = 0;
        for (int klc : {g.KL, L - (L - 1) / g.KL * g.KL}) {
          const int rem = klc & 63, kmain = rem != 0 && rem <= 32 ? klc - rem : klc;
          if (kmain == 0) continue;
          auto upto = [&](int64_t step) { return (kmain + 64 * step - 1) / (64 * step) * 64 * step; };
          for (int64_t tl = 0; tl < ht.ntiles; ++tl) {
            const int n = ht.info[4 * tl + 3];
            std::vector<int64_t> col;   // LDS offset of every column
            int64_t cur = n * g.row_bytes;
            if (bf) cur += (ht.info[4 * tl + 2] * 4 + 15) / 16 * 16;
            for (int s = ht.info[4 * tl]; s < ht.info[4 * tl + 4]; ++s) {
              const int64_t g0 = ht.segs[2 * s] * (int64_t)L * el, cnt = ht.segs[2 * s + 1];
              const int64_t mis = bf ? g0 & 3 : 0;
              for (int64_t c = 0; c < cnt; ++c) col.push_back(cur + mis + c * klc * el);
              cur += bf ? ((g0 + cnt * klc * el + 3) & ~(int64_t)3) - (g0 - mis) : cnt * klc * el;
            }
            const int in_blocks = blocks ? nblk[tl] * g.block : 0;
            for (int q = 0; q < n; ++q) {
              const uint16_t* l = &ht.loc[(size_t)ht.stride * ht.order[ht.info[4 * tl + 1] + q]];
              const int ne = l[ht.stride - 1] >> kLocCountShift;
              int last = l[ht.stride - 1] & kMaxTileCols;
              for (int s = 0; s < ne; ++s) last = std::max<int>(last, l[s]);
              int64_t step = 1;
              if (q < in_blocks) step = std::min(U, bu);
              else if (!blocks && (two ? ne <= 18 : ne == 6)) step = U;
              const int64_t end = col[last] + upto(step) * el;
              worst = std::max(worst, end);
              over += end > lds;
            }
          }
        }
        if (over) {
          ++bad;
          std::printf("op %d dtype %d x %d (%d slices): %lld nodes read up to %lld of %lld bytes\n", op, dtype, L, U,
                      (long long)over, (long long)worst, (long long)lds);
        }
      }
  std::printf(bad ? "FAILED\n" : "OK\n");
  return bad ? 1 : 0;
}
