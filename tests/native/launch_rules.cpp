// Prints what the launch rules (lbm_plan.h) decide: one query a line on standard input, one
// answer a line.
#include <cstdio>
#include <cstring>

#include "lbm_plan.h"

int main() {
  char what[32];
  while (std::scanf("%31s", what) == 1) {
    if (!std::strcmp(what, "waves_by_node")) {  // nwaves ngroups longest Q nx rows
      lbm::WaveTable t{};
      int Q, nx;
      long long rows;
      if (std::scanf("%d %d %d %d %d %lld", &t.nwaves, &t.ngroups, &t.longest, &Q, &nx, &rows) != 6)
        return 1;
      std::printf("%d\n", (int)lbm::waves_by_node(t, Q, nx, rows));
    } else if (!std::strcmp(what, "multi_plan")) {  // nx ny wy bytes lds_cu lds_block ncu
      int nx, ny, wy, elem, cu, block, ncu;
      if (std::scanf("%d %d %d %d %d %d %d", &nx, &ny, &wy, &elem, &cu, &block, &ncu) != 7)
        return 1;
      const lbm::MultiPlan p = lbm::multi_plan(nx, ny, wy != 0, (size_t)elem,
                                               lbm::workgroup_lds(cu, block), ncu);
      std::printf("%d %d %d %d %d %d %u\n", p.K, p.wx, p.ox, p.oy, p.ntx, p.nty, p.lds);
    } else if (!std::strcmp(what, "multi_rows")) {  // ny oy K wy
      int ny, oy, K, wy;
      if (std::scanf("%d %d %d %d", &ny, &oy, &K, &wy) != 4) return 1;
      std::printf("%lld\n", (long long)lbm::multi_rows(ny, oy, K, wy != 0));
    } else if (!std::strcmp(what, "batch_pays")) {  // bytes K tiles rows blocks nodes ncu
      int elem, K, ncu;
      long long tiles, rows, blocks, nodes;
      if (std::scanf("%d %d %lld %lld %lld %lld %d", &elem, &K, &tiles, &rows, &blocks, &nodes,
                     &ncu) != 7)
        return 1;
      std::printf("%d\n", (int)lbm::multi_pays(lbm::BATCH_RATES, (size_t)elem, K, tiles, rows,
                                                blocks, nodes, ncu));
    } else if (!std::strcmp(what, "default_launch")) {  // Q bytes nx ny buffers across_x walls
      int Q, elem, nx, ny, across_x, walls;
      long long bytes;
      if (std::scanf("%d %d %d %d %lld %d %d", &Q, &elem, &nx, &ny, &bytes, &across_x, &walls) != 7)
        return 1;
      const lbm::StepLaunch l = lbm::default_launch(Q, (size_t)elem, nx, ny, (size_t)bytes,
                                                    across_x != 0, walls != 0);
      std::printf("%d %d %d %d\n", l.bx, l.by, l.variant, (int)lbm::linear_blocks(nx, l.bx, l.by));
    } else if (!std::strcmp(what, "rows_plain")) {  // Q bytes across_x walls
      int Q, elem, across_x, walls;
      if (std::scanf("%d %d %d %d", &Q, &elem, &across_x, &walls) != 4) return 1;
      std::printf("%d\n", (int)lbm::rows_plain(Q, (size_t)elem, across_x != 0, walls != 0));
    } else if (!std::strcmp(what, "pieces")) {  // n size -> count, last start, last length
      long long n;
      int size, count = 0, start = 0, length = 0;
      if (std::scanf("%lld %d", &n, &size) != 2) return 1;
      lbm::each_piece(n, size, [&](int i, int len) {
        ++count;
        start = i;
        length = len;
      });
      std::printf("%d %d %d %d\n", count, start, length, n ? lbm::ceil_div((int)n, size) : 0);
    } else if (!std::strcmp(what, "batch_grid")) {  // blocks_per_cu ncu ntiles
      int bpc, ncu, ntiles;
      if (std::scanf("%d %d %d", &bpc, &ncu, &ntiles) != 3) return 1;
      std::printf("%d\n", lbm::batch_grid(bpc, ncu, ntiles));
    } else {
      return 1;
    }
  }
  return 0;
}
