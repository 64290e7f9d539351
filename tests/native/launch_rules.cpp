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
    } else {
      return 1;
    }
  }
  return 0;
}
