// Test driver (host only): evaluates the library's launch rules
// (paper_2605_07612_amd/csrc/launch_rules.h) on queries read from stdin and
// prints one number per query.
//
//   planes f64 n_cu n_sets {N blocks} ...   planes per stage work item
//   slabs configured N planes               k-slabs per tile in a batch
//   weno blocks N n_cu                      planes per WENO5 workgroup
//   advect blocks N n_cu                    log2 of an advection block's slabs
//   ghost records face_values n_cu          workgroups per ghost record
#include <cstdio>
#include <cstring>
#include <vector>

#include "launch_rules.h"

int main() {
  char what[16];
  while (std::scanf("%15s", what) == 1) {
    if (!std::strcmp(what, "planes")) {
      int f64, cu, n;
      if (std::scanf("%d %d %d", &f64, &cu, &n) != 3) return 2;
      std::vector<f4::BlockSet> sets(n);
      for (auto &s : sets) {
        long b;
        if (std::scanf("%d %ld", &s.N, &b) != 2) return 2;
        s.blocks = b;
      }
      std::printf("%d\n", f4::slab_planes(sets.data(), sets.size(), f64 != 0, cu));
    } else if (!std::strcmp(what, "slabs")) {
      int c, N, p;
      if (std::scanf("%d %d %d", &c, &N, &p) != 3) return 2;
      std::printf("%d\n", f4::batch_slabs(c, N, p));
    } else {
      long a, b;
      int cu;
      if (std::scanf("%ld %ld %d", &a, &b, &cu) != 3) return 2;
      if (!std::strcmp(what, "weno")) std::printf("%d\n", f4::weno_planes(a, (int)b, cu));
      else if (!std::strcmp(what, "advect")) std::printf("%d\n", f4::advect_log2_slabs(a, (int)b, cu));
      else if (!std::strcmp(what, "ghost")) std::printf("%d\n", f4::ghost_split(a, b, cu));
      else return 3;
    }
  }
  return 0;
}
