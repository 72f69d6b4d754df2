// Which workgroups the blocks of a launch take (xcd.hpp), over launches of many
// sizes: every workgroup exactly once, and no XCD more than its share of either
// leading kind by more than one, where these are more than stay on one XCD.
// Then the cap of workgroups per CU by unused LDS.
#include <cstdio>
#include <vector>

#include "xcd.hpp"

using namespace mf;
using namespace mf::wave;

static int fail(const char* what, int nwg, int lead, int lead2) {
  printf("FAIL %s: %d workgroups, %d + %d leading\n", what, nwg, lead, lead2);
  return 1;
}

int main() {
  const XcdRuns runs[3] = {kNoRuns, {3000, 5}, {40, 1}};
  const int counts[] = {0, 1, 7, 8, 9, 31, 32, 33, 40, 64, 65, 200, 777};
  for (const XcdRuns& r : runs)
    for (int lead : counts)
      for (int lead2 : counts)
        for (int rest : counts) {
          const int nwg = lead + lead2 + rest, grid = xcd_grid(nwg, lead, lead2, r);
          std::vector<int> seen(nwg, 0);
          int share[2][kXCD] = {};
          for (int b = 0; b < grid; ++b) {
            const int n = xcd_wg_at(b, nwg, lead, lead2, r);
            if (n < -1 || n >= nwg) return fail("workgroup out of range", nwg, lead, lead2);
            if (n < 0) continue;
            ++seen[n];
            if (n < lead + lead2) ++share[n < lead ? 0 : 1][b % kXCD];
          }
          for (int s : seen)
            if (s != 1) return fail("workgroup not taken once", nwg, lead, lead2);
          if (nwg >= r.from) continue;
          for (int k = 0; k < 2; ++k) {
            const int l = k == 0 ? lead : lead2;
            if (xcd_head(nwg, l) == 0 || (k == 1 && lead > 0 && xcd_head(nwg, lead) == 0)) continue;
            for (int q = 0; q < kXCD; ++q)
              if (share[k][q] > (l + kXCD - 1) / kXCD) return fail("one XCD takes too many", nwg, lead, lead2);
          }
        }
  for (int n = 1; n <= 8; ++n)
    for (int own : {0, 64, 4096, 4160, 8192}) {
      const int bytes = own + lds_cap(5000, 3000, n, own);
      const int granted = (bytes + kLdsStep - 1) / kLdsStep * kLdsStep;
      if (kLdsPerCu / granted != n) return printf("FAIL cap %d with %d bytes: %d\n", n, own, kLdsPerCu / granted), 1;
    }
  if (lds_cap(2999, 3000, 4, 0) != 0 || lds_cap(5000, 3000, 0, 0) != 0) return printf("FAIL no cap\n"), 1;
  printf("OK\n");
  return 0;
}
