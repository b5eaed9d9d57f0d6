// The first factor pool of a stored ACA against the caller's budget.
#include <stdio.h>

#include "../paper_2505_08174_amd/csrc/internal.h"

int main() {
  int bad = 0;
  for (size_t es : {4, 8})
    for (int64_t est = 1000; est < (1ll << 33); est = est * 3 / 2 + 1)
      for (int g : {1, 2, 3})                 // terms that the tolerance suggests / 20
        for (int w : {3, 4})                  // l_max / 20
          for (double share : {0.5, 0.45, 0.2, 0.01}) {   // est of the budget, at most half
            const size_t budget = (size_t)((double)est * es / share) + 4096;
            const int64_t p = first_pool(est, g * est, w * est, es, budget);
            const bool room = (double)w * est * es <= 0.5 * budget && w * est * es <= (1ll << 30);
            if (p < est || (double)p * es > 0.5 * budget + 4096 || (room && p != w * est)) {
              printf("est %lld guess %dx worst %dx share %g: pool %lld of %zu bytes\n",
                     (long long)est, g, w, share, (long long)p, budget);
              ++bad;
            }
          }
  if (!bad) printf("ok\n");
  return bad != 0;
}
