// Prints the odd-p plans and tile shapes of csrc/pass_geom.h:
//   plan p f64 m d0,r,wdig,le ...
//   shape p f64 le rd kt kt3
#include <stdio.h>

#include "pass_geom.h"

int main() {
  for (int p : {3, 5, 7})
    for (int f64 = 0; f64 < 2; ++f64) {
      int64_t n = p;
      for (int m = 1; n <= (int64_t(1) << 26); ++m, n *= p) {
        printf("plan %d %d %d", p, f64, m);
        for (const fdwt::PassGeom& g : fdwt::odd_plan(p, m, f64)) {
          int64_t tiles = n;
          for (int i = 0; i < g.le; ++i) tiles /= p;
          printf(" %d,%d,%d,%d,%d", g.d0, g.r, g.wdig, g.le, (int)fdwt::odd_kt3(p, f64, g.le, tiles));
        }
        printf("\n");
      }
      for (int le = 1; le <= 9; ++le)
        for (int rd = 1; rd <= le; ++rd)
          if (fdwt::odd_has_shape(p, f64, le, rd))
            printf("shape %d %d %d %d %d %d\n", p, f64, le, rd, fdwt::odd_kt(p, le, rd, f64),
                   (int)(p == 3 && !f64 && fdwt::odd_kt3_shape(le, rd)));
    }
  return 0;
}
