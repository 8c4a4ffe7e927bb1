// Prints the pair exponents of csrc/pair_scale.h for
//   p m s gamma_1..gamma_s rp_0..rp_m   (on stdin, repeated)
#include <stdio.h>

#include "pair_scale.h"

int main() {
  int p, m, s;
  while (scanf("%d %d %d", &p, &m, &s) == 3) {
    std::vector<double> g(s), r(m + 1);
    for (double& v : g)
      if (scanf("%lf", &v) != 1) return 1;
    for (double& v : r)
      if (scanf("%lf", &v) != 1) return 1;
    std::vector<int32_t> ix(s);
    fdwt::pair_exponents(p, m, s, g.data(), r.data(), ix.data());
    for (int32_t x : ix) printf("%d ", x);
    printf("\n");
  }
  return 0;
}
