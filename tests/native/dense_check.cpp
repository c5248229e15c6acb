// Host-only check of the row levels behind the coarse kernel's matrix products: for every axis length and number of
// levels, the stacked rows of the levels and nothing past them.  Prints "ok <axes>".
#include <cstdio>

#include "composite.h"

int main() {
  int axes = 0;
  for (int n = 2; n <= es::kDenseSide; n += 2) {
    for (int K = 1; K <= es::kDenseLevels && n % (1 << K) == 0; ++K) {
      int r = 0;
      for (int i = 1; i <= K; ++i)
        for (int k = 0; k < n >> i; ++k, ++r)
          if (es::dense_level(n, r) != i) return printf("n %d K %d row %d: level %d, not %d\n", n, K, r, es::dense_level(n, r), i), 1;
      for (; r < n; ++r)
        if (es::dense_level(n, r) <= K) return printf("n %d K %d row %d: level %d past the last\n", n, K, r, es::dense_level(n, r)), 1;
      ++axes;
    }
  }
  // the most levels that a block of the longest sides has below it: 2^(K + 1) divides them
  int most = 0;
  while (es::kDenseSide % (1 << (most + 2)) == 0) ++most;
  if (most != es::kDenseLevels) return printf("%d levels, tables for %d\n", most, es::kDenseLevels), 1;
  printf("ok %d\n", axes);
  return 0;
}
