// Whether the table of logarithms of the wave analysis serves a largest
// count: reads lines "lnt_n mx" (decimal) on stdin, prints 0 or 1 for each.
#include <cstdio>

#include "dpsnn_internal.h"

int main() {
  unsigned n, mx;
  while (std::scanf("%u %u", &n, &mx) == 2) std::printf("%d\n", (int)dpsnn::lnt_covers(n, mx));
  return 0;
}
