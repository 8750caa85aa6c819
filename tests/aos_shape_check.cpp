// Host-side check of the staged AoS step's launch shape (launch.h): for each
// line "integrator aligned n stride block" read from standard input, prints
// the records per tile and the threads per workgroup.
#include <stdio.h>

#include "launch.h"

int main() {
  int integ, aligned, stride, block;
  long long n;
  while (scanf("%d %d %lld %d %d", &integ, &aligned, &n, &stride, &block) == 5) {
    const int tile = soax::aos_shape(integ, aligned != 0, n, stride, &block);
    printf("%d %d\n", tile, block);
  }
  return 0;
}
