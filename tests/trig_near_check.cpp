// Host-side evaluation of the library's fp64 sincos (trig.h): reads doubles
// (hexadecimal, one a line) and prints the sine and the cosine of each, in
// hexadecimal.
#include <stdio.h>

#include "trig.h"

int main() {
  double x;
  while (scanf("%la", &x) == 1) {
    double s, c;
    soax::trig::sincos_fast(x, &s, &c);
    printf("%a %a\n", s, c);
  }
  return 0;
}
