// resident_pays for triples "n64 n128 source" on standard input, one answer per line.
#include "resident_rule.hpp"

#include <cstdio>

int main() {
  int a, b, s;
  while (std::scanf("%d %d %d", &a, &b, &s) == 3) std::printf("%d\n", (int)ttsh::resident_pays(a, b, s != 0));
  return 0;
}
