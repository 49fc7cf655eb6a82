// Host-only check of the rule that picks AdamW's four-wide form: every array at 16
// bytes, the copy at 8 or more.  Nothing is launched.  Exit status 1 on a violation.
#include <cstdio>
#include "update.hip"
int main() {
  int bad = 0;
  alignas(16) static char mem[64];
  auto at = [&](int off) { return (const void *)(mem + off); };
  for (int off = 0; off < 16; off += 4) {
    const void *x[4] = {at(0), at(0), at(0), at(0)};
    for (int k = 0; k < 4; ++k) {
      x[k] = at(off);
      bad += adamw_vec(x[0], x[1], x[2], x[3], nullptr) != (off == 0);
      x[k] = at(0);
    }
    bad += adamw_vec(at(0), at(0), at(0), at(0), at(off)) != (off % 8 == 0);
  }
  printf("violations: %d\n", bad);
  return bad != 0;
}
