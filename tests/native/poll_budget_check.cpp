// Host check of the bounded waits' poll count (the library's poll_budget.h, included
// verbatim): a limit of n polls allows exactly n, for limits on both sides of 32
// bits.  Long runs are shortened by taking all but the last polls before a multiple
// of 2^31 at once.
#include <stdio.h>

#define __host__
#define __device__
#include "poll_budget.h"

int main() {
  const unsigned long long limits[] = {1, 2, 31, 32, 33, 1ull << 21, 0x7ffffffeull, 0x7fffffffull, 0x80000000ull,
                                       0xfffffffeull, 0xffffffffull, 0x100000000ull, 0x100000009ull, 0x380000003ull};
  int bad = 0;
  for (unsigned long long n : limits) {
    auto left = n;
    unsigned long long taken = 0;
    for (;;) {
      const unsigned long long skip = (left & 0x7fffffffull) > 8 ? (left & 0x7fffffffull) - 4 : 0;
      left -= skip;
      taken += skip;
      if (!take_poll(&left)) break;
      ++taken;
    }
    if (taken != n || take_poll(&left)) {
      printf("limit %llu: %llu polls\n", n, taken);
      ++bad;
    }
  }
  printf("failures %d\n", bad);
  return bad ? 1 : 0;
}
