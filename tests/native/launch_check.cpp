// Host-only check of the launchers' arguments (linked with the built library; no device): a launch without a filter bank
// and with a length that no kernel has is refused, whatever else its arguments hold.  Prints "ok".
#include <cstdio>

#include "internal.h"

int main() {
  es::Filter* f = new es::Filter();  // one filter, as every launch of one length passes
  for (int taps : {0, -2, 3, 18}) {
    es::TaskArgs a{};
    a.table = reinterpret_cast<const es::Task*>(0x1000);
    a.count = a.total_wg = a.vec = 1;
    for (int kind : {es::K_LP_DOWN, es::K_LP_UP})
      if (es::launch_level(kind, 2, taps, 1, a, 8, *f, nullptr) != hipErrorInvalidValue)
        return printf("level kind %d, %d taps: not refused\n", kind, taps), 1;
    es::TailArgs t{};
    t.table = reinterpret_cast<const es::TailTask*>(0x1000);
    t.count = t.total_wg = 1;
    if (es::launch_tail(3, 2, taps, t, 8, 0, *f, nullptr) != hipErrorInvalidValue)
      return printf("coarse, %d taps: not refused\n", taps), 1;
  }
  delete f;
  printf("ok\n");
  return 0;
}
