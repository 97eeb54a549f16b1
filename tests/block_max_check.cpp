// The workgroup maximum behind the CFL signal, taken once per work item in a
// loop as the passes that share items out over a fixed grid do: every item's
// value must be its own maximum in every order of the wavefronts.
#include "workgroup_emulator.h"

#include <algorithm>
#include <cmath>

#include "ctmhd_workgroup.h"

int main() {
  constexpr int kItems = 5;
  int order[4] = {0, 1, 2, 3}, bad = 0, orders = 0;
  // signal of thread t of item i: the maximum sits in another wavefront and on
  // another scale from item to item; item 2 holds a NaN, item 3 only zeros
  auto signal = [](int i, int t) {
    if (i == 3) return 0.0;
    if (i == 2 && t == 77) return std::nan("");
    return (i == 0 ? 1.0 : i == 1 ? 100.0 : 10.0) + ((t * 37 + i * 91) % 256) / 256.0;
  };
  do {
    unsigned long long got[kItems];
    if (!emu::run(order, [&] {
          for (int i = 0; i < kItems; ++i) {
            const unsigned long long m = ctmhd::block_max_bits(signal(i, (int)threadIdx.x));
            if (threadIdx.x == 0) got[i] = m;
          }
        })) {
      std::printf("the workgroup does not finish\n");
      return 1;
    }
    for (int i = 0; i < kItems; ++i) {
      unsigned long long want = 0;
      for (int t = 0; t < 256; ++t)
        want = std::max(want, (unsigned long long)__double_as_longlong(signal(i, t)));
      if (got[i] != want) {
        std::printf("order %d%d%d%d item %d: %g, not %g\n", order[0], order[1], order[2], order[3],
                    i, __longlong_as_double((long long)got[i]),
                    __longlong_as_double((long long)want));
        ++bad;
      }
    }
    ++orders;
  } while (std::next_permutation(order, order + 4));
  std::printf("%d orders, %d wrong maxima\n", orders, bad);
  return bad != 0;
}
