// The dt of a batched step with one dt per box: a bad dt in one box stops the
// step, and every other box still reports its own dt of that step, in every
// order of the wavefronts; a call that was stopped before reports zeros.
#include "workgroup_emulator.h"

#include <algorithm>
#include <cmath>

#include "ctmhd_workgroup.h"

int main() {
  constexpr int kBoxes = 300, kPhases = 2;
  int bad = 0, runs = 0;
  for (int given = 0; given < 2; ++given)
    for (int where : {0, 63, 64, 130, 255, 256, 299})
      for (int before = 0; before < 2; ++before) {
        int order[4] = {0, 1, 2, 3};
        do {
          std::vector<double> fixed(kBoxes), dt(kBoxes, -1.0), out(kBoxes, -1.0);
          std::vector<unsigned long long> slots(2 * kBoxes);
          std::vector<int> nflag(4 * kBoxes, 0), done(kPhases * kBoxes, 7), cursor(4, 7);
          for (int b = 0; b < kBoxes; ++b) {
            fixed[b] = 1e-3 * (b + 1);
            // the CFL maximum: of the fix-up where one ran
            nflag[4 * b + 2] = b % 3 == 0;
            slots[2 * b] = __double_as_longlong(2.0 + b);
            slots[2 * b + 1] = __double_as_longlong(5.0 + b);
          }
          fixed[where] = std::nan("");
          slots[2 * where] = slots[2 * where + 1] = __double_as_longlong(std::nan(""));
          std::vector<double> want(kBoxes);
          for (int b = 0; b < kBoxes; ++b)
            want[b] = given ? fixed[b]
                            : 0.3 / __longlong_as_double(
                                        (long long)slots[2 * b + (nflag[4 * b + 2] ? 1 : 0)]);
          int stop = before, err = 0;
          long long diag[4] = {9, 9, 9, 9};
          if (!emu::run(order, [&] {
                ctmhd::k_bdt_final(kBoxes, kPhases, 1, 0, slots.data(), nflag.data(), done.data(),
                                   cursor.data(), 0.3, given ? fixed.data() : nullptr, dt.data(),
                                   out.data(), &stop, &err, diag);
              })) {
            std::printf("the workgroup does not finish\n");
            return 1;
          }
          int wrong = stop != 1 || diag[0] || diag[1] || diag[2] || diag[3] != 1;
          for (int b = 0; b < kBoxes; ++b) {
            const double w = before ? 0.0 : want[b];
            wrong += std::memcmp(&out[b], &dt[b], 8) != 0 ||
                     !(out[b] == w || (std::isnan(out[b]) && std::isnan(w)));
            wrong += slots[2 * b] != 0 || slots[2 * b + 1] != 0 || nflag[4 * b + 2] != 0;
          }
          if (wrong) {
            if (bad < 8)
              std::printf("order %d%d%d%d, bad box %d, %s dt: %d wrong values\n", order[0],
                          order[1], order[2], order[3], where, given ? "given" : "CFL", wrong);
            ++bad;
          }
          ++runs;
        } while (std::next_permutation(order, order + 4));
      }
  std::printf("%d runs, %d wrong\n", runs, bad);
  return bad != 0;
}
