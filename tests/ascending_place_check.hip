// Host check of ascending_place (csrc/common.h), whose results index memory in
// the eigensolves: a permutation for every input, ascending where no value is NaN.
#include "../paper_2603_10295_amd/csrc/common.h"

#include <cmath>
#include <cstdio>
#include <vector>

int main() {
  uint64_t x = 1;
  auto next = [&] { return (x = x * 6364136223846793005ull + 1442695040888963407ull) >> 33; };
  int bad = 0;
  for (int n = 1; n <= 256; n += n < 40 ? 1 : 27)
    for (int kind = 0; kind < 6; ++kind) {
      std::vector<double> v(n);
      for (double& e : v) {
        e = (double)(next() % 17) - 8.0;            // ties
        if (kind >= 1 && next() % 4 == 0) e = kind == 1 ? HUGE_VAL : -HUGE_VAL;
        if (kind >= 3 && next() % 3 == 0) e = NAN;
        if (kind == 5) e = NAN;
      }
      if (kind == 4) v[n - 1] = NAN;
      std::vector<int> at(n, -1);
      bool nan = false;
      for (int i = 0; i < n; ++i) {
        const int p = ephw::ascending_place([&](int j) { return v[j]; }, n, i);
        nan = nan || std::isnan(v[i]);
        if (p < 0 || p >= n || at[p] >= 0) ++bad;
        else at[p] = i;
      }
      for (int p = 1; p < n && !nan && bad == 0; ++p)
        if (v[at[p - 1]] > v[at[p]] || (v[at[p - 1]] == v[at[p]] && at[p - 1] > at[p])) ++bad;
    }
  if (bad) std::printf("%d values out of place\n", bad);
  else std::printf("ascending_place_check: ok\n");
  return bad ? 1 : 0;
}
