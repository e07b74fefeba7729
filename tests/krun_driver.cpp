// Checks the padded contracted order (csrc/planner.cpp, padded_k_runs) over
// many mode lists: every contracted index counts exactly once, the entries
// that do not count repeat elements of the same run, and every chunk is u
// consecutive indices of one run of the first mode.
#include <cstdio>
#include <vector>

#include "internal.hpp"

using namespace famlies;

int main() {
  long checked = 0;
  for (int u : {2, 4})
    for (long e = 1; e <= 70; ++e)
      for (long rest : {1L, 2L, 7L})
        for (int unit = 0; unit < 4; ++unit) {
          Analysis an;
          an.esize = 16 / u;
          an.x_kfast = an.y_kfast = true;
          an.K = e * rest;
          an.P.push_back({0, e, unit & 1 ? 1 : 5, unit & 2 ? 1 : -1, 0});
          if (rest > 1) an.P.push_back({1, rest, 1000, 2000, 0});
          const int64_t n = padded_k_length(an, u);
          const bool want = unit != 0 && e >= u && 4 * ((e + u - 1) / u * u) <= 5 * e;
          if ((n != 0) != want) return std::printf("length u %d e %ld unit %d: %ld\n", u, e, unit, (long)n), 1;
          if (!n) continue;
          KRuns kr;
          padded_k_runs(an, u, &kr);
          if ((int64_t)kr.index.size() != n || (int64_t)kr.skip.size() != n || n % u) return std::printf("size\n"), 1;
          std::vector<int> count((size_t)an.K, 0);
          for (int64_t i = 0; i < n; ++i) {
            const int64_t k = kr.index[(size_t)i];
            if (k < 0 || k >= an.K) return std::printf("range\n"), 1;
            if (kr.skip[(size_t)i] == 0) ++count[(size_t)k];
            const int64_t c = i / u * u, j = i % u;
            if (k != kr.index[(size_t)c] + j || k / e != kr.index[(size_t)c] / e) return std::printf("run\n"), 1;
            if (j == u - 1 && kr.skip[(size_t)i]) return std::printf("skip\n"), 1;
          }
          for (int v : count)
            if (v != 1) return std::printf("count u %d e %ld rest %ld\n", u, e, rest), 1;
          ++checked;
        }
  std::printf("checked %ld\n", checked);
  return 0;
}
