// The spreading's choice of strip size (spread_table_log) on the host: strips of
// 32 cells at any size of launch where they are spread by cells, from eight points
// in 128 cells on (band plans: sixteen); elsewhere the size of the launch decides.
#include <cstdio>

#include "../../paper_0901_1913_amd/csrc/spread.hip"

using namespace fchi2;

int main() {
  int bad = 0, checked = 0;
  for (int band = 0; band < 2; ++band)
    for (int logl = 11; logl <= 26; ++logl)
      for (int P : {2, 5, 12, 24})
        for (int nc : {1, 20, 400, 4000})
          for (int per128 : {0, 1, 3, 4, 7, 8, 15, 16, 30, 1000}) {  // points in 128 cells
            Geom g{};
            g.band = band;
            g.L = (int64_t)1 << logl;
            g.P = P;
            const int64_t n = per128 * (g.L / 128);
            const int64_t waves = (g.L >> 9) * P * nc;
            const int most = per128 >= 4 ? 65536 : per128 < 1 ? 0 : 20000;
            const bool small = per128 >= (band ? 16 : 8) || (4 * n >= g.L / 128 && waves < most);
            const int want = small ? kStripLogMin : kStripLogMax;
            ++checked;
            if (spread_table_log(g, nc, n, n) != want) {
              ++bad;
              printf("band %d L 2^%d P %d curves %d, %d points in 128 cells: not 2^%d\n", band,
                     logl, P, nc, per128, want);
            }
          }
  if (bad) return 1;
  printf("ALL OK (%d)\n", checked);
  return 0;
}
