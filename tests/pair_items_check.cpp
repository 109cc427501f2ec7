// Host check of the pair kernels' work items: the counts that size the grids against
// the decoding that the workgroups do, for jobs that may and may not take the shared
// form, every waves-per-workgroup choice and odd numbers of tiles and splits.
#include <cstdio>
#include <set>
#include <tuple>

#include "lingam_internal.h"

#define CHECK(c)                                          \
  do {                                                    \
    if (!(c)) {                                           \
      std::printf("line %d: %s\n", __LINE__, #c);         \
      return 1;                                           \
    }                                                     \
  } while (0)

int main() {
  for (const bool shared : {true, false})
    for (const int w : {1, 2, 4})
      for (const int tiles : {1, 3, 10})
        for (const int splits : {1, 2, 7}) {
          lg::JobStep s{};
          s.m = 100;
          s.learned = 1;
          lg::job_split(s, 64 * 64, 1, 256, lg::Tune{8, 8, w, w}, shared);
          s.ntiles = s.nct = s.nct2 = s.nct3 = tiles;
          s.nsplit = s.nsplit_c = s.nsplit_s = splits;
          const int n = tiles * splits * (4 / w) * (shared ? 1 : 2);
          for (const int kind : {lg::kKPair, lg::kKPairC, lg::kKPairE, lg::kKPairS})
            CHECK(lg::kind_count(s, kind) == n);
          // every (item, direction, quadrant) once
          std::set<std::tuple<int, int, int>> seen;
          for (int local = 0; local < n; ++local) {
            const lg::PairItem it = lg::pair_item_at(local, 4 / w, shared);
            CHECK(it.item >= 0 && it.item < tiles * splits);
            CHECK(it.part >= 0 && it.part < 4 / w);
            CHECK(it.half == 0 || (!shared && it.half == 1));
            for (int v = 0; v < w; ++v)
              CHECK(seen.insert({it.item, it.half, it.part * w + v}).second);
          }
          CHECK((int)seen.size() == tiles * splits * 4 * (shared ? 1 : 2));
        }
  std::printf("ok\n");
  return 0;
}
