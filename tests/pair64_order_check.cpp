// Host check of the FP64 pair kernel's item order: the samples that each XCD gets, in
// batches of jobs of even and uneven lengths.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "lingam_internal.h"

struct Job {
  int d, n;
};

// Most samples of an XCD over their mean, workgroups dispatched round-robin.
static double imbalance(const std::vector<Job>& jobs, int t) {
  std::vector<long long> len;  // of every item in the schedule's order
  long long pairs = 0;
  int64_t lo = INT64_MAX, hi = 0;
  std::vector<lg::JobStep> js;
  for (const Job& j : jobs) {
    js.push_back(lg::job_step_base(j.d, t));
    const int64_t p = lg::pairs64(js.back());
    pairs += p;
    if (p > 0) {
      lo = std::min<int64_t>(lo, j.n);
      hi = std::max<int64_t>(hi, j.n);
    }
  }
  for (size_t k = 0; k < jobs.size(); ++k) {
    lg::job_split64(js[k], pairs, 256);
    len.insert(len.end(), lg::kind_count(js[k], lg::kKP64), jobs[k].n);
  }
  const int g = (int)len.size();
  std::vector<char> seen(g, 0);
  long long load[8] = {0}, sum = 0;
  for (int b = 0; b < g; ++b) {
    const int at = lg::xcd_ranges64(lo, hi) ? lg::xcd_item(b, g) : b;
    if (at < 0 || at >= g || seen[at]) return 1e9;  // not a permutation
    seen[at] = 1;
    load[b & 7] += len[at];
    sum += len[at];
  }
  return 8.0 * (double)*std::max_element(load, load + 8) / (double)sum;
}

int main() {
  std::vector<std::vector<Job>> batches(5);
  for (int k = 0; k < 50; ++k) batches[0].push_back({50, 1000});
  for (int k = 0; k < 64; ++k) batches[1].push_back({30 + (k * 7) % 35, k % 8 ? 500 : 20000});
  for (int k = 0; k < 40; ++k) batches[2].push_back({8 + (k * 11) % 57, 500 + 115 * k});
  for (int k = 0; k < 30; ++k) batches[3].push_back({60, 5000 + 15 * k});
  for (int k = 0; k < 30; ++k) batches[4].push_back({60, k < 15 ? 1000 : 1150});
  for (size_t b = 0; b < batches.size(); ++b)
    for (const int t : {0, 2}) {
      const double x = imbalance(batches[b], t);
      if (!(x <= 1.1)) {
        std::printf("batch %zu step %d: %.3f\n", b, t, x);
        return 1;
      }
    }
  std::printf("ok\n");
  return 0;
}
