// Host checks of Pauli-sum plans at their limits (no GPU).  Argument:
//   plan  planning many groups takes less host time than one pass over the state per group would
//         at the rate of a large copy.
// Exit status 0 when the check holds.
#include <cstdio>
#include <cstring>
#include <ctime>
#include <random>

#include "engine.h"
using namespace qsv;

static std::vector<PauliGroup> random_groups(int n, int terms, int weight, std::mt19937_64& rng) {
  std::vector<double> c(terms, 1.0);
  std::vector<uint64_t> x(terms, 0), z(terms, 0);
  for (uint64_t& m : x)
    while (__builtin_popcountll(m) < weight) m |= 1ull << (rng() % n);
  const qsv_pauli_sum h{(size_t)terms, c.data(), x.data(), z.data()};
  return group_pauli_sum(&h);
}

static int check_plan() {
  std::mt19937_64 rng(3);
  int bad = 0;
  for (int weight : {2, 6, 9}) {
    const int n = 24;
    const auto groups = random_groups(n, 40000, weight, rng);
    const std::clock_t t0 = std::clock();
    const auto plan = plan_pauli(groups, n, QSV_C64, false);
    const double host = (double)(std::clock() - t0) / CLOCKS_PER_SEC;
    const double passes = (double)groups.size() * 8.0 * (1ull << n) / 4.9e12;
    std::vector<char> seen(groups.size(), 0);
    for (const PauliLaunch& L : plan)
      for (int32_t g : L.groups) bad |= seen[g]++ != 0;
    for (char v : seen) bad |= !v;
    printf("weight %d: %zu groups in %zu launches, planned in %.0f ms (a pass each: %.0f ms)\n", weight, groups.size(),
           plan.size(), 1e3 * host, 1e3 * passes);
    if (!(host <= passes) || plan.size() > groups.size()) bad = 1;
  }
  return bad;
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!strcmp(what, "plan")) return check_plan();
  return 2;
}
