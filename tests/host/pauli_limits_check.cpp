// Host checks of Pauli-sum plans at their limits (no GPU).  Argument:
//   plan  planning many groups takes less host time than two passes over the state per group
//         would at the rate of a large copy (0.3 of one pass on the machine that this was written
//         on; 2.5 when tiles grew over all groups).
//   grid  launches over batches start no workgroups beyond a batch item's chunks of 256 outputs,
//         expectations of few chunks in all up to 128 that share them.
//   order  plans without tiles keep the groups' order.
//   coefficients  of the largest size stay finite in the tables of expectations.
// Exit status 0 when the check holds.
#include <cmath>
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
    if (!(host <= 2.0 * passes) || plan.size() > groups.size()) bad = 1;
  }
  return bad;
}

static int check_coefficients() {
  int bad = 0;
  for (int n : {9, 20, 24})
    for (double c : {0.5, 8.9e307, 1.7e308}) {
      // two x masks; on the higher one, one term or two that sum up to within the range
      const uint64_t x[3] = {1, 1ull << (n - 1), 1ull << (n - 1)}, z[3] = {0, 0, 6};
      const double co[3] = {1.0, c, 0.25 * c};
      const qsv_pauli_sum h{c < 1e308 ? 3u : 2u, co, x, z};
      const auto groups = group_pauli_sum(&h);
      for (const PauliLaunch& L : plan_pauli(groups, n, QSV_C128, false)) {
        if (L.kind == PL_GROUP) continue;
        std::vector<PauliMultiGroup> mg;
        std::vector<PauliMultiTerm> mt;
        pauli_multi_tables(groups, L, n, false, mg, mt);
        for (const PauliMultiGroup& g : mg) {
          double f = 0.0;
          for (int e = 0; e < g.n_re + g.n_im; ++e) f += mt[g.first + e].c;
          if (!std::isfinite(f)) {
            printf("n=%d c=%g: factor %g\n", n, c, f);
            bad = 1;
          }
          if (c == 0.5 && g.x >> 6 && !g.half) bad = 1;  // ordinary sums keep their half passes
        }
      }
    }
  return bad;
}

static int check_order() {
  std::mt19937_64 rng(9);
  int bad = 0;
  for (int n : {23, 24, 28})
    for (int first : {0, 1}) {
      // all pairs of Z (one diagonal group) with one X, or with strings too wide for a tile
      for (int wide : {0, 5}) {
        std::vector<uint64_t> x, z;
        for (int a = 0; a < n; ++a)
          for (int b = 0; b < a; ++b) {
            x.push_back(0);
            z.push_back(1ull << a | 1ull << b);
          }
        std::vector<uint64_t> mx{1ull << (n - 1)};
        if (wide) mx.clear();
        for (int k = 0; k < wide; ++k) mx.push_back(((1ull << n) - 1) & ~(1ull << k));
        for (uint64_t m : mx) {
          x.insert(first ? x.begin() : x.end(), m);
          z.insert(first ? z.begin() : z.end(), 0);
        }
        const std::vector<double> c(x.size(), 0.5);
        const qsv_pauli_sum h{x.size(), c.data(), x.data(), z.data()};
        const auto groups = group_pauli_sum(&h);
        const auto plan = plan_pauli(groups, n, n == 23 ? QSV_C128 : QSV_C64, false);
        if (plan.size() != groups.size()) bad = 1;
        for (size_t i = 0; i < plan.size(); ++i)
          if (plan[i].kind != PL_GROUP || plan[i].groups[0] != (int32_t)i) bad = 1;
      }
    }
  return bad;
}

static int check_grid() {
  int bad = 0;
  for (int n = 1; n <= 34; ++n)
    for (size_t batch : {1, 2, 3, 100, 127, 128, 5000, 65535})
      for (bool lambda : {false, true}) {
        const uint64_t chunks = ((1ull << n) + 255) / 256, b = pauli_multi_blocks(n, batch, lambda);
        const bool shared = !lambda && chunks * batch < 128;
        // whole workgroups per chunk, all of them with work, enough of them
        if (b < 1 || b > 2048 || (b > chunks && (!shared || b % chunks || b * batch > 128)) ||
            (shared && 2 * b * batch <= 128) || (!shared && b != std::min<uint64_t>(chunks, 2048))) {
          printf("n=%d batch=%zu lambda=%d: %zu workgroups\n", n, batch, (int)lambda, (size_t)b);
          bad = 1;
        }
      }
  return bad;
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!strcmp(what, "plan")) return check_plan();
  if (!strcmp(what, "coefficients")) return check_coefficients();
  if (!strcmp(what, "order")) return check_order();
  if (!strcmp(what, "grid")) return check_grid();
  return 2;
}
