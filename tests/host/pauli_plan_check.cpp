// Host check of the Pauli-sum launch plan and tables (no GPU): random sums on 1 to 34 qubits, both
// amplitude types, in order or not.  Every group is in exactly one launch, tile launches hold only
// x masks inside their tile, ordered plans keep the groups' order, and the factors read back from the
// group and term records (thread, outside and slot bits of random outputs, half sums) equal
// those of the terms.  Exit status 0 when every check holds.
#include <cstdio>
#include <random>

#include "engine.h"
using namespace qsv;

static int local_of(uint64_t y, uint64_t tile) {
  int r = 0;
  for (int b = 0; tile; ++b, tile &= tile - 1)
    if (y & tile & (~tile + 1)) r |= 1 << b;
  return r;
}

int main() {
  std::mt19937_64 rng(11);
  int bad = 0, tiles = 0, gathers = 0, singles = 0, halves = 0;
  for (int trial = 0; trial < 400 && !bad; ++trial) {
    const int n = 1 + trial % 34, terms = 1 + (int)(rng() % 70);
    std::vector<double> c(terms);
    std::vector<uint64_t> x(terms), z(terms);
    const uint64_t full = (1ull << n) - 1;
    for (int k = 0; k < terms; ++k) {
      c[k] = 0.25 * (1 + (int)(rng() % 8));  // exact in binary
      x[k] = z[k] = 0;
      const int loc = trial % 5 == 4 ? n : 1 + (int)(rng() % 4);
      for (int l = 0; l < loc; ++l) {
        const uint64_t q = 1ull << (rng() % n);
        const int p = (int)(rng() % 3);
        if (p != 2) x[k] |= q;
        if (p != 0) z[k] |= q;
      }
    }
    const qsv_pauli_sum h{(size_t)terms, c.data(), x.data(), z.data()};
    const auto groups = group_pauli_sum(&h);
    for (int dtype : {QSV_C64, QSV_C128})
      for (bool in_order : {false, true})
        for (bool lambda : {false, true}) {
          const auto plan = plan_pauli(groups, n, dtype, in_order);
          std::vector<int> seen(groups.size(), 0);
          int last = -1;
          for (const PauliLaunch& L : plan) {
            std::vector<PauliMultiGroup> mg;
            std::vector<PauliMultiTerm> mt;
            if (L.kind != PL_GROUP) pauli_multi_tables(groups, L, n, lambda, mg, mt);
            else if (L.groups.size() != 1) bad = 1;
            (L.kind == PL_TILE ? tiles : L.kind == PL_GATHER ? gathers : singles)++;
            for (size_t i = 0; i < L.groups.size(); ++i) {
              const int g = L.groups[i];
              ++seen[g];
              if (in_order && g < last) bad = 2;
              last = g;
              if (L.kind == PL_GROUP) continue;
              const PauliGroup& P = groups[g];
              if (L.kind == PL_TILE && ((P.xmask & ~L.tile) || __builtin_popcountll(L.tile) != kPauliTileQubits)) bad = 3;
              const int bits = L.kind == PL_TILE ? kPauliTileQubits : n;
              const int slots = L.kind == PL_TILE ? kPauliTileQubits - kPauliTileThreadBits : n >= kPauliGatherFour ? 2 : 0;
              for (int s = 0; s < 20; ++s) {
                const uint64_t y = rng() & full;
                const uint64_t ly = L.kind == PL_TILE ? (uint64_t)local_of(y, L.tile) : y;
                const uint64_t t = ly & ((1ull << (bits - slots)) - 1), k = ly >> (bits - slots);
                const uint64_t hi = L.kind == PL_TILE ? y & ~L.tile : 0;
                if (mg[i].half) {
                  ++halves;
                  if (lambda || !(mg[i].x & mg[i].half) || mg[i].half < 64) bad = 4;
                  if ((mg[i].half >> (bits - slots)) == 0 && mg[i].half >= (1ull << bits)) bad = 4;
                }
                double f[2] = {0, 0}, ref[2] = {0, 0};
                for (int e = 0; e < mg[i].n_re + mg[i].n_im; ++e) {
                  const PauliMultiTerm& m = mt[mg[i].first + e];
                  const int par = __builtin_popcountll(t & m.zt) + __builtin_popcountll(hi & m.zo) + __builtin_popcountll(k & m.pat);
                  f[e >= mg[i].n_re] += (par & 1) ? -m.c : m.c;
                }
                const uint64_t src = y ^ P.xmask;
                for (size_t e = 0; e < P.zmasks.size(); ++e) {
                  const double sg = (__builtin_popcountll(src & P.zmasks[e]) & 1) ? -1 : 1;
                  ref[0] += sg * P.cre[e];
                  ref[1] += sg * P.cim[e];
                }
                const double w = mg[i].half ? 2.0 : 1.0;
                if (f[0] != w * ref[0] || f[1] != w * ref[1]) bad = 5;
                const uint64_t lsrc = L.kind == PL_TILE ? (uint64_t)local_of(src, L.tile) : src;
                if ((ly ^ mg[i].x) != lsrc || (L.kind == PL_TILE && ((src ^ y) & ~L.tile))) bad = 6;
              }
            }
          }
          for (int v : seen)
            if (v != 1) bad = 7;
        }
    if (bad) printf("trial %d n=%d: check %d failed\n", trial, n, bad);
  }
  printf("launches: tiles %d, gathers %d, single groups %d; half sums %d\n", tiles, gathers, singles, halves);
  return bad || tiles < 100 || gathers < 100 || singles < 100 || halves < 100;
}
