// Host check of the rounding errors of complex128 forward plans (no GPU): layered circuits planned
// with a state's options and replayed (plan_replay.h), with the gates drawn anew in every
// layer or the same in all of them (where errors of the tables add up), against long double
// arithmetic on the gates' matrices in double.  Two measures, root mean squares over trials: the
// distance of the states and the drift of the norm.
//
//   fixed  layers of gates that plans run one by one (RY RZ, RX RZ, H T, T H RY): no further off
//          than each gate in double by itself.  Tables of their products, rounded to double, are up
//          to 10 (states) and 60 (norms) times further off.
//   chain  layers of general gates (U3, explicit unitaries): closer than the same gates split
//          one by one in double, the phases between them carried in double (2 to 15 times closer;
//          carries formed in double from the numbers before rounding are 1.0 to 1.2 times as
//          far off).
//
// Argument: fixed or chain.  Exit status 0 when every family holds.
#include <cstdio>
#include <cstring>
#include <random>

#include "plan_replay.h"
using namespace replay;

namespace {

const int N = 9;

struct Layers {
  std::vector<qsv_gate> gates;
  std::vector<double> mats;
};

qsv_gate blank(int kind, int q) {
  qsv_gate g{};
  g.kind = kind;
  g.targets[0] = q;
  g.targets[1] = -1;
  g.matrix_offset = -1;
  for (int a = 0; a < 3; ++a) g.param_index[a] = -1;
  return g;
}

std::vector<cplx> numbers(const Layers& k, const qsv_gate& g) {  // in double, as a program forms them
  const double h = 0.5 * g.angle_const[0], r = std::sqrt(0.5);
  const cplx i(0, 1);
  switch (g.kind) {
    case QSV_GATE_X: return {0, 1, 1, 0};
    case QSV_GATE_Z: return {1, 0, 0, -1};
    case QSV_GATE_RY: return {std::cos(h), -std::sin(h), std::sin(h), std::cos(h)};
    case QSV_GATE_RX: return {std::cos(h), -i * std::sin(h), -i * std::sin(h), std::cos(h)};
    case QSV_GATE_RZ: return {std::polar(1.0, -h), 0, 0, std::polar(1.0, h)};
    case QSV_GATE_T: return {1, 0, 0, std::polar(1.0, M_PI / 4)};
    case QSV_GATE_H: return {r, r, r, -r};
    case QSV_GATE_U3: {
      const double th = g.angle_const[0], ph = g.angle_const[1], la = g.angle_const[2];
      const double c = std::cos(th / 2), s = std::sin(th / 2);
      return {std::polar(c, -(ph + la) / 2), std::polar(1.0, -(ph - la) / 2) * -s, std::polar(1.0, (ph - la) / 2) * s,
              std::polar(c, (ph + la) / 2)};
    }
    default: {
      std::vector<cplx> m;
      for (int e = 0; e < 4; ++e) m.push_back(cplx(k.mats[2 * (g.matrix_offset + e)], k.mats[2 * (g.matrix_offset + e) + 1]));
      return m;
    }
  }
}

struct Family {
  const char* name;
  std::vector<int> kinds;
};

// again: 0 gates drawn anew, 1 one gate for every qubit and layer, 2 one per qubit.
// cx: a CX ladder after each layer, else CZ bricks.
Layers draw(const Family& f, int again, bool cx, int layers, std::mt19937_64& rng) {
  std::uniform_real_distribution<double> u(0.0, 2 * M_PI);
  std::normal_distribution<double> nd;
  Layers k;
  std::vector<std::vector<qsv_gate>> kept(N);
  for (int l = 0; l < layers; ++l) {
    for (int q = 0; q < N; ++q) {
      const bool fresh = again == 0 || (l == 0 && (again == 2 || q == 0));
      if (fresh) kept[q].clear();
      for (size_t e = 0; fresh && e < f.kinds.size(); ++e) {
        qsv_gate g = blank(f.kinds[e], q);
        for (double& a : g.angle_const) a = u(rng);
        if (g.kind == QSV_GATE_MAT1) {
          cplx a0(nd(rng), nd(rng)), a1(nd(rng), nd(rng)), b0(nd(rng), nd(rng)), b1(nd(rng), nd(rng));
          for (int rep = 0; rep < 2; ++rep) {
            const double na = std::sqrt(std::norm(a0) + std::norm(a1));
            a0 /= na;
            a1 /= na;
            const cplx d = std::conj(a0) * b0 + std::conj(a1) * b1;
            b0 -= d * a0;
            b1 -= d * a1;
            const double nb = std::sqrt(std::norm(b0) + std::norm(b1));
            b0 /= nb;
            b1 /= nb;
          }
          g.matrix_offset = (int64_t)(k.mats.size() / 2);
          for (const cplx& z : {a0, b0, a1, b1}) {
            k.mats.push_back(z.real());
            k.mats.push_back(z.imag());
          }
        }
        kept[q].push_back(g);
      }
      for (qsv_gate g : kept[again == 1 ? 0 : q]) {
        g.targets[0] = q;
        k.gates.push_back(g);
      }
    }
    for (int a = cx ? 0 : l % 2; a + 1 < N; a += cx ? 1 : 2) {
      qsv_gate g = blank(cx ? QSV_GATE_X : QSV_GATE_Z, a + 1);
      g.ctrl_mask = 1ull << a;
      k.gates.push_back(g);
    }
  }
  return k;
}

template <typename F>
void pairs(std::vector<cplx>& x, const qsv_gate& g, F f) {
  const uint64_t t = 1ull << g.targets[0];
  for (uint64_t k = 0; k < x.size(); ++k)
    if (!(k & t) && (k & g.ctrl_mask) == g.ctrl_mask) f(x[k], x[k | t]);
}

void by_itself(std::vector<cplx>& x, const Layers& k, const qsv_gate& g) {
  const std::vector<cplx> m = numbers(k, g);
  pairs(x, g, [&](cplx& a, cplx& b) {
    if (g.kind == QSV_GATE_X) std::swap(a, b);
    else if (g.kind == QSV_GATE_RY || g.kind == QSV_GATE_H) real_form(m.data(), a, b);
    else if (g.kind == QSV_GATE_RX) x_form(m.data(), a, b);
    else if (m[1] == 0.0 && m[2] == 0.0) {
      if (m[0] != 1.0) times(a, m[0]);
      times(b, m[3]);
    } else general(m.data(), a, b);
  });
}

// General gates one by one: M = diag(l0, l1) [[c, -s], [s, c]] diag(1, p), l carried to the
// qubit's next gate, its last gate whole; all in double.
std::vector<cplx> split_in_double(const Layers& k, std::vector<cplx> x) {
  std::vector<int> left(N, 0);  // gates up to the end of the chain: the qubit's next X, or the last
  std::vector<std::vector<int>> chains(N, std::vector<int>(1, 0));
  for (const qsv_gate& g : k.gates) {
    if (g.kind == QSV_GATE_U3 || g.kind == QSV_GATE_MAT1) ++chains[g.targets[0]].back();
    else if (g.kind == QSV_GATE_X) chains[g.targets[0]].push_back(0);
  }
  std::vector<size_t> at(N, 0);
  for (int q = 0; q < N; ++q) left[q] = chains[q][0];
  std::vector<cplx> carry(2 * N, 1.0);
  for (const qsv_gate& g : k.gates) {
    const int q = g.targets[0];
    if (g.kind != QSV_GATE_U3 && g.kind != QSV_GATE_MAT1) {
      by_itself(x, k, g);
      if (g.kind == QSV_GATE_X) left[q] = chains[q][++at[q]];
      continue;
    }
    std::vector<cplx> m = numbers(k, g);
    for (int e = 0; e < 4; ++e) m[e] *= carry[2 * q + (e & 1)];
    if (--left[q] == 0) {
      pairs(x, g, [&](cplx& a, cplx& b) { general(m.data(), a, b); });
      carry[2 * q] = carry[2 * q + 1] = 1.0;
      continue;
    }
    const double a = std::abs(m[0]), b = std::abs(m[2]), nrm = std::hypot(a, b);
    carry[2 * q] = m[0] / a;
    carry[2 * q + 1] = m[2] / b;
    const cplx p = a >= b ? m[3] / carry[2 * q + 1] : -m[1] / carry[2 * q];
    const cplx out[4] = {cplx(a / nrm, -b / nrm), cplx(b / nrm, a / nrm), p / std::abs(p), 0.0};
    pairs(x, g, [&](cplx& y, cplx& z) { chained(out, y, z); });
  }
  return x;
}

struct Error2 {
  double state = 0.0, norm = 0.0;  // sums of squares
  int n = 0;
  void add(const std::vector<cplx>& x, const std::vector<lcplx>& ref) {
    long double d = 0.0L, a = 0.0L, b = 0.0L;
    for (size_t k = 0; k < x.size(); ++k) {
      d += std::norm(lcplx(x[k]) - ref[k]);
      a += std::norm(lcplx(x[k]));
      b += std::norm(ref[k]);
    }
    state += (double)d;
    norm += (double)((a / b - 1.0L) * (a / b - 1.0L));
    ++n;
  }
};

}  // namespace

int main(int argc, char** argv) {
  const bool chain = argc > 1 && !strcmp(argv[1], "chain");
  const std::vector<Family> families =
      chain ? std::vector<Family>{{"U3", {QSV_GATE_U3}},
                                  {"unitaries", {QSV_GATE_MAT1}},
                                  {"U3 twice", {QSV_GATE_U3, QSV_GATE_U3}},
                                  {"three", {QSV_GATE_MAT1, QSV_GATE_U3, QSV_GATE_MAT1}}}
            : std::vector<Family>{{"RY RZ", {QSV_GATE_RY, QSV_GATE_RZ}},
                                  {"RX RZ", {QSV_GATE_RX, QSV_GATE_RZ}},
                                  {"H T", {QSV_GATE_H, QSV_GATE_T}},
                                  {"T H RY", {QSV_GATE_T, QSV_GATE_H, QSV_GATE_RY}}};
  int bad = 0;
  for (const Family& f : families)
    for (int again = 0; again < 3; ++again)
      for (bool cx : {false, true}) {
        if (chain && cx && f.kinds.size() == 1) continue;  // (a CX ends its target's chain)
        Error2 plan, base;
        for (int trial = 0; trial < 10; ++trial) {
          std::mt19937_64 rng(7 + 100 * trial + 10 * again + cx);
          Layers k = draw(f, again, cx, 24, rng);
          const qsv_circuit c{N, 0, k.gates.data(), k.gates.size(), k.mats.data(), k.mats.size()};
          std::vector<cplx> zero((size_t)1 << N, 0.0);
          zero[0] = 1.0;
          std::vector<lcplx> ref(zero.begin(), zero.end());
          std::vector<cplx> one = zero;
          for (const qsv_gate& g : k.gates) {
            const std::vector<cplx> m = numbers(k, g);
            apply_definition(ref, g, std::vector<lcplx>(m.begin(), m.end()));
            by_itself(one, k, g);
          }
          if (chain) one = split_in_double(k, zero);
          const Plan p = build_plan(&c, false, state_plan_options(QSV_C128, N, 9, 9, false, true, false));
          plan.add(Machine(p, &c, {}, zero).v, ref);
          base.add(one, ref);
        }
        const double s = std::sqrt(plan.state / plan.n), s0 = std::sqrt(base.state / base.n);
        const double d = std::sqrt(plan.norm / plan.n), d0 = std::sqrt(base.norm / base.n);
        // ten trials of the same errors vary by a tenth (states) and a factor of two (norms, which
        // no table moves by more than its last bit)
        const double most_s = (chain ? 0.9 : 1.1) * s0, most_d = (chain ? 0.5 : 2.0) * d0 + 5e-16;
        printf("%-10s %s %s: states off by %.1e (single gates %.1e), norms by %.1e (%.1e)\n", f.name,
               again == 0 ? "anew " : again == 1 ? "one  " : "per q", cx ? "CX" : "CZ", s, s0, d, d0);
        if (!(s <= most_s) || !(d <= most_d)) {
          printf("  beyond %.1e and %.1e\n", most_s, most_d);
          bad = 1;
        }
      }
  return bad;
}
