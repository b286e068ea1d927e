// Host check of what plans compute (no GPU).  Random circuits of every gate kind and layered ones
// are planned as states and batches of circuits plan them, the records are interpreted
// (plan_replay.h) on a random state, and the result is compared with the circuit gate by gate in
// long double: forward plans of both amplitude types (the records of one serve the other's
// arithmetic, done here in double), with and without relayout, for launches of few and of many
// tiles; reverse sweeps with their gradients.  States of the largest amplitudes go through chains
// like small ones.  Exit status 0 when every check holds.
#include <cstdio>
#include <random>

#include "plan_replay.h"
using namespace replay;

namespace {

const int kAngles[QSV_GATE_KIND_COUNT] = {0, 0, 0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1, 1, 3, 0, 0, 0};
const int kTargets[QSV_GATE_KIND_COUNT] = {1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 2, 2, 2, 1, 2, 1, 2};

struct Circ {
  std::vector<qsv_gate> gates;
  std::vector<double> mats;
  qsv_circuit c{};
  void finish(int n) { c = qsv_circuit{n, 0, gates.data(), gates.size(), mats.data(), mats.size()}; }
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

// d x d unitary by Gram-Schmidt.
void push_unitary(Circ& k, qsv_gate& g, int d, std::mt19937_64& rng) {
  std::normal_distribution<double> nd;
  std::vector<std::vector<cplx>> col(d, std::vector<cplx>(d));
  for (int j = 0; j < d; ++j) {
    for (cplx& z : col[j]) z = cplx(nd(rng), nd(rng));
    for (int rep = 0; rep < 2; ++rep)
      for (int i = 0; i < j; ++i) {
        cplx dot = 0.0;
        for (int r = 0; r < d; ++r) dot += std::conj(col[i][r]) * col[j][r];
        for (int r = 0; r < d; ++r) col[j][r] -= dot * col[i][r];
      }
    double nrm = 0.0;
    for (const cplx& z : col[j]) nrm += std::norm(z);
    for (cplx& z : col[j]) z /= std::sqrt(nrm);
  }
  g.matrix_offset = (int64_t)(k.mats.size() / 2);
  for (int r = 0; r < d; ++r)
    for (int j = 0; j < d; ++j) {
      k.mats.push_back(col[j][r].real());
      k.mats.push_back(col[j][r].imag());
    }
}

void random_circuit(Circ& k, int n, int count, int n_params, std::mt19937_64& rng) {
  std::uniform_real_distribution<double> u(-3.0, 3.0);
  for (int i = 0; i < count; ++i) {
    int kind = (int)(rng() % QSV_GATE_KIND_COUNT);
    if (rng() % 6 == 0) kind = QSV_GATE_X;
    qsv_gate g = blank(kind, (int)(rng() % n));
    if (kTargets[kind] == 2)
      do g.targets[1] = (int)(rng() % n); while (g.targets[1] == g.targets[0]);
    uint64_t used = 1ull << g.targets[0] | (g.targets[1] >= 0 ? 1ull << g.targets[1] : 0);
    for (int j = (int)(rng() % 4) - 1; j > 0 && __builtin_popcountll(used) < n; --j) {
      int q;
      do q = (int)(rng() % n); while (used >> q & 1);
      used |= 1ull << q;
      g.ctrl_mask |= 1ull << q;
    }
    for (int a = 0; a < kAngles[kind]; ++a) {
      if (rng() % 4) g.param_index[a] = (int)(rng() % n_params);
      g.param_coeff[a] = rng() % 2 ? 1.0 : -0.5;
      g.angle_const[a] = u(rng);
    }
    if (kind == QSV_GATE_MAT1 || kind == QSV_GATE_MAT2) push_unitary(k, g, kind == QSV_GATE_MAT1 ? 2 : 4, rng);
    k.gates.push_back(g);
  }
  k.finish(n);
}

// Layers of one-qubit gates between CZs and now and then a CX or a swap: chains, blocks, runs of
// phases on one qubit before, between and after its gates.
void layered_circuit(Circ& k, int n, int layers, std::mt19937_64& rng) {
  const int kinds[] = {QSV_GATE_MAT1, QSV_GATE_U3, QSV_GATE_RY, QSV_GATE_RZ, QSV_GATE_S, QSV_GATE_Z, QSV_GATE_H,
                       QSV_GATE_T, QSV_GATE_RX};
  std::uniform_real_distribution<double> u(-3.0, 3.0);
  for (int l = 0; l < layers; ++l) {
    for (int q = 0; q < n; ++q)
      for (int rep = 0; rep < 1 + (int)(rng() % 3); ++rep) {
        qsv_gate g = blank(l % 3 == 0 ? QSV_GATE_MAT1 : kinds[rng() % 9], q);
        for (int a = 0; a < kAngles[g.kind]; ++a) g.angle_const[a] = u(rng);
        if (g.kind == QSV_GATE_MAT1) push_unitary(k, g, 2, rng);
        k.gates.push_back(g);
      }
    for (int a = l % 2; a + 1 < n; a += 2) {
      qsv_gate g = blank(rng() % 5 ? QSV_GATE_Z : QSV_GATE_X, a + 1);
      g.ctrl_mask = 1ull << a;
      k.gates.push_back(g);
    }
    if (l % 4 == 3) {
      qsv_gate g = blank(QSV_GATE_SWAP, 0);
      g.targets[1] = n - 1;
      k.gates.push_back(g);
    }
  }
  k.finish(n);
}

std::vector<lcplx> gate_by_gate(const Circ& k, const std::vector<double>& params, std::vector<lcplx> x) {
  for (const qsv_gate& g : k.gates) {
    long double a[3];
    angles_of(g, params, a);
    apply_definition(x, g, definition(&k.c, g, a));
  }
  return x;
}

std::vector<cplx> random_state(int n, std::mt19937_64& rng) {
  std::normal_distribution<double> nd;
  std::vector<cplx> x((size_t)1 << n);
  double s = 0.0;
  for (cplx& z : x) s += std::norm(z = cplx(nd(rng), nd(rng)));
  for (cplx& z : x) z /= std::sqrt(s);
  return x;
}
std::vector<lcplx> wide(const std::vector<cplx>& x) { return std::vector<lcplx>(x.begin(), x.end()); }
double distance(const std::vector<cplx>& x, const std::vector<lcplx>& y) {
  long double s = 0.0L;
  for (size_t k = 0; k < x.size(); ++k) s += std::norm(lcplx(x[k]) - y[k]);
  return (double)std::sqrt(s);
}

long g_plans = 0, g_flips = 0, g_phases = 0, g_chains = 0, g_blocks = 0, g_remaps = 0, g_half = 0, g_one = 0, g_grads = 0;
int g_bad = 0;
double g_largest = 0.0;

void count(const Plan& p, const Machine& m) {
  ++g_plans;
  g_flips += m.flips;
  g_phases += m.phases;
  g_chains += m.chains;
  g_blocks += m.blocks;
  g_remaps += m.remaps;
  for (const DevPass& dp : p.passes) (p.adjoint ? g_one : g_half) += dp.alt;
}

// The plans a state of n qubits (tile >= 9) or a batch of circuits (any tile) makes.
std::vector<PlanOptions> options(int n, bool adjoint) {
  std::vector<PlanOptions> all;
  for (int dtype : {QSV_C64, QSV_C128}) {
    if (n >= 9) {
      for (int tile = 9; tile <= std::min(n, 11); ++tile)
        for (size_t batch : {(size_t)1, (size_t)4096})
          for (bool relayout : {false, true}) {
            if (adjoint && (batch > 1 || relayout)) continue;
            all.push_back(state_plan_options(dtype, n, tile, tile, adjoint, true, relayout, batch));
          }
    }
    PlanOptions o = state_plan_options(dtype, 9, 9, 9, adjoint, true, false);  // the type's rules
    o.tile_qubits = std::min(n, 4 + n % 4);
    o.low_qubits = 2;
    o.rb_min = 4;
    o.reg_bits = 3;
    o.blocks = false;
    all.push_back(o);
  }
  return all;
}

void check_forward(const Circ& k, int n, const std::vector<double>& params, std::mt19937_64& rng, const char* what) {
  const std::vector<cplx> psi = random_state(n, rng);
  const std::vector<lcplx> ref = gate_by_gate(k, params, wide(psi));
  for (const PlanOptions& o : options(n, false)) {
    const Plan p = build_plan(&k.c, false, o);
    double err = 1.0;
    try {
      Machine m(p, &k.c, params, psi);
      err = distance(m.v, ref);
      count(p, m);
    } catch (const std::exception& e) {
      printf("%s n=%d: %s\n", what, n, e.what());
    }
    if (!(err <= 1e-15 * (20.0 + k.gates.size()))) {
      printf("%s n=%d dtype=%d tile=%d low=%d relayout=%d half=%d: off by %.2e\n", what, n, o.dtype, o.tile_qubits,
             o.low_qubits, (int)o.relayout, (int)o.half_remap, err);
      g_bad = 1;
    }
  }
}

// psi = U x and a random lambda: the sweep gives x, U^+ lambda, and d/dp 2 Re <lambda|U(p) x>.
void check_reverse(const Circ& k, int n, const std::vector<double>& params, std::mt19937_64& rng, const char* what) {
  const std::vector<cplx> x = random_state(n, rng), lam = random_state(n, rng);
  const std::vector<lcplx> end = gate_by_gate(k, params, wide(x));
  std::vector<cplx> psi;
  for (const lcplx& z : end) psi.push_back(cplx((double)z.real(), (double)z.imag()));
  std::vector<lcplx> back = wide(lam);
  for (size_t i = k.gates.size(); i-- > 0;) {
    long double a[3];
    angles_of(k.gates[i], params, a);
    const std::vector<lcplx> m = definition(&k.c, k.gates[i], a);
    const int d = m.size() == 16 ? 4 : 2;
    std::vector<lcplx> t(m.size());
    for (int r = 0; r < d; ++r)
      for (int q = 0; q < d; ++q) t[r * d + q] = std::conj(m[q * d + r]);
    apply_definition(back, k.gates[i], t);
  }
  std::vector<long double> grad(params.size(), 0.0L);
  for (size_t i = 0; i < k.gates.size(); ++i)
    for (int s = 0; s < 3; ++s) {
      const qsv_gate& g = k.gates[i];
      if (g.param_index[s] < 0) continue;
      std::vector<lcplx> y = wide(x);
      for (size_t e = 0; e < k.gates.size(); ++e) {
        long double a[3];
        angles_of(k.gates[e], params, a);
        std::vector<lcplx> m = definition(&k.c, k.gates[e], a);
        if (e == i) {
          const long double h = 1e-6L;
          a[s] += h;
          const std::vector<lcplx> up = definition(&k.c, g, a);
          a[s] -= 2 * h;
          const std::vector<lcplx> dn = definition(&k.c, g, a);
          for (size_t j = 0; j < m.size(); ++j) m[j] = (up[j] - dn[j]) / (2 * h);
        }
        apply_definition(y, k.gates[e], m, e == i);
      }
      long double dot = 0.0L;
      for (size_t j = 0; j < y.size(); ++j) dot += (std::conj(lcplx(lam[j])) * y[j]).real();
      grad[g.param_index[s]] += 2 * g.param_coeff[s] * dot;
    }
  for (const PlanOptions& o : options(n, true)) {
    const Plan p = build_plan(&k.c, true, o);
    double err = 1.0, gerr = 1.0;
    try {
      Machine m(p, &k.c, params, psi, lam);
      err = std::max(distance(m.v, wide(x)), distance(m.w, back));
      gerr = 0.0;
      for (size_t q = 0; q < grad.size(); ++q) gerr = std::max(gerr, std::abs(m.grad[q] - (double)grad[q]));
      ++g_grads;
      count(p, m);
    } catch (const std::exception& e) {
      printf("%s n=%d: %s\n", what, n, e.what());
    }
    // (the central differences of the reference are good to h^2 / 24 and 1e-19 / h, below 1e-12)
    if (!(err <= 1e-15 * (20.0 + k.gates.size())) || !(gerr <= 1e-10)) {
      printf("%s reverse n=%d dtype=%d tile=%d low=%d: off by %.2e, gradient %.2e\n", what, n, o.dtype, o.tile_qubits,
             o.low_qubits, err, gerr);
      g_bad = 1;
    }
  }
}

// Chains store amplitudes up to 2^(kChainGates n) times their size: a state of the largest
// amplitudes that leave room for it comes out as its small copy does, bit for bit.
void check_scale() {
  const int n = 10;
  std::mt19937_64 rng(5);
  for (int kind = 0; kind < 2; ++kind) {
    Circ k;
    for (int l = 0; l < 50; ++l) {
      for (int q = 0; q < n; ++q) {
        qsv_gate g = blank(kind ? QSV_GATE_MAT1 : QSV_GATE_U3, q);
        if (kind) {
          push_unitary(k, g, 2, rng);
        } else {
          g.angle_const[0] = M_PI / 2;
          g.angle_const[2] = M_PI / 4;
        }
        k.gates.push_back(g);
      }
      for (int a = l % 2; a + 1 < n; a += 2) {
        qsv_gate g = blank(QSV_GATE_Z, a + 1);
        g.ctrl_mask = 1ull << a;
        k.gates.push_back(g);
      }
    }
    k.finish(n);
    const Plan p = build_plan(&k.c, false, state_plan_options(QSV_C128, n, 9, 9, false, true, false));
    const std::vector<cplx> psi = random_state(n, rng);  // (amplitudes below 1)
    std::vector<cplx> big = psi;
    const double up = std::ldexp(1.0, 1023 - kChainGates * n - 1);
    for (cplx& z : big) z *= up;
    const Machine small(p, &k.c, {}, psi), large(p, &k.c, {}, big);
    if (!(small.largest <= std::ldexp(1.0, kChainGates * n))) {
      printf("stored amplitudes up to %.2e\n", small.largest);
      g_bad = 1;
    }
    for (size_t i = 0; i < psi.size(); ++i)
      if (large.v[i] != small.v[i] * up) g_bad = 1;
    if (g_bad) printf("scaled state, kind %d\n", kind);
    if (kind == 0) g_largest = small.largest;
  }
}

// Numbers that neighbours share are looked up only where gates may share their angle: layers of RX
// with one parameter, equal or shifted angles, against RY and RZ with parameters of their own.
void check_shared() {
  const int n = 9;
  std::mt19937_64 rng(8);
  for (int kind = 0; kind < 3; ++kind) {
    Circ k;
    const int layers = 3;
    for (int l = 0; l < layers; ++l) {
      for (int q = 0; q < n; ++q) {
        qsv_gate g = blank(kind < 2 ? QSV_GATE_RX : q % 2 ? QSV_GATE_RY : QSV_GATE_RX, q);
        g.param_index[0] = kind < 2 ? l : n * l + q;
        g.param_coeff[0] = 1.0;
        if (kind == 1) g.angle_const[0] = 0.25 * (q / 3);
        k.gates.push_back(g);
      }
      qsv_gate z = blank(QSV_GATE_Z, 0);
      z.ctrl_mask = 2;
      k.gates.push_back(z);
    }
    k.finish(n);
    std::vector<double> params(n * layers);
    for (double& v : params) v = std::uniform_real_distribution<double>(-3.0, 3.0)(rng);
    int marked = 0;
    for (bool adjoint : {false, true}) {
      const Plan p = build_plan(&k.c, adjoint, state_plan_options(QSV_C128, n, 9, 9, adjoint, true, false));
      for (const Fill& f : p.fills) marked += f.kind == F_PRIM_MATRIX && f.count > 0;
    }
    if (kind < 2 ? marked < layers * (n - 1) : marked != 0) {
      printf("layers of kind %d: %d gates look for their neighbour's numbers\n", kind, marked);
      g_bad = 1;
    }
    check_forward(k, n, params, rng, "shared angles");
    check_reverse(k, n, params, rng, "shared angles");
  }
}

}  // namespace

int main() {
  std::mt19937_64 rng(62);
  try {
    for (int n : {4, 5, 6, 7, 8, 9, 10, 11, 12}) {
      for (int rep = 0; rep < (n <= 9 ? 6 : 2); ++rep) {
        std::vector<double> params(5);
        for (double& v : params) v = std::uniform_real_distribution<double>(-3.0, 3.0)(rng);
        Circ a, b;
        random_circuit(a, n, 70, 5, rng);
        validate_circuit(&a.c, params.size(), n);
        check_forward(a, n, params, rng, "random");
        layered_circuit(b, n, 12, rng);
        validate_circuit(&b.c, params.size(), n);
        check_forward(b, n, params, rng, "layered");
        Circ r;
        random_circuit(r, n, n <= 9 ? 40 : 24, 5, rng);
        check_reverse(r, n, params, rng, "random");
      }
    }
    check_scale();
    check_shared();
  } catch (const Error& e) {
    printf("planner error %d: %s\n", e.status, e.msg.c_str());
    return 2;
  }
  printf("plans replayed %ld (gradients %ld): flips %ld, phase runs %ld, chain gates %ld, blocks %ld, remaps %ld, "
         "passes with halved remaps %ld, with single phases %ld; stored amplitudes up to %.1e\n",
         g_plans, g_grads, g_flips, g_phases, g_chains, g_blocks, g_remaps, g_half, g_one, g_largest);
  return g_bad || g_plans < 300 || g_flips < 1000 || g_phases < 1000 || g_chains < 500 || g_blocks < 100 ||
         g_remaps < 500 || g_half < 20 || g_one < 20;
}
