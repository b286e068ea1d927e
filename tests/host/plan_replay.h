// An interpreter of register-blocked plans: it walks a plan's passes, op records, entries, layouts
// and bound tables as the tile kernels do (same fields, same branches, the multiply-adds of a
// gate in the same order) in double on the host, and knows nothing of how the planner made them.
// Below it, the same circuits gate by gate in long double, from the gates' definitions.
#pragma once
#include <cmath>
#include <complex>
#include <cstring>
#include <stdexcept>
#include <vector>

#include "engine.h"
#include "qsv_ops.h"

namespace replay {
using namespace qsv;


inline double fma3(double a, double b, double c) { return std::fma(a, b, c); }

// ---- the arithmetic of a gate on one pair of amplitudes -----------------------------------------
inline void general(const cplx* U, cplx& a0, cplx& a1) {
  const double x0 = a0.real(), y0 = a0.imag(), x1 = a1.real(), y1 = a1.imag();
  const double p0r = fma3(-U[0].imag(), y0, fma3(U[1].real(), x1, -U[1].imag() * y1));
  const double p0i = fma3(U[0].imag(), x0, fma3(U[1].real(), y1, U[1].imag() * x1));
  const double p1r = fma3(U[2].real(), x0, fma3(-U[2].imag(), y0, -U[3].imag() * y1));
  const double p1i = fma3(U[2].real(), y0, fma3(U[2].imag(), x0, U[3].imag() * x1));
  a0 = cplx(fma3(U[0].real(), x0, p0r), fma3(U[0].real(), y0, p0i));
  a1 = cplx(fma3(U[3].real(), x1, p1r), fma3(U[3].real(), y1, p1i));
}
inline void times(cplx& a, cplx p) {
  const double pr = -a.imag() * p.imag(), pi = a.real() * p.imag();
  a = cplx(fma3(p.real(), a.real(), pr), fma3(p.real(), a.imag(), pi));
}
// A gate of a phase chain: its form, in U[3].x, says which entries are read at all.
inline void chained(const cplx* U, cplx& a0, cplx& a1) {
  const int form = (int)U[3].real();
  if (form == kChainFull) {
    times(a1, U[2]);
    const double p0r = U[0].imag() * a1.real(), p0i = U[0].imag() * a1.imag();
    const double p1r = U[1].real() * a0.real(), p1i = U[1].real() * a0.imag();
    a0 = cplx(fma3(U[0].real(), a0.real(), p0r), fma3(U[0].real(), a0.imag(), p0i));
    a1 = cplx(fma3(U[1].imag(), a1.real(), p1r), fma3(U[1].imag(), a1.imag(), p1i));
    return;
  }
  const bool imag = (form - kChainUnit) & kChainImag, cross = (form - kChainUnit) & kChainCross;
  if (form < kChainUnit || form > kChainUnit + kChainImag + kChainCross) throw std::runtime_error("chain form");
  const double t = imag ? U[2].real() : U[2].imag();
  const double r0 = cross ? U[0].real() : U[0].imag(), r1 = cross ? U[1].imag() : U[1].real();
  const double x = imag ? fma3(t, a1.real(), -a1.imag()) : fma3(-t, a1.imag(), a1.real());
  const double y = imag ? fma3(t, a1.imag(), a1.real()) : fma3(t, a1.real(), a1.imag());
  a1 = cross ? cplx(fma3(r1, x, a0.real()), fma3(r1, y, a0.imag())) : cplx(fma3(r1, a0.real(), x), fma3(r1, a0.imag(), y));
  a0 = cross ? cplx(fma3(r0, a0.real(), x), fma3(r0, a0.imag(), y)) : cplx(fma3(r0, x, a0.real()), fma3(r0, y, a0.imag()));
}
// Real and X-like forms read one component of each entry.
inline void real_form(const cplx* U, cplx& a0, cplx& a1) {
  const cplx b0 = a0;
  a0 = cplx(fma3(U[0].real(), a0.real(), U[1].real() * a1.real()), fma3(U[0].real(), a0.imag(), U[1].real() * a1.imag()));
  a1 = cplx(fma3(U[3].real(), a1.real(), U[2].real() * b0.real()), fma3(U[3].real(), a1.imag(), U[2].real() * b0.imag()));
}
inline void x_form(const cplx* U, cplx& a0, cplx& a1) {
  const cplx b0 = a0;
  a0 = cplx(fma3(U[0].real(), a0.real(), -U[1].imag() * a1.imag()), fma3(U[0].real(), a0.imag(), U[1].imag() * a1.real()));
  a1 = cplx(fma3(U[3].real(), a1.real(), -U[2].imag() * b0.imag()), fma3(U[3].real(), a1.imag(), U[2].imag() * b0.real()));
}
inline double im_conj(cplx w, cplx g) { return w.real() * g.imag() - w.imag() * g.real(); }

// ---- plans ---------------------------------------------------------------------------------------
struct Machine {
  const Plan& p;
  std::vector<cplx> tab;
  std::vector<cplx> v, w;      // the state; reverse sweeps: and the costate
  std::vector<double> grad;    // reverse sweeps: per parameter
  double largest = 0.0;        // largest component of a stored state
  long flips = 0, phases = 0, chains = 0, blocks = 0, remaps = 0;  // ops met

  Machine(const Plan& plan, const qsv_circuit* c, const std::vector<double>& params, std::vector<cplx> psi,
          std::vector<cplx> lam = {})
      : p(plan), tab((size_t)plan.ctab_size + 1), v(std::move(psi)), w(std::move(lam)), grad(params.size(), 0.0) {
    bind_ctab(plan, c, params.data(), nullptr, 0, tab.data());
    for (const DevPass& dp : p.passes) run(dp);
  }

  static uint64_t runs(const uint64_t* d, int at, uint64_t tile) {
    uint64_t r = 0;
    for (int i = 0; i < (int)d[at]; ++i) {
      const uint64_t e = d[at + 1 + i];
      r |= ((tile >> ((e >> 16) & 255)) & ((1ull << ((e >> 8) & 255)) - 1)) << (e & 255);
    }
    return r;
  }
  const DiagEntry* entries(const DevPass& dp, int first, int count) const {
    if (first < dp.diag_lo || count < 0 || first + count > dp.diag_lo + dp.diag_n) throw std::runtime_error("entry range");
    return p.diag.data() + first;
  }

  void run(const DevPass& dp) {
    if (!dp.rb) throw std::runtime_error("not a register-blocked pass");
    const bool adj = p.adjoint, split = dp.alt && !adj, one = dp.alt && adj;
    const int RB = dp.rb, NR = 1 << RB, NT = 1 << (dp.m - RB);
    const int S = (p.dtype == QSV_C64 ? 4 : 3) + (split ? 1 : 0);
    const uint64_t* dep = p.deps.data() + dp.dep_first;
    std::vector<cplx> out(v.size()), outw(w.size());
    std::vector<char> written(v.size(), 0);
    std::vector<double> slots(dp.pslot_count, 0.0);
    for (uint64_t tile = 0; tile < (1ull << (p.n_qubits - dp.m)); ++tile) {
      const uint64_t base = runs(dep, kRunsLogical, tile);
      uint32_t reg = dp.lay0_reg;
      uint64_t thr = dp.lay0_thr, units = dp.lay0_units;
      auto lane_part = [&](int t, uint64_t th) {
        int j = 0;
        for (int b = 0; b < dp.m - RB; ++b) j |= ((t >> b) & 1) << ((th >> (4 * b)) & 15);
        return j;
      };
      auto spread = [&](int k) {
        int j = 0;
        for (int i = 0; i < RB; ++i) j |= ((k >> i) & 1) << ((reg >> (8 * i)) & 255);
        return j;
      };
      auto slot_offset = [&](uint64_t u, int k) {
        int o = 0;
        for (int i = 0; i < RB; ++i)
          if ((k >> i) & 1) o ^= (int)((u >> (16 * i)) & 0xffff);
        return o;
      };
      std::vector<std::vector<cplx>> a(NT, std::vector<cplx>(NR)), b(a);
      const uint64_t lb = dp.relayout ? runs(dep, kRunsLoad, tile) : base;
      for (int t = 0; t < NT; ++t)
        for (int k = 0; k < NR; ++k) {
          const int j = lane_part(t, thr) | spread(k);
          const uint64_t x = lb | dep[j & 127] | dep[128 + (j >> 7)];
          a[t][k] = v.at(x);
          if (adj) b[t][k] = w.at(x);
        }
      double acc = 0.0;
      for (int oi = 0; oi < dp.op_count; ++oi) {
        const TileOp& O = p.ops[dp.op_first + oi];
        const cplx* U = tab.data() + (O.mat > 0 ? O.mat : 0);
        const cplx* G = tab.data() + (O.gen > 0 ? O.gen : 0);
        // f(pair of slots k, k1 of thread t)
        auto pairs = [&](int slot, auto f) {
          for (int t = 0; t < NT; ++t)
            for (int k = 0; k < NR; ++k)
              if (!(k >> slot & 1)) f(t, k, k | 1 << slot);
        };
        auto sign_run = [&] {
          const DiagEntry* d = entries(dp, O.first, O.count);
          for (int e = 0; e < O.count; ++e) {
            if ((base & d[e].ocmask) != d[e].ocmask) continue;
            for (int t = 0; t < NT; ++t)
              if (((uint32_t)lane_part(t, thr) & d[e].tmask) == d[e].tmask)
                for (int k = 0; k < NR; ++k)
                  if (d[e].kmask >> k & 1) {
                    a[t][k] = -a[t][k];
                    if (adj) b[t][k] = -b[t][k];
                  }
          }
        };
        auto gate = [&](int slot, uint32_t lm, int form) {
          pairs(slot, [&](int t, int k, int k1) {
            if (((uint32_t)(lane_part(t, thr) | spread(k)) & lm) != lm) return;
            if (adj && O.gen >= 0) {
              const cplx g0 = G[0] * a[t][k] + G[1] * a[t][k1], g1 = G[2] * a[t][k] + G[3] * a[t][k1];
              acc += im_conj(b[t][k], g0) + im_conj(b[t][k1], g1);
            }
            for (int side = 0; side < (adj ? 2 : 1); ++side) {
              cplx& x = side ? b[t][k] : a[t][k];
              cplx& y = side ? b[t][k1] : a[t][k1];
              if (form == kPlainSplit) chained(U, x, y);
              else if (form == kPlainReal) real_form(U, x, y);
              else if (form == kPlainXlike) x_form(U, x, y);
              else general(U, x, y);
            }
          });
        };
        if (one ? O.plain && !(O.plain & kPlainPhases) : O.plain != 0) {
          const int slot = (O.plain & 7) - 1;
          if (!adj && (O.plain & kPlainBlock)) {
            if (O.plain & kPlainSigns) sign_run();
            block(O, slot, a, NR, NT);
          } else if (slot < 0) {
            sign_run();
          } else if (O.plain & kPlainFlip) {
            ++flips;
            if ((O.plain & kPlainOutside) && (base & O.omask) != O.omask) continue;
            const uint32_t ks = (uint32_t)O.plain >> 16;
            for (int t = 0; t < NT; ++t)
              if ((lane_part(t, thr) & O.first) == O.first)
                for (int k = 0; k < NR; ++k)
                  if (ks >> k & 1) {
                    if (k >> slot & 1) throw std::runtime_error("flip pair");
                    std::swap(a[t][k], a[t][k | 1 << slot]);
                    if (adj) std::swap(b[t][k], b[t][k | 1 << slot]);
                  }
          } else {
            if (O.plain & kPlainSigns) sign_run();
            chains += (O.plain & kPlainForm) == kPlainSplit;
            gate(slot, 0, O.plain & kPlainForm);
          }
        } else {
          int type = OP_DIAG, ob = 1;
          uint32_t lraw = 0;
          if (!one || !O.plain) {
            type = O.type;
            lraw = O.lmask;
            ob = O.b;
          }
          const bool on = !(lraw & kHasOutsideControls) || (base & O.omask) == O.omask;
          const uint32_t lm = lraw & ~kHasOutsideControls;
          if (on && ((type == OP_DIAG && !ob) || (type == OP_DENSE1 && ob))) sign_run();
          if (type == OP_REMAP || type == OP_XSWAP) {
            const uint64_t nu = (uint64_t)(uint32_t)O.gkind << 32 | (uint32_t)O.pslot;
            if (type == OP_XSWAP) {
              const int i = O.mat & 3, L = (O.mat & 255) >> 4;
              for (auto* r : {&a, &b}) {
                if (r == &b && !adj) continue;
                auto old = *r;
                pairs(i, [&](int t, int k, int k1) {
                  if (t >> L & 1) (*r)[t][k] = old[t ^ 1 << L][k1];
                  else (*r)[t][k1] = old[t ^ 1 << L][k];
                });
              }
            } else {
              ++remaps;
              for (auto* r : {&a, &b}) {
                if (r == &b && !adj) continue;
                std::vector<cplx> lds((size_t)1 << dp.m);
                std::vector<char> full(lds.size(), 0);
                for (int t = 0; t < NT; ++t)
                  for (int k = 0; k < NR; ++k) {
                    const size_t at = (size_t)(lds_swizzle(lane_part(t, thr), S) ^ slot_offset(units, k));
                    if (full.at(at)) throw std::runtime_error("two amplitudes at one LDS address");
                    full[at] = 1;
                    lds[at] = (*r)[t][k];
                  }
                for (int t = 0; t < NT; ++t)
                  for (int k = 0; k < NR; ++k)
                    (*r)[t][k] = lds.at((size_t)(lds_swizzle(lane_part(t, O.omask), S) ^ slot_offset(nu, k)));
              }
            }
            reg = (uint32_t)O.b;
            thr = O.omask;
            units = nu;
          } else if (on && type == OP_DENSE1) {
            gate(O.a, lm, 0);
          } else if (on && type == OP_DENSE2) {
            if (split) throw std::runtime_error("two-qubit matrix in a pass with halved remaps");
            for (auto* r : {&a, &b}) {
              if (r == &b && !adj) continue;
              std::vector<cplx> lds((size_t)1 << dp.m);
              auto at = [&](int t, int k) { return (size_t)(lds_swizzle(lane_part(t, thr), S) ^ slot_offset(units, k)); };
              for (int t = 0; t < NT; ++t)
                for (int k = 0; k < NR; ++k) lds.at(at(t, k)) = (*r)[t][k];
              for (int j = 0; j < (1 << dp.m); ++j) {
                if ((j >> O.a & 1) || (j >> O.b & 1) || ((uint32_t)j & lm) != lm) continue;
                const int idx[4] = {j, j | 1 << O.a, j | 1 << O.b, j | 1 << O.a | 1 << O.b};
                cplx x[4], y[4];
                for (int q = 0; q < 4; ++q) x[q] = lds[lds_swizzle(idx[q], S)];
                for (int q = 0; q < 4; ++q) y[q] = U[4 * q] * x[0] + U[4 * q + 1] * x[1] + U[4 * q + 2] * x[2] + U[4 * q + 3] * x[3];
                for (int q = 0; q < 4; ++q) lds[lds_swizzle(idx[q], S)] = y[q];
              }
              for (int t = 0; t < NT; ++t)
                for (int k = 0; k < NR; ++k) (*r)[t][k] = lds[at(t, k)];
            }
          } else if (on && type == OP_DIAG && ob) {
            phase_run(dp, O, one, base, NR, NT, a, b, acc, [&](int t) { return lane_part(t, thr); });
          } else if (on && type == OP_ZZ) {
            zz_run(O, lraw, base, RB, NR, NT, a, b, acc, [&](int t) { return lane_part(t, thr); });
          }
        }
        if (adj && O.flush) {
          slots.at(O.pslot) += acc;
          acc = 0.0;
        }
      }
      const uint64_t sb = dp.relayout ? runs(dep, kRunsStore, tile) : base;
      const uint64_t* sd = dep + (dp.relayout ? 256 : 0);
      for (int t = 0; t < NT; ++t)
        for (int k = 0; k < NR; ++k) {
          const int j = lane_part(t, thr) | spread(k);
          const uint64_t x = sb | sd[j & 127] | sd[128 + (j >> 7)];
          if (written.at(x)) throw std::runtime_error("two amplitudes stored at one index");
          written[x] = 1;
          out[x] = a[t][k];
          if (adj) outw[x] = b[t][k];
          largest = std::max(largest, std::max(std::abs(a[t][k].real()), std::abs(a[t][k].imag())));
        }
    }
    v.swap(out);
    w.swap(outw);
    for (int k = 0; k < dp.pslot_count; ++k) grad.at(p.pslot_param[dp.pslot_first + k]) += slots[k];
  }

  // 16x16x4 matrix-core products: lane l gives row l % 16 of the k-chunk's column l / 16 of A,
  // and column l % 16 of B's row l / 16; accumulator register r of lane l is row 4 (l / 16) + r
  // (complex64) or 4 r + l / 16 (complex128) of column l % 16.
  void block(const TileOp& O, int slot, std::vector<std::vector<cplx>>& a, int NR, int NT) {
    ++blocks;
    for (int w0 = 0; w0 < NT; w0 += 64)
      for (int k = 0; k < NR; ++k) {
        if (k >> slot & 1) continue;
        const int k1 = k | 1 << slot;
        double D[16][16] = {};
        for (int chunk = 0; chunk < 4; ++chunk) {
          double A[16][4], B[4][16];
          for (int l = 0; l < 64; ++l) {
            const int at = 4 * l + chunk;
            const cplx e = tab.at(O.mat + at / 2);
            A[l % 16][l / 16] = (at & 1) ? e.imag() : e.real();
            const cplx z = chunk < 2 ? a[w0 + l][k] : a[w0 + l][k1];
            B[l / 16][l % 16] = (chunk & 1) ? z.imag() : z.real();
          }
          for (int i = 0; i < 16; ++i)
            for (int j = 0; j < 16; ++j)
              for (int q = 0; q < 4; ++q) D[i][j] = fma3(A[i][q], B[q][j], D[i][j]);
        }
        for (int l = 0; l < 64; ++l) {
          auto acc = [&](int r) { return D[p.dtype == QSV_C64 ? 4 * (l / 16) + r : 4 * r + l / 16][l % 16]; };
          a[w0 + l][k] = cplx(acc(0), acc(1));
          a[w0 + l][k1] = cplx(acc(2), acc(3));
        }
      }
  }

  template <typename J>
  void phase_run(const DevPass& dp, const TileOp& O, bool one, uint64_t base, int NR, int NT,
                 std::vector<std::vector<cplx>>& a, std::vector<std::vector<cplx>>& b, double& acc, J jt) {
    const bool adj = p.adjoint;
    const DiagEntry* d = entries(dp, O.first, O.count);
    auto lane_bit = [&](int j, uint32_t src) {
      return src < 32 ? (j >> src & 1) != 0 : src < kNoBit && ((base >> (src - 32)) & 1);
    };
    auto apply = [&](int t, int k, cplx ph, double weight) {
      if (adj) {
        acc += weight * im_conj(b[t][k], a[t][k]);
        times(b[t][k], ph);
      }
      times(a[t][k], ph);
    };
    ++phases;
    if (one && O.count == 1 && (d[0].where & kWhereOne)) {
      const int at = (int)(d[0].where >> 24) - 1;
      for (int t = 0; t < NT; ++t)
        for (int k = 0; k < NR; ++k) {
          const bool bit = at < 0 ? lane_bit(jt(t), d[0].where & 255u) : (k >> at & 1) != 0;
          apply(t, k, tab.at(O.mat + bit), O.gen >= 0 ? tab.at(O.gen + bit).real() : 0.0);
        }
      return;
    }
    for (int e = 0; e < O.count; ++e) {
      const DiagEntry& f = d[e];
      if ((base & f.ocmask) != f.ocmask) continue;
      for (int t = 0; t < NT; ++t) {
        const int j = jt(t);
        if (((uint32_t)j & f.tmask) != f.tmask) continue;
        if (f.where & kWhereSign) {
          for (int k = 0; k < NR; ++k)
            if (f.kmask >> k & 1) {
              a[t][k] = -a[t][k];
              if (adj) b[t][k] = -b[t][k];
            }
          continue;
        }
        const bool t0 = lane_bit(j, f.where & 255u), t1 = lane_bit(j, (f.where >> 8) & 255u);
        for (uint32_t u = 0; u < 4; ++u) {
          if (((u & 1) && !f.bits0) || ((u & 2) && !f.bits1)) continue;
          const uint32_t ks = f.kmask & ((u & 1) ? f.bits0 : ~f.bits0) & ((u & 2) ? f.bits1 : ~f.bits1);
          const int idx = (t0 || (u & 1) ? 1 : 0) | ((f.where & kWhereTwo) && (t1 || (u & 2)) ? 2 : 0);
          for (int k = 0; k < NR; ++k)
            if (ks >> k & 1) apply(t, k, tab.at(f.tab + idx), f.gtab >= 0 ? tab.at(f.gtab + idx).real() : 0.0);
        }
      }
    }
  }

  template <typename J>
  void zz_run(const TileOp& O, uint32_t lraw, uint64_t base, int RB, int NR, int NT, std::vector<std::vector<cplx>>& a,
              std::vector<std::vector<cplx>>& b, double& acc, J jt) {
    std::vector<uint32_t> cls;
    for (uint32_t c = 0; c < (1u << RB); ++c)
      if (__builtin_popcount(c) <= 2) cls.push_back(c);
    const uint32_t cw[3] = {(uint32_t)O.a, (uint32_t)O.b, lraw};
    for (int t = 0; t < NT; ++t)
      for (int k = 0; k < NR; ++k) {
        int cnt = 0, e = O.first;
        for (size_t c = 0; c < cls.size(); ++c)
          for (uint32_t i = 0; i < ((cw[c >> 2] >> (8 * (c & 3))) & 255u); ++i, ++e)
            cnt += (__builtin_popcount((uint32_t)jt(t) & p.edges.at(e).tmask) +
                    __builtin_popcountll(base & p.edges.at(e).omask) + __builtin_popcount((uint32_t)k & cls[c])) & 1;
        if (e != O.first + O.count) throw std::runtime_error("edge classes");
        const cplx ph = tab.at(O.mat + cnt);
        if (p.adjoint) {
          if (O.gen >= 0) acc += tab.at(O.gen + cnt).real() * im_conj(b[t][k], a[t][k]);
          times(b[t][k], ph);
        }
        times(a[t][k], ph);
      }
  }
};

// ---- the same gate by gate -----------------------------------------------------------------------
// A gate's matrix on its targets (index bit b is targets[b]) from its definition.
inline std::vector<lcplx> definition(const qsv_circuit* c, const qsv_gate& g, const long double* a) {
  const lcplx i(0, 1);
  auto pol = [](long double t) { return lcplx(std::cos(t), std::sin(t)); };
  const long double h = a[0] / 2, cs = std::cos(h), sn = std::sin(h), r = std::sqrt(0.5L), pi = std::acos(-1.0L);
  auto rz = [&](long double t) { return std::vector<lcplx>{pol(-t / 2), 0, 0, pol(t / 2)}; };
  switch (g.kind) {
    case QSV_GATE_X: return {0, 1, 1, 0};
    case QSV_GATE_Y: return {0, -i, i, 0};
    case QSV_GATE_Z: return {1, 0, 0, -1};
    case QSV_GATE_H: return {r, r, r, -r};
    case QSV_GATE_S: return {1, 0, 0, i};
    case QSV_GATE_SDG: return {1, 0, 0, -i};
    case QSV_GATE_T: return {1, 0, 0, pol(pi / 4)};
    case QSV_GATE_TDG: return {1, 0, 0, pol(-pi / 4)};
    case QSV_GATE_RX: return {cs, -i * sn, -i * sn, cs};
    case QSV_GATE_RY: return {cs, -sn, sn, cs};
    case QSV_GATE_RZ: return rz(a[0]);
    case QSV_GATE_PS: return {1, 0, 0, pol(a[0])};
    case QSV_GATE_RXX: return {cs, 0, 0, -i * sn, 0, cs, -i * sn, 0, 0, -i * sn, cs, 0, -i * sn, 0, 0, cs};
    case QSV_GATE_RYY: return {cs, 0, 0, i * sn, 0, cs, -i * sn, 0, 0, -i * sn, cs, 0, i * sn, 0, 0, cs};
    case QSV_GATE_RZZ: return {pol(-h), 0, 0, 0, 0, pol(h), 0, 0, 0, 0, pol(h), 0, 0, 0, 0, pol(-h)};
    case QSV_GATE_U3: {
      const auto x = rz(a[1]), z = rz(a[2]);
      return {x[0] * cs * z[0], x[0] * -sn * z[3], x[3] * sn * z[0], x[3] * cs * z[3]};
    }
    case QSV_GATE_SWAP: return {1, 0, 0, 0, 0, 0, 1, 0, 0, 1, 0, 0, 0, 0, 0, 1};
    default: {
      const int d = g.kind == QSV_GATE_MAT1 ? 4 : 16;
      std::vector<lcplx> m;
      for (int k = 0; k < d; ++k)
        m.push_back(lcplx(c->matrices[2 * (g.matrix_offset + k)], c->matrices[2 * (g.matrix_offset + k) + 1]));
      return m;
    }
  }
}
inline void angles_of(const qsv_gate& g, const std::vector<double>& params, long double* a) {
  for (int s = 0; s < 3; ++s)
    a[s] = g.angle_const[s] + (g.param_index[s] >= 0 ? (long double)g.param_coeff[s] * params[g.param_index[s]] : 0.0L);
}
// only: amplitudes whose controls are not all 1 become 0 (for derivatives)
inline void apply_definition(std::vector<lcplx>& x, const qsv_gate& g, const std::vector<lcplx>& m, bool only = false) {
  const bool two = m.size() == 16;
  const uint64_t t0 = 1ull << g.targets[0], t1 = two ? 1ull << g.targets[1] : 0;
  for (uint64_t k = 0; k < x.size(); ++k) {
    if (k & (t0 | t1)) continue;
    const uint64_t idx[4] = {k, k | t0, k | t1, k | t0 | t1};
    const int d = two ? 4 : 2;
    lcplx o[4] = {};
    if ((k & g.ctrl_mask) == g.ctrl_mask) {
      for (int r = 0; r < d; ++r)
        for (int q = 0; q < d; ++q) o[r] += m[r * d + q] * x[idx[q]];
    } else {
      for (int r = 0; r < d && !only; ++r) o[r] = x[idx[r]];
    }
    for (int r = 0; r < d; ++r) x[idx[r]] = o[r];
  }
}

}  // namespace replay
