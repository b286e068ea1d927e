// Register-blocked tile passes: kernels and launchers, instantiated one amplitude type and
// direction at a time by tile_rb.hip.
#pragma once
#include <algorithm>
#include <type_traits>

#include "device_util.h"
#include "qsv_kernels.h"

namespace qsv {

// ------------------------------------------------------------------------------------------
// Register-blocked tile pass.  Each of the 2^(m-RB) threads keeps 2^RB amplitudes of the
// tile in registers.  The local bits in the current register mask are "register bits":
// a gate on them is pure VALU work inside one thread.  A REMAP op changes which local bits
// are register bits by one write and one read of the tile through LDS (XOR-swizzled so
// every access pattern spreads over the banks).  Gates on other bits are never issued:
// the planner groups each pass's gates into register rounds.
// ------------------------------------------------------------------------------------------
template <int S>  // S = log2(elements per 128-byte LDS row)
__device__ __forceinline__ int swz(int j) { return lds_swizzle(j, S); }

// dst <- src in the lanes set in the wave-uniform lane mask, written in place (a select
// whose result the compiler could put in a new register would make it carry the register
// block in two register sets).
__device__ __forceinline__ void sel_in32(uint32_t& d, uint32_t src, uint64_t lanes) {
  asm("v_cndmask_b32_e64 %0, %0, %1, %2" : "+v"(d) : "v"(src), "s"(lanes));
}
__device__ __forceinline__ void sel_in(float2& d, float2 s, uint64_t lanes) {
  uint32_t x = __float_as_uint(d.x), y = __float_as_uint(d.y);
  sel_in32(x, __float_as_uint(s.x), lanes);
  sel_in32(y, __float_as_uint(s.y), lanes);
  d.x = __uint_as_float(x);
  d.y = __uint_as_float(y);
}
__device__ __forceinline__ void sel_in(double2& d, double2 s, uint64_t lanes) {
  const uint64_t a = (uint64_t)__double_as_longlong(d.x), b = (uint64_t)__double_as_longlong(d.y);
  const uint64_t e = (uint64_t)__double_as_longlong(s.x), f = (uint64_t)__double_as_longlong(s.y);
  uint32_t w[4] = {(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)};
  sel_in32(w[0], (uint32_t)e, lanes);
  sel_in32(w[1], (uint32_t)(e >> 32), lanes);
  sel_in32(w[2], (uint32_t)f, lanes);
  sel_in32(w[3], (uint32_t)(f >> 32), lanes);
  d.x = __longlong_as_double((long long)((uint64_t)w[1] << 32 | w[0]));
  d.y = __longlong_as_double((long long)((uint64_t)w[3] << 32 | w[2]));
}

template <typename C> __device__ __forceinline__ C csel(bool c, C a, C b) {
  C r;
  r.x = c ? a.x : b.x;
  r.y = c ? a.y : b.y;
  return r;
}

// Cross-lane transposition of a register slot bit and lane bit L (4 or 5) of the wave.  X
// and Y are the two slots that differ in the slot bit.  Afterwards X holds the amplitudes
// whose old lane bit L was 0 and Y those whose old lane bit L was 1, each at the lane whose
// bit L equals their old slot bit:
//   X' = c ? Y(lane ^ 2^L) : X,   Y' = c ? Y : X(lane ^ 2^L)   (c = the lane's bit L),
// which is what gfx950's row swap (bit 4: odd 16-lane rows of the first operand with even
// rows of the second) and half-wave swap (bit 5) do, in place, one 32-bit word each.
template <int L>
__device__ __forceinline__ void xlane32(uint32_t& x, uint32_t& y) {
  static_assert(L == 4 || L == 5, "cross-lane transpositions use lane bits 4 and 5");
  if constexpr (L == 5) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    x = r[0];
    y = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = r[0];
    y = r[1];
  }
}
template <int L>
__device__ __forceinline__ void xlane(float2& X, float2& Y) {
  uint32_t x0 = __float_as_uint(X.x), x1 = __float_as_uint(X.y), y0 = __float_as_uint(Y.x), y1 = __float_as_uint(Y.y);
  xlane32<L>(x0, y0);
  xlane32<L>(x1, y1);
  X.x = __uint_as_float(x0); X.y = __uint_as_float(x1);
  Y.x = __uint_as_float(y0); Y.y = __uint_as_float(y1);
}
template <int L>
__device__ __forceinline__ void xlane(double2& X, double2& Y) {
  const uint64_t a = (uint64_t)__double_as_longlong(X.x), b = (uint64_t)__double_as_longlong(X.y);
  const uint64_t e = (uint64_t)__double_as_longlong(Y.x), f = (uint64_t)__double_as_longlong(Y.y);
  uint32_t x[4] = {(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)};
  uint32_t y[4] = {(uint32_t)e, (uint32_t)(e >> 32), (uint32_t)f, (uint32_t)(f >> 32)};
#pragma unroll
  for (int d = 0; d < 4; ++d) xlane32<L>(x[d], y[d]);
  X.x = __longlong_as_double((long long)((uint64_t)x[1] << 32 | x[0]));
  X.y = __longlong_as_double((long long)((uint64_t)x[3] << 32 | x[2]));
  Y.x = __longlong_as_double((long long)((uint64_t)y[1] << 32 | y[0]));
  Y.y = __longlong_as_double((long long)((uint64_t)y[3] << 32 | y[2]));
}
template <int I, int L, int NR, typename C>
__device__ __forceinline__ void xswap1(C* v) {
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    if (k & (1 << I)) continue;
    xlane<L>(v[k], v[k | (1 << I)]);
  }
}
// code = slot bit | lane bit << 4 (lane bit 4 or 5)
template <int RB, typename C>
__device__ __forceinline__ void xswap_dispatch(int code, C* v) {
  constexpr int NR = 1 << RB;
  switch (code) {
    case 0 | 4 << 4: xswap1<0, 4, NR>(v); break;
    case 0 | 5 << 4: xswap1<0, 5, NR>(v); break;
    case 1 | 4 << 4: xswap1<1, 4, NR>(v); break;
    case 1 | 5 << 4: xswap1<1, 5, NR>(v); break;
    case 2 | 4 << 4: xswap1<2, 4, NR>(v); break;
    case 2 | 5 << 4: xswap1<2, 5, NR>(v); break;
    default:
      if constexpr (RB > 3) {
        if (code == (3 | 4 << 4)) xswap1<(RB > 3 ? 3 : 0), 4, NR>(v);
        else if (code == (3 | 5 << 4)) xswap1<(RB > 3 ? 3 : 0), 5, NR>(v);
      }
      break;
  }
}

// x and y trade places in the lanes of the wave-uniform lane mask, in place: one instruction
// per 32-bit word under a narrowed exec mask.
__device__ __forceinline__ void swap_lanes(float2& x, float2& y, uint64_t lanes) {
  uint32_t x0 = __float_as_uint(x.x), x1 = __float_as_uint(x.y), y0 = __float_as_uint(y.x), y1 = __float_as_uint(y.y);
  uint64_t all;
  asm("s_and_saveexec_b64 %4, %5\n\tv_swap_b32 %0, %2\n\tv_swap_b32 %1, %3\n\ts_mov_b64 exec, %4"
      : "+v"(x0), "+v"(x1), "+v"(y0), "+v"(y1), "=&s"(all) : "s"(lanes) : "scc");
  x.x = __uint_as_float(x0); x.y = __uint_as_float(x1);
  y.x = __uint_as_float(y0); y.y = __uint_as_float(y1);
}
__device__ __forceinline__ void swap_lanes(double2& x, double2& y, uint64_t lanes) {
  const uint64_t a = (uint64_t)__double_as_longlong(x.x), b = (uint64_t)__double_as_longlong(x.y);
  const uint64_t e = (uint64_t)__double_as_longlong(y.x), f = (uint64_t)__double_as_longlong(y.y);
  uint32_t u[4] = {(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)};
  uint32_t w[4] = {(uint32_t)e, (uint32_t)(e >> 32), (uint32_t)f, (uint32_t)(f >> 32)};
  uint64_t all;
  asm("s_and_saveexec_b64 %8, %9\n\tv_swap_b32 %0, %4\n\tv_swap_b32 %1, %5\n\tv_swap_b32 %2, %6\n\t"
      "v_swap_b32 %3, %7\n\ts_mov_b64 exec, %8"
      : "+v"(u[0]), "+v"(u[1]), "+v"(u[2]), "+v"(u[3]), "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "=&s"(all)
      : "s"(lanes) : "scc");
  x.x = __longlong_as_double((long long)((uint64_t)u[1] << 32 | u[0]));
  x.y = __longlong_as_double((long long)((uint64_t)u[3] << 32 | u[2]));
  y.x = __longlong_as_double((long long)((uint64_t)w[1] << 32 | w[0]));
  y.y = __longlong_as_double((long long)((uint64_t)w[3] << 32 | w[2]));
}
// X on slot bit I of the slot pairs in `pairs`, in the lanes of `lanes`.
template <int I, int NR, typename C>
__device__ __forceinline__ void flip1(C* v, uint32_t pairs, uint64_t lanes) {
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    if (k & (1 << I)) continue;
    if ((pairs >> k) & 1u) swap_lanes(v[k], v[k | (1 << I)], lanes);
  }
}
template <int RB, typename C>
__device__ __forceinline__ void flip_dispatch(int slot, C* v, uint32_t pairs, uint64_t lanes) {
  constexpr int NR = 1 << RB;
  switch (slot) {
    case 0: flip1<0, NR>(v, pairs, lanes); break;
    case 1: flip1<1, NR>(v, pairs, lanes); break;
    case 2: flip1<2, NR>(v, pairs, lanes); break;
    default:
      if constexpr (RB > 3) flip1<(RB > 3 ? 3 : 0), NR>(v, pairs, lanes);
      break;
  }
}

// The local bits of register slot k in a layout whose slot bit i is local bit
// (reg >> 8i) & 255 (wave-uniform).
template <int NR>
__device__ __forceinline__ int spread_of(uint32_t reg, int k) {
  int j = 0;
#pragma unroll
  for (int i = 0; (1 << i) < NR; ++i)
    if ((k >> i) & 1) j |= 1 << (int)((reg >> (8 * i)) & 255);
  return j;
}

// 2x2 gate on register bit I.  Gates without local controls (the common case, a
// wave-uniform test) run straight-line; controlled ones compute every pair and keep the
// old values by select where a control bit is 0, so no lane-divergent branch is formed.
// Re(conj(w) * g) in fp64
template <typename C> __device__ __forceinline__ double re_conj_mul(C w, C g) {
  return (double)w.x * (double)g.x + (double)w.y * (double)g.y;
}
// The adjoint gradient term of a slot pair, Im<w|G|v> over (k, k1): a general 2x2 G, or
// k X / k Y without the multiplications by their zeros (k applied by the caller).
template <int GK, typename C>
__device__ __forceinline__ double grad_term(C w0, C w1, C v0, C v1, const C* G) {
  if constexpr (GK == GEN_X) return im_conj_mul(w0, v1) + im_conj_mul(w1, v0);
  else if constexpr (GK == GEN_Y) return re_conj_mul(w1, v0) - re_conj_mul(w0, v1);
  else return im_conj_mul(w0, cdot2(G[0], v0, G[1], v1)) + im_conj_mul(w1, cdot2(G[2], v0, G[3], v1));
}

template <int I, int NR, bool ADJ, int GK, typename C, int F = FORM_GENERAL>
__device__ __forceinline__ void reg1(C* v, C* w, int jt, uint32_t reg, uint32_t lm, const C* U, bool grad,
                                     const C* G, double& acc) {
  if constexpr (F == FORM_SPLIT) {  // forward, uncontrolled
    const auto each = [&](auto f) {
#pragma unroll
      for (int k = 0; k < NR; ++k)
        if (!(k & (1 << I))) f(v[k], v[k | (1 << I)]);
    };
    const uint32_t form = high_word(U[3].x);  // wave-uniform
    using R = decltype(U[0].x);
    if (form == high_word((R)kChainUnit))
      each([&](C& a, C& b) { apply2unit<false, false>(U[0].y, U[1].x, U[2].y, a, b); });
    else if (form == high_word((R)(kChainUnit + kChainImag)))
      each([&](C& a, C& b) { apply2unit<true, false>(U[0].y, U[1].x, U[2].x, a, b); });
    else if (form == high_word((R)(kChainUnit + kChainCross)))
      each([&](C& a, C& b) { apply2unit<false, true>(U[0].x, U[1].y, U[2].y, a, b); });
    else if (form == high_word((R)(kChainUnit + kChainImag + kChainCross)))
      each([&](C& a, C& b) { apply2unit<true, true>(U[0].x, U[1].y, U[2].x, a, b); });
    else
      each([&](C& a, C& b) { apply2split(U[0], U[1], U[2], a, b); });
    return;
  }
  if (lm == 0) {
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      if (k & (1 << I)) continue;
      const int k1 = k | (1 << I);
      if (ADJ) {
        double g = 0.0;
        if (grad) g = grad_term<GK>(w[k], w[k1], v[k], v[k1], G);
        apply2f<F>(U, w[k], w[k1], g);
        apply2f<F>(U, v[k], v[k1], g);
        acc += g;
      } else {
        apply2f<F>(U, v[k], v[k1]);
      }
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    if (k & (1 << I)) continue;
    const int k1 = k | (1 << I);
    const bool ok = ((uint32_t)(jt | spread_of<NR>(reg, k)) & lm) == lm;
    C n0 = v[k], n1 = v[k1];
    if (ADJ) {
      C m0 = w[k], m1 = w[k1];
      double g = 0.0;
      if (grad) g = grad_term<GK>(m0, m1, n0, n1, G);
      apply2(U[0], U[1], U[2], U[3], m0, m1, g);
      acc += ok ? g : 0.0;
      const uint64_t okm = __builtin_amdgcn_ballot_w64(ok);
      sel_in(w[k], m0, okm);
      sel_in(w[k1], m1, okm);
    }
    apply2(U[0], U[1], U[2], U[3], n0, n1);
    const uint64_t okv = __builtin_amdgcn_ballot_w64(ok);
    sel_in(v[k], n0, okv);
    sel_in(v[k1], n1, okv);
  }
}

template <typename C>
__device__ __forceinline__ void mat4(const C* M, const C* x, C* y) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    C o = cdot2(M[4 * r], x[0], M[4 * r + 1], x[1]);
    y[r] = cdot2(C{1, 0}, o, M[4 * r + 2], x[2]);
    y[r] = cdot2(C{1, 0}, y[r], M[4 * r + 3], x[3]);
  }
}

template <int RB, bool ADJ, int GK, typename C, int F = FORM_GENERAL>
__device__ __forceinline__ void reg1_slot(int i, C* v, C* w, int jt, uint32_t reg, uint32_t lm, const C* U,
                                          bool grad, const C* G, double& acc) {
  constexpr int NR = 1 << RB;
  switch (i) {
    case 0: reg1<0, NR, ADJ, GK, C, F>(v, w, jt, reg, lm, U, grad, G, acc); break;
    case 1: reg1<1, NR, ADJ, GK, C, F>(v, w, jt, reg, lm, U, grad, G, acc); break;
    case 2: reg1<2, NR, ADJ, GK, C, F>(v, w, jt, reg, lm, U, grad, G, acc); break;
    default:
      if constexpr (RB > 3) reg1<(RB > 3 ? 3 : 0), NR, ADJ, GK, C, F>(v, w, jt, reg, lm, U, grad, G, acc);
      break;
  }
}
// Forward passes and gradient-free adjoint gates use the general form (its gradient
// code is not reached); gradient-bearing adjoint gates with an X or Y generator get the
// shorter gradient term, scaled by k once per op.
template <int RB, bool ADJ, typename C>
__device__ __forceinline__ void reg1_dispatch(int i, C* v, C* w, int jt, uint32_t reg, uint32_t lm, const C* U,
                                              bool grad, int gkind, const C* G, double& acc) {
  if (ADJ && grad && gkind != GEN_GENERAL) {
    const double kf = gkind == GEN_X ? (double)G[1].x : (double)G[2].y;
    double part = 0.0;
    if (gkind == GEN_X) reg1_slot<RB, ADJ, GEN_X>(i, v, w, jt, reg, lm, U, true, G, part);
    else reg1_slot<RB, ADJ, GEN_Y>(i, v, w, jt, reg, lm, U, true, G, part);
    acc = __builtin_fma(kf, part, acc);
    return;
  }
  reg1_slot<RB, ADJ, GEN_GENERAL>(i, v, w, jt, reg, lm, U, grad, G, acc);
}

// Fused 8x8 block on (lane bit 4, lane bit 5, slot bit I) with the matrix cores.  A lane
// holds, for each pair of slots (k0, k1 = k0 | 2^I), the block components
// (re k0, im k0, re k1, im k1): real rows q + 4i of the 16-row real vector, q = its lane
// bits 4-5, i = 0..3; its lane bits 0-3 select one of 16 columns.  Four 16x16x4 products
// (k-chunk i = component i) give the 16x16 result, whose accumulator layout the planner's
// row order already matches, so every component returns to the register it came from.
typedef float qsv_f4 __attribute__((ext_vector_type(4)));
typedef double qsv_d4 __attribute__((ext_vector_type(4)));
template <int I, int NR>
__device__ __forceinline__ void block16(float2* v, const float* a) {
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    if (k & (1 << I)) continue;
    const int k1 = k | (1 << I);
    qsv_f4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], v[k].x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], v[k].y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], v[k1].x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], v[k1].y, acc, 0, 0, 0);
    v[k].x = acc[0];
    v[k].y = acc[1];
    v[k1].x = acc[2];
    v[k1].y = acc[3];
  }
}
template <int I, int NR>
__device__ __forceinline__ void block16(double2* v, const double* a) {
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    if (k & (1 << I)) continue;
    const int k1 = k | (1 << I);
    qsv_d4 acc = {0.0, 0.0, 0.0, 0.0};
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], v[k].x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1], v[k].y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[2], v[k1].x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[3], v[k1].y, acc, 0, 0, 0);
    v[k].x = acc[0];
    v[k].y = acc[1];
    v[k1].x = acc[2];
    v[k1].y = acc[3];
  }
}
template <int RB, typename C, typename R>
__device__ __forceinline__ void block_dispatch(int slot, C* v, const R* a) {
  constexpr int NR = 1 << RB;
  switch (slot) {
    case 0: block16<0, NR>(v, a); break;
    case 1: block16<1, NR>(v, a); break;
    case 2: block16<2, NR>(v, a); break;
    default:
      if constexpr (RB > 3) block16<(RB > 3 ? 3 : 0), NR>(v, a);
      break;
  }
}

// One-qubit phases of the reverse sweep: slots whose slot bit I is 0 times p0, the others times
// p1 (wave-uniform), with the gradient weights g0 and g1; I = -1: every slot times p0 (per lane).
template <int I, int NR, typename C>
__device__ __forceinline__ void phase1(C* v, C* w, C p0, C p1, double g0, double g1, double& acc) {
  double s0 = 0.0, s1 = 0.0;
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    const bool one = I >= 0 && (k >> (I >= 0 ? I : 0)) & 1;
    // Slot by slot: otherwise the products that the dispatch's cases share are formed for every
    // slot before it (50 more registers, three waves per SIMD instead of four).
    asm volatile("" : "+v"(v[k].x), "+v"(v[k].y), "+v"(w[k].x), "+v"(w[k].y));
    double g = im_conj_mul(w[k], v[k]);
    if constexpr (I < 0) {
      cmul_in(w[k], p0, g);
      cmul_in(v[k], p0, g);
    } else {
      cmul_in_s(w[k], one ? p1 : p0, g);
      cmul_in_s(v[k], one ? p1 : p0, g);
    }
    (one ? s1 : s0) += g;
  }
  acc = I < 0 ? __builtin_fma(g0, s0, acc) : __builtin_fma(g0, s0, __builtin_fma(g1, s1, acc));
}
template <int RB, typename C>
__device__ __forceinline__ void phase1_dispatch(int slot, C* v, C* w, C p0, C p1, double g0, double g1, double& acc) {
  constexpr int NR = 1 << RB;
  switch (slot) {
    case 0: phase1<0, NR>(v, w, p0, p1, g0, g1, acc); break;
    case 1: phase1<1, NR>(v, w, p0, p1, g0, g1, acc); break;
    case 2: phase1<2, NR>(v, w, p0, p1, g0, g1, acc); break;
    default:
      if constexpr (RB > 3) phase1<(RB > 3 ? 3 : 0), NR>(v, w, p0, p1, g0, g1, acc);
      break;
  }
}

__device__ __forceinline__ int insert_zero(int t, int p) { return ((t >> p) << (p + 1)) | (t & ((1 << p) - 1)); }

// Dynamic LDS of the register-blocked passes, sized per launch: the ctab window, then
// (adjoint) the deferred gradient sums.
extern __shared__ __align__(16) unsigned char qsv_dyn_lds[];
template <typename R> __host__ __device__ constexpr size_t win_bytes(int win_n) {
  return ((size_t)(win_n > 0 ? win_n : 0) * 2 * sizeof(R) + 15) & ~(size_t)15;
}
// Enough for every workgroup of a launch whose items have at most win_n window entries and
// pslots gradient slots: an item defers its sums only when pslots x waves fits the cap.
template <typename R> static size_t rb_dyn_lds(int maxm, bool adj, int win_n, int pslots) {
  const int nw = (1 << (maxm - 3)) >= 64 ? (1 << (maxm - 3)) / 64 : 1;
  const int sums = adj ? std::min(pslots * nw, kMaxDeferredSums) : 0;
  return win_bytes<R>(win_n) + (size_t)(sums > 0 ? sums : 0) * sizeof(double);
}

// ZZ edge classes of a register block of RB bits: the register-bit masks with at most two
// bits set, in increasing order (the planner packs class sizes in this order).
template <int RB> __host__ __device__ constexpr int zz_classes() { return RB == 3 ? 7 : 11; }
template <int RB> __host__ __device__ constexpr int zz_class(int i) {
  return RB == 3 ? i : (i < 7 ? i : (i == 7 ? 8 : (i == 8 ? 9 : (i == 9 ? 10 : 12))));
}

// Sign-only diagonal entries in a register-blocked pass: bit k of the result is the
// parity of the entries satisfied by register slot k, from the per-entry thread mask and
// slot set (jt = the thread's local index with its register bits zero).
// The three fields are contiguous (16 bytes), so each entry is one scalar load, and four
// entries are requested before the first is used.
struct SignFields {
  uint64_t ocmask;
  uint32_t tmask, kmask;
};
static_assert(offsetof(DiagEntry, tmask) == offsetof(DiagEntry, ocmask) + 8 &&
                  offsetof(DiagEntry, kmask) == offsetof(DiagEntry, ocmask) + 12,
              "sign fields must be contiguous");
__device__ __forceinline__ SignFields sign_fields(const DiagEntry* d) {
  return ld_record(reinterpret_cast<const SignFields*>(&d->ocmask));
}
struct PhaseFields {
  uint64_t ocmask;
  uint32_t tmask, kmask;
  int32_t tab, gtab;
  uint32_t where, bits0, bits1, pad;
};
static_assert(offsetof(DiagEntry, pad) == offsetof(DiagEntry, ocmask) + offsetof(PhaseFields, pad),
              "an entry's register-pass fields are contiguous");
// Also returns in `touched` (wave-uniform) the slots any entry of the run can flip.
__device__ __forceinline__ uint32_t sign_slots(const DiagEntry* d, int count, uint64_t base, uint32_t jt,
                                               uint32_t& touched) {
  uint32_t sm = 0, any = 0;
  int e = 0;
  for (; e + 4 <= count; e += 4) {
    SignFields f[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = sign_fields(d + e + i);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // entries with an outside control that is 0 in this tile do nothing
      const uint32_t km = f[i].kmask & (0u - (uint32_t)((base & f[i].ocmask) == f[i].ocmask));
      any |= km;
      sm ^= (jt & f[i].tmask) == f[i].tmask ? km : 0u;
    }
  }
  for (; e < count; ++e) {
    const SignFields f = sign_fields(d + e);
    const uint32_t km = f.kmask & (0u - (uint32_t)((base & f.ocmask) == f.ocmask));
    any |= km;
    sm ^= (jt & f.tmask) == f.tmask ? km : 0u;
  }
  touched = any;
  return sm;
}

// FULL: the tile fills the workgroup (m == MAXM), so every thread holds amplitudes.
// SPLIT (forward passes without two-qubit matrices, in launches of many tiles): remaps move the
// real and the imaginary parts one after the other through half the LDS.  A pass waits more
// than it computes (scalar loads, branches, remaps: with four waves per SIMD the vector ALU
// was busy 56 % of the time), so it wants resident waves: half the exchange buffer and 72
// registers allow seven per SIMD in complex128 where LDS allowed four (complex64, 16 amplitudes
// a thread: six).  30-qubit brick in complex128, whole step: 200 -> 143 ms (five waves 164, six
// 149; eight spill); 27 qubits in complex64: 14.7 -> 13.7 ms.  In launches that leave the chip
// idle the two further barriers only cost (10-qubit ansatz 231 -> 257 us); the reverse sweep's
// registers spill at five waves (24-qubit QAOA gradients 46 -> 54 ms).
template <typename R> constexpr int kSplitWaves = sizeof(R) == 4 ? 6 : 7;

// ONE (reverse sweeps with runs of a single uncontrolled one-qubit phase, as ansatz circuits have
// them): those runs' straight lines, which QAOA sweeps would pay for in registers (92 instead of
// 79 in complex64, five waves per SIMD instead of six: 2.4 %).
// ALT: SPLIT in forward passes, ONE in reverse sweeps.
template <typename R, int RB, int MAXM, bool ADJ, bool FULL, bool ALT, bool WARM>
__device__ __forceinline__ void rb_body(const PassArgs& A, const uint64_t tile, const int b) {
  using C = typename CT<R>::T;
  static_assert(RB == 3 || RB == 4, "register blocks of three or four bits");
  constexpr bool SPLIT = ALT && !ADJ, ONE = ALT && ADJ;
  constexpr int NT = 1 << (MAXM - RB);
  constexpr int NR = 1 << RB;
  using X = std::conditional_t<SPLIT, R, C>;    // what one exchange moves per amplitude
  constexpr int S = sizeof(X) == 16 ? 3 : sizeof(X) == 8 ? 4 : 5;
  __shared__ X buf[1 << MAXM];
  __shared__ double red[NT >= 64 ? NT / 64 : 1];

  const int tid = threadIdx.x;
  const int m = FULL ? MAXM : A.m;  // single-state launches require a full tile
  const int nloc = 1 << m;
  const bool active = FULL || tid < (nloc >> RB);
  // The tile's base indices from the planner's runs of tile-index bits: logical (bit q is
  // qubit q: controls and phases read it) and the indices the pass reads and writes (they
  // differ from the logical one when passes relayout the state).
  auto run_base = [&](int at) {
    uint64_t r = 0;
    const int nruns = (int)ld(A.dep + at);
    for (int i = 0; i < nruns; ++i) {
      const uint64_t e = ld(A.dep + at + 1 + i);
      const int lo = (int)(e & 255), len = (int)((e >> 8) & 255), sh = (int)((e >> 16) & 255);
      r |= ((tile >> sh) & ((1ull << len) - 1)) << lo;
    }
    return r;
  };
  const uint64_t base = run_base(kRunsLogical);

  C* psi = reinterpret_cast<C*>(A.psi) + (int64_t)b * A.bstride;
  C* out = A.dst ? reinterpret_cast<C*>(A.dst) + (int64_t)b * A.bstride : psi;
  C* lam = ADJ ? reinterpret_cast<C*>(A.lam) + (int64_t)b * A.bstride : nullptr;
  const C* src = A.src ? reinterpret_cast<const C*>(A.src) + (int64_t)b * A.src_bstride : psi;
  const C* T = reinterpret_cast<const C*>(A.ctab) + (int64_t)b * A.ctab_bstride;

  // Local index of register slot k in a layout: thread bit t of the thread id sits at local
  // bit (thr >> 4t) & 15, slot bit i of k at local bit (reg >> 8i) & 255.  A thread keeps
  // only its own part jt (slot 0); the slot parts are wave-uniform.
  const int nthr = m - RB;  // thread bits in use
  auto layout = [&](uint64_t thr) {
    // an opaque copy of the thread id, so the per-bit terms are not hoisted out of the op
    // loop and kept live in registers for the whole pass
    int tv = tid;
    asm volatile("" : "+v"(tv));
    int j = 0;
#pragma unroll
    for (int t = 0; t < MAXM - RB; ++t)
      if (t < nthr) j |= ((tv >> t) & 1) << (int)((thr >> (4 * t)) & 15);
    return j;
  };
  // LDS byte address of register slot k.  swz is linear over GF(2) and slot k's local index is
  // the thread part (slot 0) with the bits of k spread over the register bits, so the address
  // is a per-thread term, swz(thread part), XOR a wave-uniform term, swz(spread of k), itself
  // the XOR of the register bits' terms: 16 bits each of the planner's `units`.
  auto slot_offsets = [&](uint64_t units, int* off) {
    int u[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) u[i] = (int)((units >> (16 * i)) & 0xffff) * (int)sizeof(X);
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      int o = 0;
#pragma unroll
      for (int i = 0; i < RB; ++i)
        if ((k >> i) & 1) o ^= u[i];
      off[k] = o;
    }
  };
  auto lds_at = [&](int byte_off) -> X& { return *reinterpret_cast<X*>(reinterpret_cast<char*>(buf) + byte_off); };
  // Tables ahead of use: the ops read their records and numbers one dependent scalar load
  // after another, and right after an upload each of those loads comes from HBM.  One vector
  // load per 128-byte line brings all of them into this XCD's L2 at once, while the tile
  // loads.  10-qubit, 80-parameter ansatz (one workgroup, 116 ops): 500 -> 370 us per energy
  // and gradient.  Launches of many tiles share the lines, and the loads only cost there
  // (27-qubit brick 14.77 -> 14.93 ms), so they leave it out (kWarmTiles): by A.warm, or with the
  // code itself (WARM false) where its registers alone cost (complex64 reverse sweeps without
  // runs of phases, 64 sets of the 24-qubit QAOA: 189.2 -> 185.6 ms).
  uint32_t warm = 0;
  auto touch = [&](const void* p, int64_t bytes) {
    for (int64_t o = (int64_t)tid * 128; o < bytes; o += (int64_t)NT * 128)
      warm ^= *reinterpret_cast<const uint32_t*>(static_cast<const char*>(p) + o);
  };
  if (WARM && A.warm) {
    touch(A.ops, (int64_t)A.n_ops * sizeof(TileOp));
    touch(T + A.ctab_lo, (int64_t)A.ctab_n * sizeof(C));
    touch(A.diag + A.diag_lo, (int64_t)A.diag_n * sizeof(DiagEntry));
    touch(A.edges + A.edge_lo, (int64_t)A.edge_n * sizeof(ZZEdge));
  }
  // Index a local index is read from: two lookup tables of deposits (local bits 0..6 and
  // 7..13) computed by the planner for the pass; before the stores they are replaced by the
  // tables of the index it is written to when the pass relayouts.
  __shared__ uint64_t dep_lo[128], dep_hi[128];
  for (int i = tid; i < 128; i += NT) {
    dep_lo[i] = A.dep[i];
    dep_hi[i] = A.dep[128 + i];
  }
  // The pass's per-lane table lookups (ZZ phases and generator weights) read
  // a copy of their ctab window in dynamic LDS.
  C* win = reinterpret_cast<C*>(qsv_dyn_lds);
  const int win_n = A.win_n;
  // adjoint: per-(slot, wave) gradient sums after the window, reduced at the end of the pass
  constexpr int NW = NT >= 64 ? NT / 64 : 1;
  const bool defer = ADJ && A.pass_pslots * NW <= kMaxDeferredSums;
  double* gsum = reinterpret_cast<double*>(qsv_dyn_lds + win_bytes<R>(win_n));
  const int64_t win_lo = A.win_lo;
  for (int i = tid; i < win_n; i += NT) win[i] = T[win_lo + i];
  __syncthreads();
  auto tab = [&](int off) -> C { return win_n ? win[off - win_lo] : ldc(T + off); };

  int jt = layout(A.lay0_thr);                         // the thread's part of its local indices
  uint32_t reg_cur = A.lay0_reg;                       // register bits of the current layout
  uint64_t units_cur = A.lay0_units;                   // its register bits' terms of LDS addresses
  int sw_cur = swz<S>(jt) * (int)sizeof(X);            // per-thread term of its LDS addresses
  auto globals = [&](uint64_t tile_base, uint64_t* xo) {
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int j = jt | spread_of<NR>(reg_cur, k);
      xo[k] = tile_base | dep_lo[j & 127] | dep_hi[j >> 7];
    }
  };

  C v[NR], w[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    v[k] = C{0, 0};
    if (ADJ) w[k] = C{0, 0};
  }
  if (active) {
    uint64_t xk[NR];
    globals(A.relayout ? run_base(kRunsLoad) : base, xk);
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      v[k] = src[xk[k]];
      if (ADJ) w[k] = lam[xk[k]];
    }
  }
  asm volatile("" :: "v"(warm));
  // the value of an index bit that the thread's local index or the tile's base holds
  auto lane_bit = [&](uint32_t src) -> bool {
    return src < 32 ? ((uint32_t)jt >> src) & 1u : src < kNoBit && ((base >> (src - 32)) & 1);
  };
  double acc = 0.0;
  const TileOp* O = A.ops;
  for (int oi = 0; oi < A.n_ops; ++oi, ++O) {
    // the record's first 16 bytes (adjoint: 32 bytes) in one scalar load
    const uint64_t* hw = reinterpret_cast<const uint64_t*>(O);
    const uint64_t h0 = ld(hw), h1 = ld(hw + 1), h2 = ADJ ? ld(hw + 2) : 0, h3 = ADJ ? ld(hw + 3) : 0;
    const int plain = (int)(uint32_t)h0, mat = (int)(h0 >> 32);
    const int first = (int)(uint32_t)h1, count = (int)(h1 >> 32);
    const int gen = (int)(uint32_t)h2, pslot = (int)(h2 >> 32);
    const int flush = (int)(uint32_t)h3, gkind = (int)(h3 >> 32);
    if (ONE ? plain && !(plain & kPlainPhases) : plain) {
      // the short path: a run of sign flips, then a one-qubit gate on a register slot or a
      // fused block (or nothing), with nothing else to decode
      const int slot = (plain & 7) - 1;
      auto sign_run = [&]() {
        uint32_t touched;
        const uint32_t sm = sign_slots(A.diag + first, count, base, (uint32_t)jt, touched);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
          if (!((touched >> k) & 1u)) continue;
          const uint32_t f = (sm << (31 - k)) & 0x80000000u;
          flip_sign(v[k], f);
          if (ADJ) flip_sign(w[k], f);
        }
      };
      if (!ADJ && (plain & kPlainBlock)) {
        if (active) {
          if (plain & kPlainSigns) sign_run();
          // the lane's four A operands: 4 consecutive reals at 4 * lane of the block's table
          const R* ap = reinterpret_cast<const R*>(T + mat) + 4 * (tid & 63);
          R am[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) am[j] = ap[j];
          block_dispatch<RB>(slot, v, am);
        }
      } else if (slot < 0) {
        if (active) sign_run();
      } else if (plain & kPlainFlip) {
        // (controlled) X moves amplitudes and computes nothing.  As a 2x2 matrix with its
        // zeros, under controls, it took both products, a copy and a select per amplitude:
        // 10-qubit ansatz with 36 CNOTs 372 -> 333 us, 48 uneven
        // ansatz circuits 3337 -> 2977 us per energy and gradient.
        bool on = true;
        if (plain & kPlainOutside) {
          const uint64_t om = ld(&O->omask);
          on = (base & om) == om;
        }
        if (on && active) {
          const uint64_t lanes = __builtin_amdgcn_ballot_w64((jt & first) == first);
          const uint32_t pairs = (uint32_t)plain >> 16;
          flip_dispatch<RB>(slot, v, pairs, lanes);
          if (ADJ) flip_dispatch<RB>(slot, w, pairs, lanes);
        }
      } else if (active) {
        C U[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) U[r] = ldc(T + mat + r);
        if (plain & kPlainSigns) sign_run();
        const int form = (plain & kPlainForm) / kPlainSplit;
        if (ADJ && gen >= 0) {
          C G[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) G[r] = ldc(T + gen + r);
          // the generator forms of RX and RY come with their gates' matrix forms
          if (gkind == GEN_X && form == FORM_XLIKE) {
            double part = 0.0;
            reg1_slot<RB, ADJ, GEN_X, C, FORM_XLIKE>(slot, v, w, jt, reg_cur, 0u, U, true, G, part);
            acc = __builtin_fma((double)G[1].x, part, acc);
          } else if (gkind == GEN_Y && form == FORM_REAL) {
            double part = 0.0;
            reg1_slot<RB, ADJ, GEN_Y, C, FORM_REAL>(slot, v, w, jt, reg_cur, 0u, U, true, G, part);
            acc = __builtin_fma((double)G[2].y, part, acc);
          } else {
            reg1_dispatch<RB, ADJ>(slot, v, w, jt, reg_cur, 0u, U, true, gkind, G, acc);
          }
        } else if (!ADJ && form == FORM_SPLIT) {
          reg1_slot<RB, ADJ, GEN_GENERAL, C, FORM_SPLIT>(slot, v, w, jt, reg_cur, 0u, U, false, U, acc);
        } else if (form == FORM_REAL) {
          reg1_slot<RB, ADJ, GEN_GENERAL, C, FORM_REAL>(slot, v, w, jt, reg_cur, 0u, U, false, U, acc);
        } else if (form == FORM_XLIKE) {
          reg1_slot<RB, ADJ, GEN_GENERAL, C, FORM_XLIKE>(slot, v, w, jt, reg_cur, 0u, U, false, U, acc);
        } else {
          reg1_slot<RB, ADJ, GEN_GENERAL>(slot, v, w, jt, reg_cur, 0u, U, false, U, acc);
        }
      }
    } else {
      int type = OP_DIAG, ob = 1;  // (a run with phases: nothing else to read)
      uint32_t lm_raw = 0;
      if (!ONE || !plain) {
        type = ld(&O->type);
        lm_raw = ld(&O->lmask);
        ob = ld(&O->b);
      }
      bool on = true;
      if (lm_raw & kHasOutsideControls) {
        const uint64_t omask = ld(&O->omask);
        on = (base & omask) == omask;
      }
      const uint32_t lmask = lm_raw & ~kHasOutsideControls;
      // sign flips only (Z, CZ, multi-controlled Z), alone (DIAG with b = 0) or ahead of a
      // gate (DENSE1 with b = 1): the parity of the satisfied entries, as one bit per
      // register slot (slot 0 holds the thread's own local index)
      if (on && active && ((type == OP_DIAG && !ob) || (type == OP_DENSE1 && ob))) {
        uint32_t touched;
        const uint32_t sm = sign_slots(A.diag + first, count, base, (uint32_t)jt, touched);
        // slots no entry can reach are skipped (a wave-uniform test): an entry on a register
        // bit reaches half of them
#pragma unroll
        for (int k = 0; k < NR; ++k) {
          if (!((touched >> k) & 1u)) continue;
          const uint32_t f = (sm << (31 - k)) & 0x80000000u;
          flip_sign(v[k], f);
          if (ADJ) flip_sign(w[k], f);
        }
      }
      if (type == OP_REMAP || type == OP_XSWAP) {
        // the new layout: register slot bits, thread bits, the thread's part of its indices
        const uint32_t lr = (uint32_t)ld(&O->b);
        const int jn = layout(ld(&O->omask));
        const int sw_new = swz<S>(jn) * (int)sizeof(X);
        const uint64_t units = (uint64_t)(uint32_t)ld(&O->gkind) << 32 | (uint32_t)ld(&O->pslot);
        if (type == OP_XSWAP) {
          // one transposition per op, by cross-lane moves; every lane takes part (partners
          // of active lanes are active)
          const int code = mat & 255;
          xswap_dispatch<RB>(code, v);
          if (ADJ) xswap_dispatch<RB>(code, w);
        } else {
          int uo[NR], un[NR];
          slot_offsets(units_cur, uo);
          slot_offsets(units, un);
          if constexpr (SPLIT) {
            auto exchange = [&](auto part) {  // part(k): the component that moves
              if (active) {
#pragma unroll
                for (int k = 0; k < NR; ++k) lds_at(sw_cur ^ uo[k]) = part(k);
              }
              __syncthreads();
              if (active) {
#pragma unroll
                for (int k = 0; k < NR; ++k) part(k) = lds_at(sw_new ^ un[k]);
              }
              __syncthreads();
            };
            exchange([&](int k) -> R& { return v[k].x; });
            exchange([&](int k) -> R& { return v[k].y; });
          } else {
            if (active) {
#pragma unroll
              for (int k = 0; k < NR; ++k) lds_at(sw_cur ^ uo[k]) = v[k];
            }
            __syncthreads();
            if (active) {
#pragma unroll
              for (int k = 0; k < NR; ++k) v[k] = lds_at(sw_new ^ un[k]);
            }
            if (ADJ) {
              __syncthreads();
              if (active) {
#pragma unroll
                for (int k = 0; k < NR; ++k) lds_at(sw_cur ^ uo[k]) = w[k];
              }
              __syncthreads();
              if (active) {
#pragma unroll
                for (int k = 0; k < NR; ++k) w[k] = lds_at(sw_new ^ un[k]);
              }
            }
            __syncthreads();
          }
        }
        jt = jn;
        reg_cur = lr;
        units_cur = units;
        sw_cur = sw_new;
      } else if (on && active && type == OP_DENSE1) {
        C U[4], G[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) U[r] = ldc(T + mat + r);
        const bool grad = ADJ && gen >= 0;
        if (grad) {
#pragma unroll
          for (int r = 0; r < 4; ++r) G[r] = ldc(T + gen + r);
        }
        reg1_dispatch<RB, ADJ>(ld(&O->a), v, w, jt, reg_cur, lmask, U, grad, ADJ ? gkind : 0, G, acc);
      } else if (!SPLIT && on && type == OP_DENSE2) {
        if constexpr (!SPLIT) {
          // two-qubit dense gate on local bits a, b, applied to the tile staged in LDS (no
          // gradient: parameterized two-qubit rotations are lowered to RZZ with basis changes)
          const int a = ld(&O->a), bb = ld(&O->b);
          const int lo = a < bb ? a : bb, hi = a < bb ? bb : a;
          const uint32_t lm = lmask;
          int uo[NR];
          slot_offsets(units_cur, uo);
          auto apply_staged = [&](C (&reg)[NR]) {
            if (active) {
#pragma unroll
              for (int k = 0; k < NR; ++k) lds_at(sw_cur ^ uo[k]) = reg[k];
            }
            __syncthreads();
            for (int p = tid; p < (nloc >> 2); p += NT) {
              const int t = insert_zero(insert_zero(p, lo), hi);
              if (((uint32_t)t & lm) != lm) continue;
              const int idx[4] = {t, t | (1 << a), t | (1 << bb), t | (1 << a) | (1 << bb)};
              C x[4], y[4];
#pragma unroll
              for (int r = 0; r < 4; ++r) x[r] = buf[swz<S>(idx[r])];
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                y[r] = cdot2(ldc(T + mat + 4 * r), x[0], ldc(T + mat + 4 * r + 1), x[1]);
                y[r] = cdot2(C{1, 0}, y[r], ldc(T + mat + 4 * r + 2), x[2]);
                y[r] = cdot2(C{1, 0}, y[r], ldc(T + mat + 4 * r + 3), x[3]);
              }
#pragma unroll
              for (int r = 0; r < 4; ++r) buf[swz<S>(idx[r])] = y[r];
            }
            __syncthreads();
            if (active) {
#pragma unroll
              for (int k = 0; k < NR; ++k) reg[k] = lds_at(sw_cur ^ uo[k]);
            }
            __syncthreads();
          };
          apply_staged(v);
          if (ADJ) apply_staged(w);
        }
      } else if (on && active && type == OP_DIAG && ob) {
        // Entry by entry: one read of the entry, one of its two or four phases (and
        // weights), then each slot times the phase that its own bits, its lane's and the
        // tile's select.  The slots that share a phase go together, so an entry on a slot
        // bit forms two phases and one on lanes or outside bits a single one per lane.
        // Walking the run once per slot pair, with every index formed per slot and looked up
        // per lane, took about 12 dependent reads per entry: 10-qubit ansatz with 80 angles
        // 333 -> 254 us, 120 gates of every kind on 23 qubits in complex64 711 -> 500 us, 48
        // uneven ansatz circuits 2977 -> 2400 us.
        // Complex64 passes multiply a run's phases (and sum its weights) per slot first and then
        // the amplitudes once; complex128 passes, where a second register block would cut the
        // resident waves, multiply the amplitudes entry by entry.
        constexpr bool gather = sizeof(R) == 4;
        // Slots at a time: complex64 reverse sweeps walk a run twice, half of the slots each, for the
        // registers of sweeps that have no such runs but share the kernel.  QAOA on 24 qubits, 32
        // sets, backward 93.8 ms; all slots at once 96.3, quarters 95.8.  (Four layers of 20 phases
        // with one parameter, 32 sets on 20 qubits: 4.1 ms, all slots at once 3.7, quarters 5.2.)
        constexpr int NG = gather && ADJ ? NR / 2 : NR;
        // The reverse sweep's runs are mostly one uncontrolled one-qubit phase each (every run has
        // one parameter): its numbers are read along with its entry, and slot-resident qubits
        // take one straight line per slot bit instead of a test per slot.  10-qubit ansatz gradient
        // 230 -> 195 us, 20-qubit one (6 layers, 4 sets, complex64) 1837 -> 1539 us, 48 uneven
        // ansatz circuits 2570 -> 2200 us.
        bool done = false;
        if constexpr (ONE) {
          if (count == 1) {
            const C q0 = ldc(T + mat), q1 = ldc(T + mat + 1);
            double w0 = 0.0, w1 = 0.0;
            if (gen >= 0) {
              w0 = (double)ldc(T + gen).x;
              w1 = (double)ldc(T + gen + 1).x;
            }
            const PhaseFields f = ld_record(reinterpret_cast<const PhaseFields*>(&A.diag[first].ocmask));
            if (f.where & kWhereOne) {
              const int at = (int)(f.where >> 24) - 1;
              if (at < 0) {  // the same phase in every slot
                const bool t = lane_bit(f.where & 255u);
                phase1<-1, NR>(v, w, csel(t, q1, q0), q1, t ? w1 : w0, 0.0, acc);
              } else {
                phase1_dispatch<RB>(at, v, w, q0, q1, w0, w1, acc);
              }
              done = true;
            }
          }
        }
        if (!done) {
#pragma unroll
          for (int kg = 0; kg < NR; kg += NG) {
            uint32_t flips = 0, touched = 0;
            C ph[gather ? NG : 1];
            double gws[gather && ADJ ? NG : 1];
#pragma unroll
            for (int k = 0; k < (gather ? NG : 0); ++k) {
              ph[k] = C{1, 0};
              if (ADJ) gws[k] = 0.0;
            }
            for (int e = 0; e < count; ++e) {
              const PhaseFields f = ld_record(reinterpret_cast<const PhaseFields*>(&A.diag[first + e].ocmask));
              if ((base & f.ocmask) != f.ocmask) continue;  // an outside control is 0 in this tile
              const bool in = ((uint32_t)jt & f.tmask) == f.tmask;
              if (f.where & kWhereSign) {
                flips ^= in ? f.kmask : 0u;
                touched |= f.kmask;
                continue;
              }
              const bool two = (f.where & kWhereTwo) != 0, grad = ADJ && f.gtab >= 0;
              const bool t0 = lane_bit(f.where & 255u), t1 = lane_bit((f.where >> 8) & 255u);
              for (uint32_t u = 0; u < 4; ++u) {
                if (((u & 1) && !f.bits0) || ((u & 2) && !f.bits1)) continue;
                const uint32_t ks = f.kmask & ((u & 1) ? f.bits0 : ~f.bits0) & ((u & 2) ? f.bits1 : ~f.bits1);
                // half of the table that a lane's second bit selects, then the entry its first does
                const bool i0 = t0 || (u & 1), i1 = t1 || (u & 2);
                C p = csel(i0, ldc(T + f.tab + 1), ldc(T + f.tab));
                if (two) p = csel(i1, csel(i0, ldc(T + f.tab + 3), ldc(T + f.tab + 2)), p);
                p = csel(in, p, C{1, 0});
                double gw = 0.0;
                if (grad) {
                  gw = (double)(i0 ? ldc(T + f.gtab + 1).x : ldc(T + f.gtab).x);
                  if (two) gw = i1 ? (double)(i0 ? ldc(T + f.gtab + 3).x : ldc(T + f.gtab + 2).x) : gw;
                }
                if constexpr (gather) {
                  const double gs = in ? gw : 0.0;
#pragma unroll
                  for (int k = 0; k < NG; ++k) {
                    if (!((ks >> (kg + k)) & 1u)) continue;
                    ph[k] = cmul(ph[k], p);
                    if (ADJ) gws[k] += gs;
                  }
                  continue;
                }
                if (grad) {
                  double g = 0.0;
#pragma unroll
                  for (int k = 0; k < NR; ++k)
                    if ((ks >> k) & 1u) g += im_conj_mul(w[k], v[k]);
                  acc = __builtin_fma(in ? gw : 0.0, g, acc);
                }
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                  if (!((ks >> k) & 1u)) continue;
                  if (ADJ) cmul_in(w[k], p);
                  cmul_in(v[k], p);
                }
              }
            }
#pragma unroll
            for (int i = 0; i < NG; ++i) {
              const int k = kg + i;
              const uint32_t f = (flips << (31 - k)) & 0x80000000u;
              if constexpr (gather) {
                flip_sign(ph[i], f);
                if (ADJ) {
                  double g = gws[i] * im_conj_mul(w[k], v[k]);
                  cmul_in(w[k], ph[i], g);
                  cmul_in(v[k], ph[i], g);
                  acc += g;
                } else {
                  cmul_in(v[k], ph[i]);
                }
              } else {
                if (!((touched >> k) & 1u)) continue;
                flip_sign(v[k], f);
                if (ADJ) flip_sign(w[k], f);
              }
            }
          }
        }
      } else if (on && active && type == OP_ZZ) {
        // c(x) = number of edges whose endpoints differ.  Edges come grouped by register
        // class c; an edge of class c differs in slot k iff its thread/outside parity
        // differs from the parity of (k & c), so with a_c = the class's edges whose
        // thread/outside parity is odd, c(slot k) = sum_c a_c + sum_{c: k & c odd} (n_c - 2 a_c).
        // classes are register-bit masks of at most two bits, listed by zz_class<RB>(i); the
        // edge count of class i is byte i of (a, b, lmask)
        const uint32_t cw[3] = {(uint32_t)ld(&O->a), (uint32_t)ld(&O->b), lm_raw};
        const ZZEdge* ed = A.edges + first;
        constexpr int NCLS = zz_classes<RB>();
        int sum_a = 0, dcls[NCLS];
        int e = 0;
#pragma unroll
        for (int c = 0; c < NCLS; ++c) {
          const int nc = (int)((cw[c >> 2] >> (8 * (c & 3))) & 255u);
          int a_c = 0;
          for (int i = 0; i < nc; ++i, ++e) {
            const uint32_t tm = ld(&ed[e].tmask);
            const uint64_t om = ld(&ed[e].omask);
            a_c += (__popc(jt & tm) + __popcll(base & om)) & 1;
          }
          sum_a += a_c;
          dcls[c] = nc - 2 * a_c;
        }
#pragma unroll
        for (int k = 0; k < NR; ++k) {
          int cnt = sum_a;
#pragma unroll
          for (int c = 1; c < NCLS; ++c)
            if (__builtin_popcount(k & zz_class<RB>(c)) & 1) cnt += dcls[c];
          const C p = tab(mat + cnt);
          if (ADJ) {
            double g = 0.0;
            if (gen >= 0) g = (double)tab(gen + cnt).x * im_conj_mul(w[k], v[k]);
            cmul_in(w[k], p, g);
            cmul_in(v[k], p, g);
            acc += g;
          } else {
            cmul_in(v[k], p);
          }
        }
      }
    }
    if (ADJ && flush) {
      const double sv = wave_sum(acc);
      if (defer) {
        if ((tid & 63) == 0) gsum[pslot * NW + (tid >> 6)] = sv;
      } else {
        if ((tid & 63) == 0) red[tid >> 6] = sv;
        __syncthreads();
        if (tid == 0) {
          double s = 0.0;
          for (int q = 0; q < NW; ++q) s += red[q];
          A.partials[((int64_t)b * A.n_pslots + pslot) * A.n_tiles + (int64_t)tile] = s;
        }
        __syncthreads();
      }
      acc = 0.0;
    }
  }
  if (defer) {
    __syncthreads();
    for (int q = tid; q < A.pass_pslots; q += NT) {
      double s = 0.0;
      for (int w2 = 0; w2 < NW; ++w2) s += gsum[q * NW + w2];
      A.partials[((int64_t)b * A.n_pslots + q) * A.n_tiles + (int64_t)tile] = s;
    }
  }

  uint64_t store_base = base;
  if (A.relayout) {
    __syncthreads();
    for (int i = tid; i < 128; i += NT) {
      dep_lo[i] = A.dep[256 + i];
      dep_hi[i] = A.dep[384 + i];
    }
    __syncthreads();
    store_base = run_base(kRunsStore);
  }
  if (active) {
    uint64_t xk[NR];
    globals(store_base, xk);
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      out[xk[k]] = v[k];
      if (ADJ) lam[xk[k]] = w[k];
    }
  }
}

template <typename R, int RB, int MAXM, bool ADJ, bool ALT, bool WARM>
__global__ __launch_bounds__(1 << (MAXM - RB), ALT && !ADJ ? kSplitWaves<R> : 1) void tile_pass_rb(PassArgs A) {
  // Workgroups go to the 8 XCDs in turn; give each XCD a contiguous range of tiles, so
  // tiles that share cache lines (they differ only in low qubits outside the tile) run
  // back to back behind the same L2.
  const uint32_t g = gridDim.x, w = blockIdx.x;
  const uint64_t t = (g % 8 == 0) ? (uint64_t)(w & 7) * (g >> 3) + (w >> 3) : w;
  rb_body<R, RB, MAXM, ADJ, true, ALT, WARM>(A, t, blockIdx.y);
}

// Many circuits in one launch: item i owns workgroups [prefix[i], prefix[i+1]); each
// workgroup finds its item by binary search and runs that circuit's pass on one tile.
template <typename R, int RB, int MAXM, bool ADJ>
__global__ __launch_bounds__(1 << (MAXM - RB)) void tile_pass_rb_multi(const PassArgs* items, const uint32_t* prefix,
                                                                       int n_items) {
  const uint32_t w = blockIdx.x;
  int lo = 0, hi = n_items;  // largest i with prefix[i] <= w
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (ld(prefix + mid) <= w) lo = mid; else hi = mid;
  }
  const PassArgs A = items[lo];
  rb_body<R, RB, MAXM, ADJ, false, ADJ, true>(A, (uint64_t)(w - ld(prefix + lo)), 0);
}

template <typename R, int RB, int MAXM, bool ADJ>
static hipError_t rb_launch_one(const PassArgs& A, dim3 grid, hipStream_t s) {
  constexpr size_t bytes = (size_t)(2 * sizeof(R)) * ((size_t)1 << MAXM);
  // four register bits: complex64 forward passes only (their registers allow 4 waves/SIMD)
  if constexpr (bytes <= 131072 && (RB == 3 || (!ADJ && sizeof(R) == 4 && MAXM >= 10))) {
    const size_t dyn = rb_dyn_lds<R>(MAXM, ADJ, A.win_n, A.pass_pslots);
    constexpr bool lean = ADJ && sizeof(R) == 4;  // (see WARM)
    if (A.alt) tile_pass_rb<R, RB, MAXM, ADJ, true, true><<<grid, 1 << (MAXM - RB), dyn, s>>>(A);
    else if (lean && !A.warm) tile_pass_rb<R, RB, MAXM, ADJ, false, !lean><<<grid, 1 << (MAXM - RB), dyn, s>>>(A);
    else tile_pass_rb<R, RB, MAXM, ADJ, false, true><<<grid, 1 << (MAXM - RB), dyn, s>>>(A);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

template <typename R, bool ADJ, int RB>
static hipError_t rb_dispatch_rb(int maxm, const PassArgs& A, dim3 grid, hipStream_t s) {
  switch (maxm) {
    case 9:  return rb_launch_one<R, RB, 9, ADJ>(A, grid, s);
    case 10: return rb_launch_one<R, RB, 10, ADJ>(A, grid, s);
    case 11: return rb_launch_one<R, RB, 11, ADJ>(A, grid, s);
    case 12: return rb_launch_one<R, RB, 12, ADJ>(A, grid, s);
    case 13: return rb_launch_one<R, RB, 13, ADJ>(A, grid, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename R, bool ADJ>
hipError_t rb_dispatch(int reg_bits, int maxm, const PassArgs& A, uint64_t n_tiles, int batch,
                              hipStream_t s) {
  const dim3 grid((unsigned)n_tiles, (unsigned)batch);
  if (reg_bits == 3) return rb_dispatch_rb<R, ADJ, 3>(maxm, A, grid, s);
  if (reg_bits == 4) return rb_dispatch_rb<R, ADJ, 4>(maxm, A, grid, s);
  return hipErrorInvalidValue;
}

template <typename R, bool ADJ>
hipError_t rb_multi_dispatch(int maxm, const PassArgs* items, const uint32_t* prefix, int n_items,
                                    uint32_t n_wg, int max_win, int max_pslots, hipStream_t s) {
  const size_t dyn = rb_dyn_lds<R>(maxm, ADJ, max_win, max_pslots);
  switch (maxm) {
#define QSV_MULTI(M)                                                                                   \
  case M:                                                                                              \
    if constexpr ((size_t)(2 * sizeof(R)) * ((size_t)1 << M) <= 131072) {                              \
      tile_pass_rb_multi<R, 3, M, ADJ><<<n_wg, 1 << (M - 3), dyn, s>>>(items, prefix, n_items);        \
      return hipGetLastError();                                                                        \
    }                                                                                                  \
    return hipErrorInvalidValue;
    QSV_MULTI(9) QSV_MULTI(10) QSV_MULTI(11) QSV_MULTI(12) QSV_MULTI(13)
#undef QSV_MULTI
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qsv
