// Device helpers shared by the kernels: complex arithmetic on register-resident amplitudes,
// cross-lane sums, and reads of the planner's tables through the scalar path.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qsv {

template <typename R> struct CT;
template <> struct CT<float>  { using T = float2; };
template <> struct CT<double> { using T = double2; };

__device__ __forceinline__ float  fmaT(float a, float b, float c)    { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <typename C> __device__ __forceinline__ C cmul(C a, C b) {
  C r;
  r.x = fmaT(a.x, b.x, -a.y * b.y);
  r.y = fmaT(a.x, b.y, a.y * b.x);
  return r;
}
// u0 * v0 + u1 * v1
template <typename C> __device__ __forceinline__ C cdot2(C u0, C v0, C u1, C v1) {
  C r;
  r.x = fmaT(u0.x, v0.x, fmaT(-u0.y, v0.y, fmaT(u1.x, v1.x, -u1.y * v1.y)));
  r.y = fmaT(u0.x, v0.y, fmaT(u0.y, v0.x, fmaT(u1.x, v1.y, u1.y * v1.x)));
  return r;
}
// Im(conj(w) * g) in fp64
template <typename C> __device__ __forceinline__ double im_conj_mul(C w, C g) {
  return (double)w.x * (double)g.y - (double)w.y * (double)g.x;
}

// Register-resident updates.  A pass keeps each amplitude in the same registers from op to
// op only if every op overwrites an input component with the one multiply-add that reads it
// last.  So each output component is finished by a multiply-add on the component it
// replaces; all other reads of the inputs feed partial sums that pass through an empty asm
// first, which orders them before every finishing multiply-add.  That multiply-add is
// itself an asm: the compiler's two-address form would tie the result to the partial sum's
// register instead.
template <typename R> __device__ __forceinline__ void order(R& a, R& b) { asm("" : "+v"(a), "+v"(b)); }
template <typename R> __device__ __forceinline__ void order(R& a, R& b, double& e) {
  asm("" : "+v"(a), "+v"(b), "+v"(e));
}
template <typename R> __device__ __forceinline__ void order(R& a, R& b, R& c, R& d) {
  asm("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}
template <typename R> __device__ __forceinline__ void order(R& a, R& b, R& c, R& d, double& e) {
  asm("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d), "+v"(e));
}
// a * b + c; fma_s takes a wave-uniform a (an SGPR operand)
__device__ __forceinline__ double fma_s(double a, double b, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "s"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ float fma_s(float a, float b, float c) {
  float r;
  asm("v_fma_f32 %0, %1, %2, %3" : "=v"(r) : "s"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ double fma_v(double a, double b, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ float fma_v(float a, float b, float c) {
  float r;
  asm("v_fma_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// (a0, a1) <- (u00 a0 + u01 a1, u10 a0 + u11 a1) in place, u wave-uniform.  The optional
// `pin` (a value computed from the old inputs, e.g. a gradient term) is held back with
// the partial sums, so it too is computed before any input is overwritten.
template <typename C, typename... Pin>
__device__ __forceinline__ void apply2(C u00, C u01, C u10, C u11, C& a0, C& a1, Pin&... pin) {
  auto p0r = fmaT(-u00.y, a0.y, fmaT(u01.x, a1.x, -u01.y * a1.y));
  auto p0i = fmaT(u00.y, a0.x, fmaT(u01.x, a1.y, u01.y * a1.x));
  auto p1r = fmaT(u10.x, a0.x, fmaT(-u10.y, a0.y, -u11.y * a1.y));
  auto p1i = fmaT(u10.x, a0.y, fmaT(u10.y, a0.x, u11.y * a1.x));
  order(p0r, p0i, p1r, p1i, pin...);
  a0.x = fma_s(u00.x, a0.x, p0r);
  a0.y = fma_s(u00.x, a0.y, p0i);
  a1.x = fma_s(u11.x, a1.x, p1r);
  a1.y = fma_s(u11.x, a1.y, p1i);
}
// a1 <- a1 * p, then (a0, a1) <- (r0.x a0 + r0.y a1, r1.x a0 + r1.y a1) with real r, in place
// (p and r wave-uniform): a phase and a real 2x2 matrix, 12 instructions per pair
template <typename C>
__device__ __forceinline__ void apply2split(C r0, C r1, C p, C& a0, C& a1) {
  {
    auto pr = -a1.y * p.y;
    auto pi = a1.x * p.y;
    order(pr, pi);
    a1.x = fma_s(p.x, a1.x, pr);
    a1.y = fma_s(p.x, a1.y, pi);
  }
  auto p0r = r0.y * a1.x;
  auto p0i = r0.y * a1.y;
  auto p1r = r1.x * a0.x;
  auto p1i = r1.x * a0.y;
  order(p0r, p0i, p1r, p1i);
  a0.x = fma_s(r0.x, a0.x, p0r);
  a0.y = fma_s(r0.x, a0.y, p0i);
  a1.x = fma_s(r1.y, a1.x, p1r);
  a1.y = fma_s(r1.y, a1.y, p1i);
}
__host__ __device__ __forceinline__ uint32_t high_word(double v) {
  uint64_t u;
  __builtin_memcpy(&u, &v, 8);
  return (uint32_t)(u >> 32);
}
__host__ __device__ __forceinline__ uint32_t high_word(float v) {
  uint32_t u;
  __builtin_memcpy(&u, &v, 4);
  return u;
}
// A gate of a phase chain whose matrices keep unit entries (chain_gate): a1 <- a1 p with p = 1 +
// i t (IMAG: t + i), then (a0, a1) <- (a0 + r0 a1, r1 a0 + a1) (CROSS: (r0 a0 + a1, a0 + r1
// a1)): one multiply-add per entry that is not 1, 6 instructions per pair, against 12 with a
// phase and a full real matrix and 16 for the general product.  30-qubit brick in complex128, whole
// step with remaps in two halves (rb_body's SPLIT): 16 instructions 205 ms, 12 172 ms, 6 143 ms;
// without, where the passes wait on their waves' latency more than on the vector ALU, 16 222 ms, 6
// 200 ms.
template <bool IMAG, bool CROSS, typename R, typename C>
__device__ __forceinline__ void apply2unit(R r0, R r1, R t, C& a0, C& a1) {
  R x = IMAG ? fmaT(t, a1.x, -a1.y) : fmaT(-t, a1.y, a1.x);
  R y = IMAG ? fmaT(t, a1.y, a1.x) : fmaT(t, a1.x, a1.y);
  order(x, y);
  a1.x = CROSS ? fma_s(r1, x, a0.x) : fma_s(r1, a0.x, x);
  a1.y = CROSS ? fma_s(r1, y, a0.y) : fma_s(r1, a0.y, y);
  order(a1.x, a1.y, x, y);  // a0 is overwritten after its last use
  a0.x = CROSS ? fma_s(r0, a0.x, x) : fma_s(r0, x, a0.x);
  a0.y = CROSS ? fma_s(r0, a0.y, y) : fma_s(r0, y, a0.y);
}
// Matrix forms of one-qubit gates (bits 5-6 of TileOp::plain): general, split (a phase then
// a real matrix), real (RY, H, X), and real diagonal with imaginary off-diagonal (RX, Y).
enum MatForm : int { FORM_GENERAL = 0, FORM_SPLIT = 1, FORM_REAL = 2, FORM_XLIKE = 3 };
// apply2 for a form: real U (entries' .x) or U = [[a, i b], [i c, d]] (a, d in .x, b, c in .y)
// in 8 instructions per pair, else the general product
template <int F, typename C, typename... Pin>
__device__ __forceinline__ void apply2f(const C* U, C& a0, C& a1, Pin&... pin) {
  if constexpr (F == FORM_REAL) {
    auto p0r = U[1].x * a1.x;
    auto p0i = U[1].x * a1.y;
    auto p1r = U[2].x * a0.x;
    auto p1i = U[2].x * a0.y;
    order(p0r, p0i, p1r, p1i, pin...);
    a0.x = fma_s(U[0].x, a0.x, p0r);
    a0.y = fma_s(U[0].x, a0.y, p0i);
    a1.x = fma_s(U[3].x, a1.x, p1r);
    a1.y = fma_s(U[3].x, a1.y, p1i);
  } else if constexpr (F == FORM_XLIKE) {
    auto p0r = -U[1].y * a1.y;
    auto p0i = U[1].y * a1.x;
    auto p1r = -U[2].y * a0.y;
    auto p1i = U[2].y * a0.x;
    order(p0r, p0i, p1r, p1i, pin...);
    a0.x = fma_s(U[0].x, a0.x, p0r);
    a0.y = fma_s(U[0].x, a0.y, p0i);
    a1.x = fma_s(U[3].x, a1.x, p1r);
    a1.y = fma_s(U[3].x, a1.y, p1i);
  } else {
    apply2(U[0], U[1], U[2], U[3], a0, a1, pin...);
  }
}
// a <- a * p in place (p per lane), with an optional `pin` as above
template <typename C, typename... Pin> __device__ __forceinline__ void cmul_in(C& a, C p, Pin&... pin) {
  auto pr = -a.y * p.y;
  auto pi = a.x * p.y;
  order(pr, pi, pin...);
  a.x = fma_v(p.x, a.x, pr);
  a.y = fma_v(p.x, a.y, pi);
}

// ... p wave-uniform
template <typename C, typename... Pin> __device__ __forceinline__ void cmul_in_s(C& a, C p, Pin&... pin) {
  auto pr = -a.y * p.y;
  auto pi = a.x * p.y;
  order(pr, pi, pin...);
  a.x = fma_s(p.x, a.x, pr);
  a.y = fma_s(p.x, a.y, pi);
}

// Negate v when f is 0x80000000 (f = 0: unchanged), by flipping the sign bits.
__device__ __forceinline__ void flip_sign(float2& v, uint32_t f) {
  v.x = __uint_as_float(__float_as_uint(v.x) ^ f);
  v.y = __uint_as_float(__float_as_uint(v.y) ^ f);
}
__device__ __forceinline__ void flip_sign(double2& v, uint32_t f) {
  const uint64_t g = (uint64_t)f << 32;
  v.x = __longlong_as_double(__double_as_longlong(v.x) ^ g);
  v.y = __longlong_as_double(__double_as_longlong(v.y) ^ g);
}

// Deposit the low bits of v into the set positions of mask (ascending).
__device__ __forceinline__ uint64_t pdep64(uint64_t v, uint64_t mask) {
  uint64_t r = 0;
  while (mask && v) {
    const uint64_t low = mask & (~mask + 1);
    if (v & 1) r |= low;
    v >>= 1;
    mask &= mask - 1;
  }
  return r;
}

// The value of a lane chosen by a DPP control (0: where the control selects no lane).
template <int CTRL> __device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// x + (x of lane l ^ 16) (L = 4) or l ^ 32 (L = 5), when x is equal across the 16 (32) lanes
// of each row (half-wave): the row (half-wave) swap of two copies leaves one of each pair.
template <int L> __device__ __forceinline__ double swap_add_f64(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  uint32_t a0 = (uint32_t)u, b0 = a0, a1 = (uint32_t)(u >> 32), b1 = a1;
  if constexpr (L == 5) {
    const auto r0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false);
    const auto r1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
    a0 = r0[0]; b0 = r0[1]; a1 = r1[0]; b1 = r1[1];
  } else {
    const auto r0 = __builtin_amdgcn_permlane16_swap(a0, b0, false, false);
    const auto r1 = __builtin_amdgcn_permlane16_swap(a1, b1, false, false);
    a0 = r0[0]; b0 = r0[1]; a1 = r1[0]; b1 = r1[1];
  }
  return __longlong_as_double((long long)(((uint64_t)a1 << 32) | a0)) +
         __longlong_as_double((long long)(((uint64_t)b1 << 32) | b0));
}
// Sum over the 64 lanes of a wave, returned in every lane (every lane must be active): a
// butterfly by cross-lane moves that stay out of LDS - quad permutes for lane bits 0 and 1,
// the half-row and row mirrors for bits 2 and 3 (each quad, then each half-row, already
// holds one value), the row and half-wave swaps for bits 4 and 5.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]: lane ^ 1
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]: lane ^ 2
  v += dpp_f64<0x141>(v);  // row_half_mirror: the other quad of the half-row
  v += dpp_f64<0x140>(v);  // row_mirror: the other half of the row
  v = swap_add_f64<4>(v);
  return swap_add_f64<5>(v);
}

// Read-only tables (op lists, diagonal entries, edges, bound matrices, Pauli terms) are
// read through the constant address space: uniform addresses then become scalar loads
// through the scalar cache instead of vector memory instructions.
#define QSV_CONST __attribute__((address_space(4)))
template <typename T> __device__ __forceinline__ T ld(const T* p) { return *(const QSV_CONST T*)p; }
// A whole record through the scalar path, dword by dword (the loads merge into wide
// scalar loads).
template <typename T> __device__ __forceinline__ T ld_record(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "record size must be a multiple of 4 bytes");
  T r;
  uint32_t* d = reinterpret_cast<uint32_t*>(&r);
  const QSV_CONST uint32_t* q = (const QSV_CONST uint32_t*)(const void*)p;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) d[i] = q[i];
  return r;
}
template <typename C> __device__ __forceinline__ C ldc(const C* p) {
  using R = decltype(p->x);
  const QSV_CONST R* q = (const QSV_CONST R*)p;
  C r;
  r.x = q[0];
  r.y = q[1];
  return r;
}

}  // namespace qsv
