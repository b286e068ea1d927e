// HIP kernels of the state-vector engine outside the fused tile passes (tile_rb.h,
// tile_lds.hip), and the launchers of the register-blocked ones.  Written for gfx950 (CDNA4,
// wave64).
//  gate1/gate2/diag_stream
//                 unfused per-gate passes over HBM (baseline path and tile-width 0).
//  pauli_group    one read pass per group of Pauli terms sharing an x-mask: expectation
//                 partials and, optionally, lambda = H psi.
//  reduce_columns fixed-order fp64 sums of per-block partials (bitwise repeatable).
#include "device_util.h"
#include "qsv_kernels.h"

namespace qsv {

// ------------------------------------------------------------------------------------------
// Unfused per-gate passes (grid-stride over amplitude pairs / quads / amplitudes).
// ------------------------------------------------------------------------------------------
template <typename R>
__global__ __launch_bounds__(256) void gate1_stream(void* psi_, int64_t bstride, int n, int t,
                                                    uint64_t cmask, const void* ctab_,
                                                    int64_t ctab_bstride, int mat) {
  using C = typename CT<R>::T;
  C* psi = reinterpret_cast<C*>(psi_) + (int64_t)blockIdx.y * bstride;
  const C* T = reinterpret_cast<const C*>(ctab_) + (int64_t)blockIdx.y * ctab_bstride + mat;
  const C u00 = T[0], u01 = T[1], u10 = T[2], u11 = T[3];
  const uint64_t half = 1ull << (n - 1);
  const uint64_t lowm = (1ull << t) - 1;
  for (uint64_t p = (uint64_t)blockIdx.x * 256 + threadIdx.x; p < half; p += (uint64_t)gridDim.x * 256) {
    const uint64_t x0 = ((p >> t) << (t + 1)) | (p & lowm);
    if ((x0 & cmask) != cmask) continue;
    const uint64_t x1 = x0 | (1ull << t);
    const C v0 = psi[x0], v1 = psi[x1];
    psi[x0] = cdot2(u00, v0, u01, v1);
    psi[x1] = cdot2(u10, v0, u11, v1);
  }
}

template <typename R>
__global__ __launch_bounds__(256) void gate2_stream(void* psi_, int64_t bstride, int n, int ta, int tb,
                                                    uint64_t cmask, const void* ctab_,
                                                    int64_t ctab_bstride, int mat) {
  using C = typename CT<R>::T;
  C* psi = reinterpret_cast<C*>(psi_) + (int64_t)blockIdx.y * bstride;
  const C* U = reinterpret_cast<const C*>(ctab_) + (int64_t)blockIdx.y * ctab_bstride + mat;
  const int lo = ta < tb ? ta : tb, hi = ta < tb ? tb : ta;
  const uint64_t quarter = 1ull << (n - 2);
  for (uint64_t p = (uint64_t)blockIdx.x * 256 + threadIdx.x; p < quarter; p += (uint64_t)gridDim.x * 256) {
    uint64_t x = ((p >> lo) << (lo + 1)) | (p & ((1ull << lo) - 1));
    x = ((x >> hi) << (hi + 1)) | (x & ((1ull << hi) - 1));
    if ((x & cmask) != cmask) continue;
    const uint64_t idx[4] = {x, x | (1ull << ta), x | (1ull << tb), x | (1ull << ta) | (1ull << tb)};
    C v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = psi[idx[r]];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      C o = cdot2(U[4 * r], v[0], U[4 * r + 1], v[1]);
      o = cdot2(C{1, 0}, o, U[4 * r + 2], v[2]);
      o = cdot2(C{1, 0}, o, U[4 * r + 3], v[3]);
      psi[idx[r]] = o;
    }
  }
}

template <typename R>
__global__ __launch_bounds__(256) void diag_stream(void* psi_, int64_t bstride, int n,
                                                   const DiagEntry* diag, int first, int count,
                                                   const void* ctab_, int64_t ctab_bstride) {
  using C = typename CT<R>::T;
  C* psi = reinterpret_cast<C*>(psi_) + (int64_t)blockIdx.y * bstride;
  const C* T = reinterpret_cast<const C*>(ctab_) + (int64_t)blockIdx.y * ctab_bstride;
  const uint64_t N = 1ull << n;
  for (uint64_t x = (uint64_t)blockIdx.x * 256 + threadIdx.x; x < N; x += (uint64_t)gridDim.x * 256) {
    C ph = C{1, 0};
    int sign = 0;
    for (int e = 0; e < count; ++e) {
      const DiagEntry* d = diag + first + e;
      const uint64_t cm = ld(&d->cmask);
      if (ld(&d->kind) == DIAG_SIGN) {
        sign ^= (int)((x & cm) == cm);
      } else if ((x & cm) == cm) {
        const int q1 = ld(&d->q1);
        const int idx = (int)((x >> ld(&d->q0)) & 1) | (q1 >= 0 ? (int)((x >> q1) & 1) << 1 : 0);
        ph = cmul(ph, ldc(T + ld(&d->mat) + idx));
      }
    }
    if (sign) { ph.x = -ph.x; ph.y = -ph.y; }
    psi[x] = cmul(psi[x], ph);
  }
}

// ------------------------------------------------------------------------------------------
// Pauli-sum group pass.
// ------------------------------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void group_factor(const PauliGroupArgs& A, uint64_t x, double& fr, double& fi) {
  fr = 0.0;
  fi = 0.0;
  for (int k = 0; k < A.n_terms; ++k) {
    const double s = (__popcll(x & ld(A.zmasks + k)) & 1) ? -1.0 : 1.0;
    fr = __builtin_fma(s, ld(A.cre + k), fr);
    fi = __builtin_fma(s, ld(A.cim + k), fi);
  }
}

// One instantiation per way of walking the group (the host picks it from the group's
// shape), so that each path is allocated registers for itself alone.  Pattern modes (0-3):
// bit 0 the term table staged in LDS once per workgroup, bit 1 lambda written.
enum PauliMode { PG_STAGED = 1, PG_LAM = 2, PG_QUAD = 4, PG_DIAG = 5, PG_XMASK = 6 };
constexpr int kPauliStageTerms = 512;

template <typename R, int MODE>
__global__ __launch_bounds__(256) void pauli_group(PauliGroupArgs A) {
  using C = typename CT<R>::T;
  __shared__ double red[2][4];
  const C* psi = reinterpret_cast<const C*>(A.psi) + (int64_t)blockIdx.y * A.bstride;
  C* lam = A.lam ? reinterpret_cast<C*>(A.lam) + (int64_t)blockIdx.y * A.bstride : nullptr;
  const uint64_t N = 1ull << A.n_qubits;
  const uint64_t stride = (uint64_t)gridDim.x * 256;
  double er = 0.0, ei = 0.0;
  if constexpr (MODE < PG_QUAD) {
    // Diagonal group with real coefficients, in chunks of 4096 consecutive amplitudes
    // x = hi | i << 8 | t (t the thread, i = 0..15 its slot).  A term's sign splits into a
    // per-chunk part on hi and a part on the 12 low bits, so per chunk the coefficient of
    // each low pattern p is C_p = sum_k c_k (-1)^{popcount(hi & z_k)} over the terms with
    // that pattern; a thread folds its own bits into E_r = sum over patterns with bits 8-11
    // equal to r of C_p (-1)^{popcount(t & p)}, and a 16-point Walsh-Hadamard transform
    // gives f(x) = sum_r E_r (-1)^{popcount(i & r)} for its 16 slots.  Each term costs a few
    // operations per chunk instead of per amplitude, which leaves the pass bound by HBM.
    // With the term table in LDS the per-chunk sums wait only on LDS, so the chunk's
    // amplitude loads, issued first, stay in flight meanwhile.
    __shared__ double cp[kPauliMaxPatterns];
    constexpr bool staged = (MODE & PG_STAGED) != 0, with_lam = (MODE & PG_LAM) != 0;
    const int P = A.n_pats;
    const int tid = threadIdx.x;
    const uint64_t* tz = A.zmasks;
    const double* tc = A.cre;
    if constexpr (staged) {
      __shared__ uint64_t sz[kPauliStageTerms];
      __shared__ double sc[kPauliStageTerms];
      for (int k = tid; k < A.n_terms; k += 256) {
        sz[k] = A.zmasks[k];
        sc[k] = A.cre[k];
      }
      tz = sz;
      tc = sc;
    }
    const uint64_t n_chunks = N >> 12;
    for (uint64_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
      const uint64_t hi = ch << 12;
      C v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = psi[hi | (uint64_t)(i << 8) | (uint64_t)tid];
      __syncthreads();  // the previous chunk's readers of cp are done (and the staging)
      for (int p = tid; p < P; p += 256) {
        const int k0 = (int)(A.pats[p] >> 12);
        const int k1 = p + 1 < P ? (int)(A.pats[p + 1] >> 12) : A.n_terms;
        double sr = 0.0;
        for (int k = k0; k < k1; ++k) {
          const bool neg = __popcll(hi & tz[k]) & 1;
          sr += neg ? -tc[k] : tc[k];
        }
        cp[p] = sr;
      }
      __syncthreads();
      double f[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        double a = 0.0;
        const int p0 = ld(A.rfirst + r), p1 = ld(A.rfirst + r + 1);
        for (int p = p0; p < p1; ++p) {
          const uint32_t pat = ld(A.pats + p) & 0xFFu;
          const bool neg = __popc((uint32_t)tid & pat) & 1;
          a += neg ? -cp[p] : cp[p];
        }
        f[r] = a;
      }
      // Walsh-Hadamard transform over the 4 slot bits
#pragma unroll
      for (int h = 1; h < 16; h <<= 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          if (r & h) continue;
          const double a = f[r], b = f[r | h];
          f[r] = a + b;
          f[r | h] = a - b;
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        er += ((double)v[i].x * v[i].x + (double)v[i].y * v[i].y) * f[i];
        if constexpr (with_lam) {
          const uint64_t x = hi | (uint64_t)(i << 8) | (uint64_t)tid;
          C o;
          o.x = (R)(f[i] * v[i].x);
          o.y = (R)(f[i] * v[i].y);
          if (A.accumulate) { const C l = lam[x]; o.x += l.x; o.y += l.y; }
          lam[x] = o;
        }
      }
    }
  } else if constexpr (MODE == PG_QUAD) {
    // Diagonal group, four consecutive amplitudes per thread: a term's sign parity on the
    // shared high bits is computed once; the two low bits flip it by the uniform pattern
    // pat(z) (bit j set when popcount(j & z) is odd).
    const bool real_c = A.real_coeffs;
    for (uint64_t q = (uint64_t)blockIdx.x * 256 + threadIdx.x; q < (N >> 2); q += stride) {
      const uint64_t x0 = q << 2;
      C v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = psi[x0 + j];
      double fr[4] = {0.0, 0.0, 0.0, 0.0}, fi[4] = {0.0, 0.0, 0.0, 0.0};
      for (int k = 0; k < A.n_terms; ++k) {
        const uint64_t z = ld(A.zmasks + k);
        const double cr = ld(A.cre + k);
        const uint32_t zl = (uint32_t)z & 3u;
        const uint32_t pat = (zl == 0u) ? 0u : (zl == 1u) ? 0xAu : (zl == 2u) ? 0xCu : 0x6u;
        const uint32_t par = (uint32_t)(__popcll(x0 & z) & 1) ? 0xFu : 0u;
        const uint32_t sg = par ^ pat;
#pragma unroll
        for (int j = 0; j < 4; ++j) fr[j] += ((sg >> j) & 1u) ? -cr : cr;
        if (!real_c) {
          const double ci = ld(A.cim + k);
#pragma unroll
          for (int j = 0; j < 4; ++j) fi[j] += ((sg >> j) & 1u) ? -ci : ci;
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double pj = (double)v[j].x * v[j].x + (double)v[j].y * v[j].y;
        er += pj * fr[j];
        ei += pj * fi[j];
        if (lam) {
          C o;
          o.x = (R)(fr[j] * v[j].x - fi[j] * v[j].y);
          o.y = (R)(fr[j] * v[j].y + fi[j] * v[j].x);
          if (A.accumulate) { const C l = lam[x0 + j]; o.x += l.x; o.y += l.y; }
          lam[x0 + j] = o;
        }
      }
    }
  } else if constexpr (MODE == PG_DIAG) {
    for (uint64_t x = (uint64_t)blockIdx.x * 256 + threadIdx.x; x < N; x += stride) {
      double fr, fi;
      group_factor<R>(A, x, fr, fi);
      const C v = psi[x];
      const double p = (double)v.x * v.x + (double)v.y * v.y;
      er += p * fr;
      ei += p * fi;
      if (lam) {
        C o;
        o.x = (R)(fr * v.x - fi * v.y);
        o.y = (R)(fr * v.y + fi * v.x);
        if (A.accumulate) { const C l = lam[x]; o.x += l.x; o.y += l.y; }
        lam[x] = o;
      }
    }
  } else {
    static_assert(MODE == PG_XMASK, "unknown Pauli pass mode");
    const int h = 63 - __clzll(A.xmask);
    const uint64_t lowm = (1ull << h) - 1;
    for (uint64_t p = (uint64_t)blockIdx.x * 256 + threadIdx.x; p < (N >> 1); p += stride) {
      const uint64_t x = ((p >> h) << (h + 1)) | (p & lowm);
      const uint64_t y = x ^ A.xmask;
      const C vx = psi[x], vy = psi[y];
      double fxr, fxi, fyr, fyi;
      group_factor<R>(A, x, fxr, fxi);
      group_factor<R>(A, y, fyr, fyi);
      // (H psi)[y] += f(x) psi[x];  (H psi)[x] += f(y) psi[y]
      const double axr = fxr * vx.x - fxi * vx.y, axi = fxr * vx.y + fxi * vx.x;
      const double ayr = fyr * vy.x - fyi * vy.y, ayi = fyr * vy.y + fyi * vy.x;
      // E += conj(vy) * a_x + conj(vx) * a_y
      er += (double)vy.x * axr + (double)vy.y * axi + (double)vx.x * ayr + (double)vx.y * ayi;
      ei += (double)vy.x * axi - (double)vy.y * axr + (double)vx.x * ayi - (double)vx.y * ayr;
      if (lam) {
        C oy, ox;
        oy.x = (R)axr; oy.y = (R)axi;
        ox.x = (R)ayr; ox.y = (R)ayi;
        if (A.accumulate) {
          const C ly = lam[y], lx = lam[x];
          oy.x += ly.x; oy.y += ly.y; ox.x += lx.x; ox.y += lx.y;
        }
        lam[y] = oy;
        lam[x] = ox;
      }
    }
  }
  er = wave_sum(er);
  ei = wave_sum(ei);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[0][w] = er; red[1][w] = ei; }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int64_t o = ((int64_t)blockIdx.y * A.ncols + A.col) * gridDim.x + blockIdx.x;
    A.partials[o] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    A.partials[o + gridDim.x] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
  }
}

// out[c] = sum_{i < len} in[c * len + i], fixed order.
__global__ __launch_bounds__(256) void reduce_columns(const double* in, int64_t len, double* out) {
  __shared__ double red[4];
  const double* col = in + (int64_t)blockIdx.x * len;
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < len; i += 256) s += col[i];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// psi_b = |index> for every batch item.
template <typename R>
__global__ __launch_bounds__(256) void set_basis(void* psi_, int64_t bstride, uint64_t N, uint64_t index) {
  using C = typename CT<R>::T;
  C* psi = reinterpret_cast<C*>(psi_) + (int64_t)blockIdx.y * bstride;
  // each workgroup writes one contiguous range
  const uint64_t per = (N + gridDim.x - 1) / gridDim.x;
  const uint64_t x0 = (uint64_t)blockIdx.x * per, x1 = x0 + per < N ? x0 + per : N;
  for (uint64_t x = x0 + threadIdx.x; x < x1; x += 256) {
    C v;
    v.x = (x == index) ? (R)1 : (R)0;
    v.y = (R)0;
    psi[x] = v;
  }
}

// dst_b = src (broadcast one state into batch items).
template <typename R>
__global__ __launch_bounds__(256) void broadcast_state(void* dst_, int64_t bstride, const void* src_, uint64_t N) {
  using C = typename CT<R>::T;
  C* dst = reinterpret_cast<C*>(dst_) + (int64_t)blockIdx.y * bstride;
  const C* src = reinterpret_cast<const C*>(src_);
  for (uint64_t x = (uint64_t)blockIdx.x * 256 + threadIdx.x; x < N; x += (uint64_t)gridDim.x * 256) dst[x] = src[x];
}

// ------------------------------------------------------------------------------------------
// Multi-circuit Pauli-sum pass in gather form: each thread owns output indices y and sums
// c_k P_k psi over all terms, (P_k psi)[y] = i^{popcount(x_k & z_k)} (-1)^{popcount((y ^ x_k) & z_k)}
// psi[y ^ x_k]; no two threads write the same lambda entry, so one launch covers every
// term.  Workgroup w handles chunk (w - prefix[i]) of job i (CHUNK amplitudes).
// A term's numbers and its load are two dependent round trips, which bound the pass: a thread
// takes NY outputs, 256 apart, through each term together, so that NY loads wait at once and
// the parity of the thread's own bits is formed once.  48 circuits of 8 to 20 qubits, complex64:
// 224 -> 93 us.  Circuits of less than 256 NY amplitudes take one output at a time.
// ------------------------------------------------------------------------------------------
template <int NY, typename C>
__device__ __forceinline__ void pauli_outputs(const PauliJob* J, const C* psi, C* lam, const uint64_t y0,
                                              double& er, double& ei) {
  const uint64_t* xm = ld(&J->xmasks);
  const uint64_t* zm = ld(&J->zmasks);
  const double* cre = ld(&J->cre);
  const double* cim = ld(&J->cim);
  const int nt = ld(&J->n_terms);
  double lr[NY] = {}, li[NY] = {};
  for (int k = 0; k < nt; ++k) {
    const uint64_t x0 = y0 ^ ld(xm + k), z = ld(zm + k);
    C v[NY];
#pragma unroll
    for (int j = 0; j < NY; ++j) v[j] = psi[x0 ^ ((uint64_t)j << 8)];
    const double sgn = (__popcll(x0 & z) & 1) ? -1.0 : 1.0;
    const double ar0 = sgn * ld(cre + k), ai0 = sgn * ld(cim + k);
#pragma unroll
    for (int j = 0; j < NY; ++j) {
      const bool neg = __popcll(z & ((uint64_t)j << 8)) & 1;  // wave-uniform
      const double ar = neg ? -ar0 : ar0, ai = neg ? -ai0 : ai0;
      lr[j] += ar * v[j].x - ai * v[j].y;
      li[j] += ar * v[j].y + ai * v[j].x;
    }
  }
#pragma unroll
  for (int j = 0; j < NY; ++j) {
    const uint64_t y = y0 ^ ((uint64_t)j << 8);
    const C py = psi[y];
    er += (double)py.x * lr[j] + (double)py.y * li[j];
    ei += (double)py.x * li[j] - (double)py.y * lr[j];
    C o;
    o.x = (decltype(o.x))lr[j];
    o.y = (decltype(o.y))li[j];
    lam[y] = o;
  }
}

template <typename R, int CHUNK>
__global__ __launch_bounds__(256) void pauli_apply_multi(const PauliJob* jobs, const uint32_t* prefix, int n_jobs) {
  using C = typename CT<R>::T;
  constexpr int NY = 8;
  static_assert(CHUNK % (256 * NY) == 0, "a chunk is whole groups of NY outputs per thread");
  __shared__ double red[2][4];
  const uint32_t w = blockIdx.x;
  int lo = 0, hi = n_jobs;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (ld(prefix + mid) <= w) lo = mid; else hi = mid;
  }
  const PauliJob* J = jobs + lo;
  const uint32_t chunk = w - ld(prefix + lo);
  const C* psi = reinterpret_cast<const C*>(ld(&J->psi));
  C* lam = reinterpret_cast<C*>(ld(&J->lam));
  const uint64_t N = 1ull << ld(&J->n_qubits);
  const uint64_t first = (uint64_t)chunk * CHUNK;
  const uint64_t last = first + CHUNK < N ? first + CHUNK : N;
  double er = 0.0, ei = 0.0;
  if (N >= 256 * NY) {  // then last - first is a multiple of 256 NY
    for (uint64_t y = first + threadIdx.x; y < last; y += 256 * NY) pauli_outputs<NY>(J, psi, lam, y, er, ei);
  } else {
    for (uint64_t y = first + threadIdx.x; y < last; y += 256) pauli_outputs<1>(J, psi, lam, y, er, ei);
  }
  er = wave_sum(er);
  ei = wave_sum(ei);
  if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = er; red[1][threadIdx.x >> 6] = ei; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double* P = ld(&J->partials);
    P[2 * chunk] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    P[2 * chunk + 1] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
  }
}

// out[c] = sum of in[offs[c] + stride[c] * i] for i < lens[c], fixed order.
__global__ __launch_bounds__(256) void reduce_segments(const double* in, const int64_t* offs, const int32_t* lens,
                                                       const int32_t* strides, double* out) {
  __shared__ double red[4];
  const int c = blockIdx.x;
  const int64_t o = ld(offs + c);
  const int32_t len = ld(lens + c), st = ld(strides + c);
  double s = 0.0;
  for (int32_t i = threadIdx.x; i < len; i += 256) s += in[o + (int64_t)st * i];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) out[c] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Fill states with |0...0>: job j covers 2^n[j] amplitudes at ptr[j] in CHUNK-sized pieces.
template <typename R>
__global__ __launch_bounds__(256) void set_zero_multi(void* const* ptrs, const int32_t* nq, const uint32_t* prefix,
                                                      int n_jobs) {
  using C = typename CT<R>::T;
  const uint32_t w = blockIdx.x;
  int lo = 0, hi = n_jobs;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (ld(prefix + mid) <= w) lo = mid; else hi = mid;
  }
  C* psi = reinterpret_cast<C*>(ld(ptrs + lo));
  const uint64_t N = 1ull << ld(nq + lo);
  const uint64_t chunk = w - ld(prefix + lo);
  for (uint64_t x = chunk * 4096 + threadIdx.x; x < N && x < (chunk + 1) * 4096; x += 256) {
    C v;
    v.x = x == 0 ? (R)1 : (R)0;
    v.y = (R)0;
    psi[x] = v;
  }
}

// dst = alpha * src (complex alpha), one state.
template <typename R>
__global__ __launch_bounds__(256) void scale_copy(void* dst_, const void* src_, uint64_t N, double ar, double ai) {
  using C = typename CT<R>::T;
  C* dst = reinterpret_cast<C*>(dst_);
  const C* src = reinterpret_cast<const C*>(src_);
  for (uint64_t x = (uint64_t)blockIdx.x * 256 + threadIdx.x; x < N; x += (uint64_t)gridDim.x * 256) {
    const C v = src[x];
    C o;
    o.x = (R)(ar * v.x - ai * v.y);
    o.y = (R)(ar * v.y + ai * v.x);
    dst[x] = o;
  }
}

// partials[blk] = sum conj(a[x]) b[x] (re at 2 blk, im at 2 blk + 1), fp64.
template <typename R>
__global__ __launch_bounds__(256) void inner_product(const void* a_, const void* b_, uint64_t N, double* partials) {
  using C = typename CT<R>::T;
  __shared__ double red[2][4];
  const C* a = reinterpret_cast<const C*>(a_);
  const C* b = reinterpret_cast<const C*>(b_);
  double re = 0.0, im = 0.0;
  for (uint64_t x = (uint64_t)blockIdx.x * 256 + threadIdx.x; x < N; x += (uint64_t)gridDim.x * 256) {
    const C u = a[x], v = b[x];
    re += (double)u.x * v.x + (double)u.y * v.y;
    im += (double)u.x * v.y - (double)u.y * v.x;
  }
  re = wave_sum(re);
  im = wave_sum(im);
  if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = re; red[1][threadIdx.x >> 6] = im; }
  __syncthreads();
  if (threadIdx.x == 0) {
    partials[blockIdx.x] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    partials[gridDim.x + blockIdx.x] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
  }
}

// ------------------------------------------------------------------------------------------
// Host launchers.
// ------------------------------------------------------------------------------------------
static inline unsigned stream_blocks(uint64_t work) {
  const uint64_t b = (work + 255) / 256;
  return (unsigned)(b < 4096 ? (b ? b : 1) : 4096);
}

// Register-blocked passes of one amplitude type and direction (instantiated by tile_rb.hip).
template <typename R, bool ADJ>
hipError_t rb_dispatch(int reg_bits, int maxm, const PassArgs& A, uint64_t n_tiles, int batch, hipStream_t s);
template <typename R, bool ADJ>
hipError_t rb_multi_dispatch(int maxm, const PassArgs* items, const uint32_t* prefix, int n_items, uint32_t n_wg,
                             int max_win, int max_pslots, hipStream_t s);

hipError_t launch_tile_pass_rb_multi(int dtype, bool adj, int maxm, const PassArgs* items, const uint32_t* prefix,
                                     int n_items, uint32_t n_wg, int max_win, int max_pslots, hipStream_t s) {
  if (max_win > kMaxWindow) return hipErrorInvalidValue;
  if (dtype == 0)
    return adj ? rb_multi_dispatch<float, true>(maxm, items, prefix, n_items, n_wg, max_win, max_pslots, s)
               : rb_multi_dispatch<float, false>(maxm, items, prefix, n_items, n_wg, max_win, max_pslots, s);
  return adj ? rb_multi_dispatch<double, true>(maxm, items, prefix, n_items, n_wg, max_win, max_pslots, s)
             : rb_multi_dispatch<double, false>(maxm, items, prefix, n_items, n_wg, max_win, max_pslots, s);
}

hipError_t launch_pauli_apply_multi(int dtype, const PauliJob* jobs, const uint32_t* prefix, int n_jobs, uint32_t n_wg,
                                    hipStream_t s) {
  if (dtype == 0) pauli_apply_multi<float, kPauliChunk><<<n_wg, 256, 0, s>>>(jobs, prefix, n_jobs);
  else pauli_apply_multi<double, kPauliChunk><<<n_wg, 256, 0, s>>>(jobs, prefix, n_jobs);
  return hipGetLastError();
}

hipError_t launch_reduce_segments(const double* in, const int64_t* offs, const int32_t* lens, const int32_t* strides,
                                  double* out, int ncols, hipStream_t s) {
  if (ncols <= 0) return hipSuccess;
  reduce_segments<<<(unsigned)ncols, 256, 0, s>>>(in, offs, lens, strides, out);
  return hipGetLastError();
}

hipError_t launch_set_zero_multi(int dtype, void* const* ptrs, const int32_t* nq, const uint32_t* prefix, int n_jobs,
                                 uint32_t n_wg, hipStream_t s) {
  if (dtype == 0) set_zero_multi<float><<<n_wg, 256, 0, s>>>(ptrs, nq, prefix, n_jobs);
  else set_zero_multi<double><<<n_wg, 256, 0, s>>>(ptrs, nq, prefix, n_jobs);
  return hipGetLastError();
}

hipError_t launch_scale_copy(int dtype, void* dst, const void* src, int n, double ar, double ai, hipStream_t s) {
  const unsigned grid = stream_blocks(1ull << n);
  if (dtype == 0) scale_copy<float><<<grid, 256, 0, s>>>(dst, src, 1ull << n, ar, ai);
  else scale_copy<double><<<grid, 256, 0, s>>>(dst, src, 1ull << n, ar, ai);
  return hipGetLastError();
}

unsigned inner_blocks(int n) {
  const unsigned b = stream_blocks(1ull << n);
  return b < 1024 ? b : 1024;
}

hipError_t launch_inner_product(int dtype, const void* a, const void* b, int n, double* partials, hipStream_t s) {
  const unsigned grid = inner_blocks(n);
  if (dtype == 0) inner_product<float><<<grid, 256, 0, s>>>(a, b, 1ull << n, partials);
  else inner_product<double><<<grid, 256, 0, s>>>(a, b, 1ull << n, partials);
  return hipGetLastError();
}

hipError_t launch_tile_pass_rb(int dtype, bool adj, int reg_bits, int maxm, const PassArgs& A, uint64_t n_tiles,
                               int batch, hipStream_t s) {
  if (A.m != maxm) return hipErrorInvalidValue;  // the kernel assumes a full workgroup
  if (A.win_n > kMaxWindow) return hipErrorInvalidValue;
  if (dtype == 0) return adj ? rb_dispatch<float, true>(reg_bits, maxm, A, n_tiles, batch, s)
                             : rb_dispatch<float, false>(reg_bits, maxm, A, n_tiles, batch, s);
  return adj ? rb_dispatch<double, true>(reg_bits, maxm, A, n_tiles, batch, s)
             : rb_dispatch<double, false>(reg_bits, maxm, A, n_tiles, batch, s);
}

hipError_t launch_gate1(int dtype, void* psi, int64_t bstride, int batch, int n, int t, uint64_t cmask,
                        const void* ctab, int64_t ctab_bstride, int mat, hipStream_t s) {
  const dim3 grid(stream_blocks(1ull << (n - 1)), (unsigned)batch);
  if (dtype == 0) gate1_stream<float><<<grid, 256, 0, s>>>(psi, bstride, n, t, cmask, ctab, ctab_bstride, mat);
  else gate1_stream<double><<<grid, 256, 0, s>>>(psi, bstride, n, t, cmask, ctab, ctab_bstride, mat);
  return hipGetLastError();
}

hipError_t launch_gate2(int dtype, void* psi, int64_t bstride, int batch, int n, int ta, int tb,
                        uint64_t cmask, const void* ctab, int64_t ctab_bstride, int mat, hipStream_t s) {
  const dim3 grid(stream_blocks(1ull << (n - 2)), (unsigned)batch);
  if (dtype == 0) gate2_stream<float><<<grid, 256, 0, s>>>(psi, bstride, n, ta, tb, cmask, ctab, ctab_bstride, mat);
  else gate2_stream<double><<<grid, 256, 0, s>>>(psi, bstride, n, ta, tb, cmask, ctab, ctab_bstride, mat);
  return hipGetLastError();
}

hipError_t launch_diag(int dtype, void* psi, int64_t bstride, int batch, int n, const DiagEntry* diag,
                       int first, int count, const void* ctab, int64_t ctab_bstride, hipStream_t s) {
  const dim3 grid(stream_blocks(1ull << n), (unsigned)batch);
  if (dtype == 0) diag_stream<float><<<grid, 256, 0, s>>>(psi, bstride, n, diag, first, count, ctab, ctab_bstride);
  else diag_stream<double><<<grid, 256, 0, s>>>(psi, bstride, n, diag, first, count, ctab, ctab_bstride);
  return hipGetLastError();
}

unsigned pauli_blocks(int n) {
  const uint64_t work = 1ull << (n > 0 ? n - 1 : 0);
  return stream_blocks(work) < 2048 ? stream_blocks(work) : 2048;
}

template <typename R>
void launch_pauli_mode(const PauliGroupArgs& A, dim3 grid, hipStream_t s) {
  if (A.xmask != 0) {
    pauli_group<R, PG_XMASK><<<grid, 256, 0, s>>>(A);
  } else if (A.n_pats > 0 && A.real_coeffs) {
    const int m = (A.n_terms <= kPauliStageTerms ? PG_STAGED : 0) | (A.lam ? PG_LAM : 0);
    switch (m) {
      case 0: pauli_group<R, 0><<<grid, 256, 0, s>>>(A); break;
      case 1: pauli_group<R, 1><<<grid, 256, 0, s>>>(A); break;
      case 2: pauli_group<R, 2><<<grid, 256, 0, s>>>(A); break;
      default: pauli_group<R, 3><<<grid, 256, 0, s>>>(A); break;
    }
  } else if (A.n_qubits >= 2) pauli_group<R, PG_QUAD><<<grid, 256, 0, s>>>(A);
  else pauli_group<R, PG_DIAG><<<grid, 256, 0, s>>>(A);
}

hipError_t launch_pauli_group(int dtype, const PauliGroupArgs& A, unsigned blocks, int batch, hipStream_t s) {
  const dim3 grid(blocks, (unsigned)batch);
  if (dtype == 0) launch_pauli_mode<float>(A, grid, s);
  else launch_pauli_mode<double>(A, grid, s);
  return hipGetLastError();
}

hipError_t launch_reduce_columns(const double* in, int64_t len, int64_t ncols, double* out, hipStream_t s) {
  if (ncols <= 0) return hipSuccess;
  reduce_columns<<<(unsigned)ncols, 256, 0, s>>>(in, len, out);
  return hipGetLastError();
}

hipError_t launch_set_basis(int dtype, void* psi, int64_t bstride, int batch, int n, uint64_t index, hipStream_t s) {
  const dim3 grid(stream_blocks(1ull << n), (unsigned)batch);
  if (dtype == 0) set_basis<float><<<grid, 256, 0, s>>>(psi, bstride, 1ull << n, index);
  else set_basis<double><<<grid, 256, 0, s>>>(psi, bstride, 1ull << n, index);
  return hipGetLastError();
}

hipError_t launch_broadcast_state(int dtype, void* dst, int64_t bstride, int batch, const void* src, int n,
                                  hipStream_t s) {
  const dim3 grid(stream_blocks(1ull << n), (unsigned)batch);
  if (dtype == 0) broadcast_state<float><<<grid, 256, 0, s>>>(dst, bstride, src, 1ull << n);
  else broadcast_state<double><<<grid, 256, 0, s>>>(dst, bstride, src, 1ull << n);
  return hipGetLastError();
}

}  // namespace qsv
