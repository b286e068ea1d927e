// Fused tile pass with the tile in LDS (tiles below the register-blocked range):
//  tile_pass      a workgroup stages a 2^m-amplitude tile (the sub-cube spanned by the pass's
//                 tile qubits) into LDS, applies the pass's op list there, and writes it back.
//                 The adjoint variant stages psi and lambda together, applies U^dag to both and
//                 accumulates Im<lambda|G|psi> per gradient slot in fp64.
#include "device_util.h"
#include "qsv_kernels.h"

namespace qsv {

// ------------------------------------------------------------------------------------------
// Fused tile pass.
// ------------------------------------------------------------------------------------------
template <typename R, int NT, int MAXM, bool ADJ>
__global__ __launch_bounds__(NT) void tile_pass(PassArgs A) {
  using C = typename CT<R>::T;
  constexpr int LGNT = (NT == 1024) ? 10 : (NT == 512) ? 9 : 8;
  constexpr int RA = ((1 << MAXM) + NT - 1) / NT;        // amplitude slots per thread (max)
  constexpr int PP = ((1 << MAXM) / 2 + NT - 1) / NT;    // pairs per thread per 1-qubit op (max)
  constexpr int QP = ((1 << MAXM) / 4 + NT - 1) / NT;    // quads per thread per 2-qubit op (max)
  __shared__ C sp[1 << MAXM];
  __shared__ C sl[ADJ ? (1 << MAXM) : 1];
  __shared__ double red[NT / 64];

  const int tid = threadIdx.x;
  const int m = A.m;
  const int nloc = 1 << m;
  const int half = nloc >> 1, quarter = nloc >> 2;
  const bool active = tid < nloc;
  const uint64_t tile = blockIdx.x;
  const int b = blockIdx.y;
  const uint64_t full = (A.n_qubits >= 64) ? ~0ull : ((1ull << A.n_qubits) - 1);
  const uint64_t base = pdep64(tile, full & ~A.tile_mask);
  const uint64_t s_tid = pdep64((uint64_t)tid, A.tile_mask);
  uint64_t hmask = A.tile_mask;               // tile bits above the thread bits
  for (int i = 0; i < LGNT; ++i) hmask &= hmask - 1;
  uint64_t xk[RA];                            // global index of each amplitude slot
#pragma unroll
  for (int k = 0; k < RA; ++k) xk[k] = base | s_tid | pdep64((uint64_t)k, hmask);

  C* psi = reinterpret_cast<C*>(A.psi) + (int64_t)b * A.bstride;
  C* lam = ADJ ? reinterpret_cast<C*>(A.lam) + (int64_t)b * A.bstride : nullptr;
  const C* src = A.src ? reinterpret_cast<const C*>(A.src) + (int64_t)b * A.src_bstride : psi;
  const C* T = reinterpret_cast<const C*>(A.ctab) + (int64_t)b * A.ctab_bstride;

  if (active) {
#pragma unroll
    for (int k = 0; k < RA; ++k) {
      const int j = tid + k * NT;
      if (j < nloc) {
        sp[j] = src[xk[k]];
        if (ADJ) sl[j] = lam[xk[k]];
      }
    }
  }
  __syncthreads();

  double acc = 0.0;
  for (int oi = 0; oi < A.n_ops; ++oi) {
    const TileOp* O = A.ops + oi;
    const int type = ld(&O->type);
    const uint64_t omask = ld(&O->omask);
    const bool on = (base & omask) == omask;
    if (on && type == OP_DENSE1) {
      const int mat = ld(&O->mat), gen = ld(&O->gen);
      const C u00 = ldc(T + mat), u01 = ldc(T + mat + 1), u10 = ldc(T + mat + 2), u11 = ldc(T + mat + 3);
      C g00, g01, g10, g11;
      const bool grad = ADJ && gen >= 0;
      if (grad) { g00 = ldc(T + gen); g01 = ldc(T + gen + 1); g10 = ldc(T + gen + 2); g11 = ldc(T + gen + 3); }
      const int a = ld(&O->a);
      const int amask = (1 << a) - 1;
      const uint32_t lm = ld(&O->lmask);
      int j0[PP];
      bool ok[PP];
      C v0[PP], v1[PP], w0[PP], w1[PP];
#pragma unroll
      for (int i = 0; i < PP; ++i) {
        const int p = tid + i * NT;
        j0[i] = ((p >> a) << (a + 1)) | (p & amask);
        ok[i] = p < half && (((uint32_t)j0[i] & lm) == lm);
        if (ok[i]) {
          v0[i] = sp[j0[i]];
          v1[i] = sp[j0[i] | (1 << a)];
          if (ADJ) { w0[i] = sl[j0[i]]; w1[i] = sl[j0[i] | (1 << a)]; }
        }
      }
#pragma unroll
      for (int i = 0; i < PP; ++i) {
        if (!ok[i]) continue;
        if (ADJ) {
          if (grad)
            acc += im_conj_mul(w0[i], cdot2(g00, v0[i], g01, v1[i])) + im_conj_mul(w1[i], cdot2(g10, v0[i], g11, v1[i]));
          sl[j0[i]] = cdot2(u00, w0[i], u01, w1[i]);
          sl[j0[i] | (1 << a)] = cdot2(u10, w0[i], u11, w1[i]);
        }
        sp[j0[i]] = cdot2(u00, v0[i], u01, v1[i]);
        sp[j0[i] | (1 << a)] = cdot2(u10, v0[i], u11, v1[i]);
      }
    } else if (on && type == OP_DENSE2) {
      const int a = ld(&O->a), bb = ld(&O->b);
      const int mat = ld(&O->mat), gen = ld(&O->gen);
      const int lo = a < bb ? a : bb, hi = a < bb ? bb : a;
      const uint32_t lm = ld(&O->lmask);
      const bool grad = ADJ && gen >= 0;
      C U[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) U[r] = ldc(T + mat + r);
#pragma unroll
      for (int i = 0; i < QP; ++i) {
        const int p = tid + i * NT;
        if (p >= quarter) continue;
        int t = ((p >> lo) << (lo + 1)) | (p & ((1 << lo) - 1));
        t = ((t >> hi) << (hi + 1)) | (t & ((1 << hi) - 1));
        if (((uint32_t)t & lm) != lm) continue;
        const int idx[4] = {t, t | (1 << a), t | (1 << bb), t | (1 << a) | (1 << bb)};
        C v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = sp[idx[r]];
        if (ADJ) {
          C w[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) w[r] = sl[idx[r]];
          if (grad) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              C gsum = cdot2(ldc(T + gen + 4 * r), v[0], ldc(T + gen + 4 * r + 1), v[1]);
              gsum = cdot2(C{1, 0}, gsum, ldc(T + gen + 4 * r + 2), v[2]);
              gsum = cdot2(C{1, 0}, gsum, ldc(T + gen + 4 * r + 3), v[3]);
              acc += im_conj_mul(w[r], gsum);
            }
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            C q = cdot2(U[4 * r], w[0], U[4 * r + 1], w[1]);
            q = cdot2(C{1, 0}, q, U[4 * r + 2], w[2]);
            q = cdot2(C{1, 0}, q, U[4 * r + 3], w[3]);
            sl[idx[r]] = q;
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          C o = cdot2(U[4 * r], v[0], U[4 * r + 1], v[1]);
          o = cdot2(C{1, 0}, o, U[4 * r + 2], v[2]);
          o = cdot2(C{1, 0}, o, U[4 * r + 3], v[3]);
          sp[idx[r]] = o;
        }
      }
    } else if (on && type == OP_DIAG) {
      const int first = ld(&O->first), count = ld(&O->count);
      if (active) {
        C v[RA], w[RA];
#pragma unroll
        for (int k = 0; k < RA; ++k) {
          const int j = tid + k * NT;
          if (j < nloc) { v[k] = sp[j]; if (ADJ) w[k] = sl[j]; }
        }
#pragma unroll
        for (int k = 0; k < RA; ++k) {
          const int j = tid + k * NT;
          if (j >= nloc) continue;
          const uint64_t x = xk[k];
          C ph = C{1, 0};
          int sign = 0;
          double gw = 0.0;
          for (int e = 0; e < count; ++e) {
            const DiagEntry* d = A.diag + first + e;
            const uint64_t cm = ld(&d->cmask);
            if (ld(&d->kind) == DIAG_SIGN) {
              sign ^= (int)((x & cm) == cm);
            } else if ((x & cm) == cm) {
              const int q1 = ld(&d->q1);
              const int idx = (int)((x >> ld(&d->q0)) & 1) | (q1 >= 0 ? (int)((x >> q1) & 1) << 1 : 0);
              ph = cmul(ph, ldc(T + ld(&d->mat) + idx));
              if (ADJ) {
                const int dg = ld(&d->gen);
                if (dg >= 0) gw += (double)ldc(T + dg + idx).x;
              }
            }
          }
          if (sign) { ph.x = -ph.x; ph.y = -ph.y; }
          sp[j] = cmul(v[k], ph);
          if (ADJ) {
            acc += gw * im_conj_mul(w[k], v[k]);
            sl[j] = cmul(w[k], ph);
          }
        }
      }
    } else if (on && type == OP_ZZ) {
      const int first = ld(&O->first), count = ld(&O->count), mat = ld(&O->mat), gen = ld(&O->gen);
      if (active) {
        const ZZEdge* ed = A.edges + first;
        C v[RA], w[RA];
#pragma unroll
        for (int k = 0; k < RA; ++k) {
          const int j = tid + k * NT;
          if (j < nloc) { v[k] = sp[j]; if (ADJ) w[k] = sl[j]; }
        }
        int cnt[RA];
#pragma unroll
        for (int k = 0; k < RA; ++k) cnt[k] = 0;
        for (int e = 0; e < count; ++e) {
          const int u = ld(&ed[e].u), vv = ld(&ed[e].v);
#pragma unroll
          for (int k = 0; k < RA; ++k) cnt[k] += (int)(((xk[k] >> u) ^ (xk[k] >> vv)) & 1);
        }
#pragma unroll
        for (int k = 0; k < RA; ++k) {
          const int j = tid + k * NT;
          if (j >= nloc) continue;
          const C ph = ldc(T + mat + cnt[k]);
          sp[j] = cmul(v[k], ph);
          if (ADJ) {
            if (gen >= 0) acc += (double)ldc(T + gen + cnt[k]).x * im_conj_mul(w[k], v[k]);
            sl[j] = cmul(w[k], ph);
          }
        }
      }
    }
    if (ADJ && ld(&O->flush)) {
      const double v = wave_sum(acc);
      if ((tid & 63) == 0) red[tid >> 6] = v;
      __syncthreads();
      if (tid == 0) {
        double s = 0.0;
        for (int w = 0; w < NT / 64; ++w) s += red[w];
        A.partials[((int64_t)b * A.n_pslots + ld(&O->pslot)) * (int64_t)gridDim.x + (int64_t)tile] = s;
      }
      acc = 0.0;
    }
    __syncthreads();
  }

  if (active) {
#pragma unroll
    for (int k = 0; k < RA; ++k) {
      const int j = tid + k * NT;
      if (j < nloc) {
        psi[xk[k]] = sp[j];
        if (ADJ) lam[xk[k]] = sl[j];
      }
    }
  }
}

template <typename R, int NT, int MAXM, bool ADJ>
static hipError_t tile_launch_one(const PassArgs& A, dim3 grid, hipStream_t s) {
  constexpr size_t bytes = (size_t)(2 * sizeof(R)) * ((size_t)1 << MAXM) * (ADJ ? 2 : 1);
  if constexpr (bytes <= 131072) {
    tile_pass<R, NT, MAXM, ADJ><<<grid, NT, 0, s>>>(A);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

template <typename R, bool ADJ>
static hipError_t tile_dispatch(int maxm, const PassArgs& A, uint64_t n_tiles, int batch, hipStream_t s) {
  const dim3 grid((unsigned)n_tiles, (unsigned)batch);
  switch (maxm) {
    case 8:  return tile_launch_one<R, 256, 8, ADJ>(A, grid, s);
    case 10: return tile_launch_one<R, 512, 10, ADJ>(A, grid, s);
    case 11: return tile_launch_one<R, 512, 11, ADJ>(A, grid, s);
    case 12: return tile_launch_one<R, 512, 12, ADJ>(A, grid, s);
    case 13: return tile_launch_one<R, 1024, 13, ADJ>(A, grid, s);
    case 14: return tile_launch_one<R, 1024, 14, ADJ>(A, grid, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_tile_pass(int dtype, bool adj, int maxm, const PassArgs& A, uint64_t n_tiles,
                            int batch, hipStream_t s) {
  if (dtype == 0) return adj ? tile_dispatch<float, true>(maxm, A, n_tiles, batch, s)
                             : tile_dispatch<float, false>(maxm, A, n_tiles, batch, s);
  return adj ? tile_dispatch<double, true>(maxm, A, n_tiles, batch, s)
             : tile_dispatch<double, false>(maxm, A, n_tiles, batch, s);
}

}  // namespace qsv
