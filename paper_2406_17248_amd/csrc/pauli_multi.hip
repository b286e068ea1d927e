// Pauli sums with several x masks in one pass.
//
// Terms that share an x mask form a group; a group's share of lambda = H psi at index y is
// f(y) psi[y ^ x], f(y) = sum over its terms of c (-1)^{popcount(y & z)} (the sign that z
// takes on x is folded into c).  One pass per group reads psi, and reads and writes lambda,
// once per group; here a thread keeps lambda for its outputs and walks many groups.
//
//  pauli_tile    psi goes through LDS one tile at a time (the sub-cube of 2^M amplitudes over
//                the launch's tile qubits, low qubits among them), for the groups whose x mask
//                lies inside the tile qubits: HBM sees psi once per launch, not per group.
//                Bound by HBM and the vector ALU about equally.  26-qubit Heisenberg chain with
//                a field, complex128, 25 x masks: one pass per group 4851 us, now 1181 us.
//  pauli_gather  psi[y ^ x] is read from global memory, lambda's partial sums are rounded to
//                the amplitude type group after group, as the passes per group do.  For states
//                that caches hold: bound by launches and latency (50 random terms on 11
//                qubits, 36 launches: 181 -> 31 us), then by the caches (24 qubits,
//                complex64, H psi 2179 -> 464 us with tiles).
#include "device_util.h"
#include "qsv_kernels.h"

namespace qsv {

__device__ __forceinline__ double flip_if(double v, uint32_t sign) {  // sign: 0 or 0x80000000
  return __longlong_as_double(__double_as_longlong(v) ^ (long long)((uint64_t)sign << 32));
}

// f[k] for the NO outputs of a thread over `count` terms: `t` is the thread's part of the
// output index, `hi` its wave-uniform part, k the output's slot.
template <int NO>
__device__ __forceinline__ void pauli_factor(const PauliMultiTerm* T, int count, uint32_t t, uint64_t hi, double* f) {
  for (int e = 0; e < count; ++e) {
    const PauliMultiTerm M = ld_record(T + e);
    const uint32_t s = (uint32_t)(__popc(t & M.zt) + __popcll(hi & M.zo)) << 31;
    const double c = flip_if(M.c, s);
#pragma unroll
    for (int k = 0; k < NO; ++k) {
      const uint32_t sk = (uint32_t)(__builtin_popcount((uint32_t)k & M.pat) & 1) << 31;  // wave-uniform
      f[k] = e == 0 ? flip_if(c, sk) : f[k] + flip_if(c, sk);
    }
  }
}

__device__ __forceinline__ void pauli_partials(double er, double ei, const PauliMultiArgs& A) {
  __shared__ double red[2][8];
  er = wave_sum(er);
  ei = wave_sum(ei);
  const int w = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6);
  if ((threadIdx.x & 63) == 0) { red[0][w] = er; red[1][w] = ei; }
  __syncthreads();
  if (threadIdx.x < 2) {
    double s = 0.0;
    for (int i = 0; i < nw; ++i) s += red[threadIdx.x][i];
    A.partials[((int64_t)blockIdx.y * A.ncols + A.col + threadIdx.x) * gridDim.x + blockIdx.x] = s;
  }
}

// NO outputs per thread: y = y0 + k N / NO.  Four groups at a time, so that their reads of psi
// are in flight together.  Without lambda the groups may be split over `splits` workgroups
// per chunk of outputs (small states: more workgroups than chunks).
template <typename R, int NO, bool LAM>
__global__ __launch_bounds__(256) void pauli_gather(PauliMultiArgs A) {
  using C = typename CT<R>::T;
  const C* psi = reinterpret_cast<const C*>(A.psi) + (int64_t)blockIdx.y * A.bstride;
  C* lam = LAM ? reinterpret_cast<C*>(A.lam) + (int64_t)blockIdx.y * A.bstride : nullptr;
  const uint64_t part = (1ull << A.n_qubits) / NO;  // outputs per slot
  const uint32_t blocks = gridDim.x / A.splits, split = blockIdx.x / blocks, bx = blockIdx.x % blocks;
  const int g0 = (int)((int64_t)A.n_groups * split / A.splits);
  const int g1 = (int)((int64_t)A.n_groups * (split + 1) / A.splits);
  // Workgroups go to the 8 XCDs in turn: each XCD takes one contiguous range of outputs, so
  // partners that differ in low bits come from the same L2.
  const uint64_t chunks = (part + 255) / 256;
  const bool xcd = chunks % 8 == 0 && blocks % 8 == 0 && chunks >= blocks;
  const uint64_t c_end = xcd ? ((bx & 7) + 1) * (chunks / 8) : chunks;
  double er = 0.0, ei = 0.0;
  for (uint64_t c = xcd ? (bx & 7) * (chunks / 8) + (bx >> 3) : bx; c < c_end; c += xcd ? blocks / 8 : blocks) {
    const uint64_t y0 = c * 256 + threadIdx.x;
    const uint64_t yw = c * 256 + (uint64_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~63u));  // the wave's bits
    if (y0 < part) {
      double ar[NO], ai[NO];  // lambda in double (for the energy)
      C l[NO];                // lambda rounded group after group
#pragma unroll
      for (int k = 0; k < NO; ++k) {
        ar[k] = ai[k] = 0.0;
        l[k] = C{0, 0};
        if (LAM && A.accumulate) l[k] = lam[y0 + k * part];
      }
      for (int g = g0; g < g1; g += 4) {
        C v[4][NO];
        PauliMultiGroup G[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          G[i] = ld_record(A.groups + (g + i < g1 ? g + i : g1 - 1));
          if (g + i >= g1) G[i].n_re = G[i].n_im = 0;
#pragma unroll
          for (int k = 0; k < NO; ++k) {
            // (left out: the output's own amplitude, read anyway, in place of its partner)
            const uint64_t x = !LAM && ((yw + k * part) & G[i].half) ? 0 : G[i].x;
            v[i][k] = psi[(y0 + k * part) ^ x];
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (G[i].n_re + G[i].n_im == 0 || (!LAM && (yw & G[i].half))) continue;
          double fr[NO], fi[NO];
#pragma unroll
          for (int k = 0; k < NO; ++k) fr[k] = fi[k] = 0.0;
          const PauliMultiTerm* T = A.terms + G[i].first;
          pauli_factor<NO>(T, G[i].n_re, (uint32_t)y0, 0, fr);
          pauli_factor<NO>(T + G[i].n_re, G[i].n_im, (uint32_t)y0, 0, fi);
#pragma unroll
          for (int k = 0; k < NO; ++k) {
            if (!LAM && ((k * part) & G[i].half)) continue;
            const double vx = v[i][k].x, vy = v[i][k].y;
            const double br = fr[k] * vx - fi[k] * vy, bi = fr[k] * vy + fi[k] * vx;
            ar[k] += br;
            ai[k] += bi;
            if (LAM) {
              l[k].x += (R)br;
              l[k].y += (R)bi;
            }
          }
        }
      }
#pragma unroll
      for (int k = 0; k < NO; ++k) {
        const C p = psi[y0 + k * part];
        er += (double)p.x * ar[k] + (double)p.y * ai[k];
        if (LAM) {
          ei += (double)p.x * ai[k] - (double)p.y * ar[k];
          lam[y0 + k * part] = l[k];
        }
      }
    }
  }
  pauli_partials(er, ei, A);
}

// 2^M amplitudes of psi in LDS, NR = 2^M / NT outputs per thread (slot k: local index tid +
// k NT).
template <typename R, int M, int NT, bool LAM>
__global__ __launch_bounds__(NT) void pauli_tile(PauliMultiArgs A) {
  using C = typename CT<R>::T;
  constexpr int NR = (1 << M) / NT, LT = NT == 512 ? 9 : 8;
  static_assert(1 << LT == NT, "threads per workgroup");
  __shared__ C buf[1 << M];
  const int tid = threadIdx.x;
  const C* psi = reinterpret_cast<const C*>(A.psi) + (int64_t)blockIdx.y * A.bstride;
  C* lam = LAM ? reinterpret_cast<C*>(A.lam) + (int64_t)blockIdx.y * A.bstride : nullptr;
  const uint64_t T = A.tile, full = A.n_qubits >= 64 ? ~0ull : (1ull << A.n_qubits) - 1;
  uint64_t th = T;  // tile qubits on slot bits
  for (int i = 0; i < LT; ++i) th &= th - 1;
  const uint64_t xt = pdep64((uint64_t)tid, T ^ th);
  uint64_t xk[NR];  // wave-uniform
#pragma unroll
  for (int k = 0; k < NR; ++k) xk[k] = pdep64((uint64_t)k, th);
  const uint64_t n_tiles = 1ull << (A.n_qubits - M);
  const int wave = __builtin_amdgcn_readfirstlane(tid & ~63);
  double er = 0.0, ei = 0.0;
  uint64_t tile = blockIdx.x, base = pdep64(tile, full & ~T);
  if (tile < n_tiles) {
#pragma unroll
    for (int k = 0; k < NR; ++k) buf[tid + k * NT] = psi[base + xt + xk[k]];
    __syncthreads();
  }
  while (tile < n_tiles) {
    // The next tile loads while this one's groups run (but for lambda in complex128, whose
    // registers would then hold only one workgroup per CU).
    constexpr bool ahead = !(LAM && sizeof(R) == 8);
    const uint64_t next = tile + gridDim.x, next_base = next < n_tiles ? pdep64(next, full & ~T) : base;
    R nx[NR], ny[NR];
    auto load_next = [&] {
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const C v = psi[next_base + xt + xk[k]];
        nx[k] = v.x;
        ny[k] = v.y;
      }
    };
    if constexpr (ahead) load_next();
    double ar[NR], ai[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) ar[k] = ai[k] = 0.0;
    for (int g = 0; g < A.n_groups; ++g) {
      const PauliMultiGroup G = ld_record(A.groups + g);
      const int half = LAM ? 0 : (int)G.half;
      if (wave & half) continue;
      const PauliMultiTerm* W = A.terms + G.first;
      const int at = tid ^ (int)G.x;
      double f[NR];
      if (G.n_re) {
        pauli_factor<NR>(W, G.n_re, (uint32_t)tid, base, f);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
          if ((k * NT) & half) continue;
          const C v = buf[at ^ (k * NT)];
          ar[k] = __builtin_fma(f[k], (double)v.x, ar[k]);
          ai[k] = __builtin_fma(f[k], (double)v.y, ai[k]);
        }
      }
      if (G.n_im) {
        pauli_factor<NR>(W + G.n_re, G.n_im, (uint32_t)tid, base, f);
#pragma unroll
        for (int k = 0; k < NR; ++k) {
          if ((k * NT) & half) continue;
          const C v = buf[at ^ (k * NT)];
          ar[k] = __builtin_fma(-f[k], (double)v.y, ar[k]);
          ai[k] = __builtin_fma(f[k], (double)v.x, ai[k]);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const C v = buf[tid + k * NT];
      er += (double)v.x * ar[k] + (double)v.y * ai[k];
      if (LAM) ei += (double)v.x * ai[k] - (double)v.y * ar[k];
    }
    if constexpr (LAM) {
      // two slots at a time: the addresses and old values of all of them at once would not
      // leave registers for more than one workgroup per CU
#pragma unroll
      for (int k0 = 0; k0 < NR; k0 += 2) {
        asm volatile("" ::: "memory");
        C* q0 = lam + base + xt + xk[k0];
        C* q1 = lam + base + xt + xk[k0 + 1];
        C l0 = C{0, 0}, l1 = C{0, 0};
        if (A.accumulate) {
          l0 = *q0;
          l1 = *q1;
        }
        *q0 = C{(R)(ar[k0] + (double)l0.x), (R)(ai[k0] + (double)l0.y)};
        *q1 = C{(R)(ar[k0 + 1] + (double)l1.x), (R)(ai[k0 + 1] + (double)l1.y)};
      }
    }
    if constexpr (!ahead) load_next();
    __syncthreads();  // the tile's readers are done
#pragma unroll
    for (int k = 0; k < NR; ++k) buf[tid + k * NT] = C{nx[k], ny[k]};
    __syncthreads();
    tile = next;
    base = next_base;
  }
  pauli_partials(er, ei, A);
}

// ------------------------------------------------------------------------------------------
template <typename R>
static void gather(PauliMultiArgs A, dim3 grid, hipStream_t s) {
  const uint64_t chunks = ((1ull << A.n_qubits) + 255) / 256;
  const bool four = A.n_qubits >= kPauliGatherFour;
  A.splits = 1;
  if (!A.lam && !four) {  // a divisor of the grid
    A.splits = (int32_t)(grid.x / chunks);
    if (A.splits < 1) A.splits = 1;
    while (A.splits > 1 && grid.x % A.splits) --A.splits;
  }
  if (four) {
    if (A.lam) pauli_gather<R, 4, true><<<grid, 256, 0, s>>>(A);
    else pauli_gather<R, 4, false><<<grid, 256, 0, s>>>(A);
  } else {
    if (A.lam) pauli_gather<R, 1, true><<<grid, 256, 0, s>>>(A);
    else pauli_gather<R, 1, false><<<grid, 256, 0, s>>>(A);
  }
}

hipError_t launch_pauli_gather(int dtype, const PauliMultiArgs& A, unsigned blocks, int batch, hipStream_t s) {
  const dim3 grid(blocks, (unsigned)batch);
  if (dtype == 0) gather<float>(A, grid, s);
  else gather<double>(A, grid, s);
  return hipGetLastError();
}

hipError_t launch_pauli_tile(int dtype, const PauliMultiArgs& A, unsigned blocks, int batch, hipStream_t s) {
  const dim3 grid(blocks, (unsigned)batch);
  if (A.n_qubits < kPauliTileQubits) return hipErrorInvalidValue;
  if (dtype == 0) {
    if (A.lam) pauli_tile<float, kPauliTileQubits, 512, true><<<grid, 512, 0, s>>>(A);
    else pauli_tile<float, kPauliTileQubits, 512, false><<<grid, 512, 0, s>>>(A);
  } else {
    if (A.lam) pauli_tile<double, kPauliTileQubits, 512, true><<<grid, 512, 0, s>>>(A);
    else pauli_tile<double, kPauliTileQubits, 512, false><<<grid, 512, 0, s>>>(A);
  }
  return hipGetLastError();
}

}  // namespace qsv
