// Imaginary-time kernels: thermal blocks and the exponential-collocation propagator.
//
// Propagator weights for one amplitude with orbital-energy difference D and
// panel width h (composite exponential Gauss collocation of the integral
// equation eqn:smu; nodes c_x, Lagrange basis l_y(u) = sum_k lc[y][k] u^k):
//   E_x  = exp(-D h c_x)
//   W_xy = h int_0^{c_x} exp(D h (u - c_x)) l_y(u) du
//        = h sum_k lc[y][k] c_x^(k+1) k! phi_{k+1}(-D h c_x)
//   We_y = h sum_k lc[y][k] k! phi_{k+1}(-D h)
// with phi_k(z) = int_0^1 exp((1-t) z) t^(k-1) / (k-1)! dt.  phi_k is summed by
// its Taylor series for |z| <= 4 and by the recurrence
// phi_{k+1} = (phi_k - 1/k!) / z from phi_1 = expm1(z)/z otherwise (both
// directions are well conditioned there).  The h-derivative used by the beta
// response is d/dh [h phi_{k+1}(a h)] = (z - k) phi_{k+1}(z) + 1/k!; the
// D-derivative used by the orbital-energy response follows from
// phi_k'(z) = phi_k(z) - k phi_{k+1}(z):
// d/dD [h phi_{k+1}(-D h c)] = -h^2 c (phi_{k+1}(z) - (k+1) phi_{k+2}(z)).
#include <hip/hip_runtime.h>
#include <math.h>

#include "gmem.h"
#include "tau_kernels.h"

namespace ftcc {

// 1/k!, compile-time so that the series' coefficients are literals: read from a table
// they were a chain of scalar loads that cost more than the series' arithmetic
// (2-block launch of a 6-site ring, 1024 elements a block: 32 us a sweep before).
struct InvFact {
  double f[48];
  constexpr InvFact() : f() {
    f[0] = 1.0;
    for (int k = 1; k < 48; ++k) f[k] = f[k - 1] / k;
  }
};
constexpr InvFact kInvFact;

// phi[k] = phi_k(z) for k = 1..kmax.  Small |z|: phi_kmax by its Taylor series,
// then downward phi_k = z phi_{k+1} + 1/k! (stable there: |z| <= 4 and every term
// of the series is positive for z > 0).
template <int kmax>
__device__ __forceinline__ void phi_all(double z, double* phi) {
  if (fabs(z) <= 4.0) {
    double acc = kInvFact.f[kmax + 34];
#pragma unroll
    for (int j = 33; j >= 0; --j) acc = fma(acc, z, kInvFact.f[j + kmax]);
    phi[kmax] = acc;
#pragma unroll
    for (int k = kmax - 1; k >= 1; --k) phi[k] = fma(z, phi[k + 1], kInvFact.f[k]);
  } else {
    double p = expm1(z) / z;
    phi[1] = p;
#pragma unroll
    for (int k = 1; k < kmax; ++k) {
      p = (p - kInvFact.f[k]) / z;
      phi[k + 1] = p;
    }
  }
}

// Weights of one amplitude for a panel of M nodes (M is a compile-time constant,
// so the arrays live in registers).
template <int M>
struct Weights {
  double E[M], W[M][M], We[M], Ee;
};

// need_end: also the panel-end row (Ee, We).  deriv: 0 the weights, 1 their
// h-derivatives at fixed D, 2 their D-derivatives at fixed h.
template <int M>
__device__ void weights(const PanelRule& R, double D, double h, Weights<M>& w, int deriv, bool need_end) {
  // R is the rule in global memory (uniform across the grid: scalar loads)
  constexpr int m = M;
  double phi[M + 2];
#pragma unroll
  for (int x = 0; x <= m; ++x) {
    if (x == m && !need_end) break;
    const double cx = (x < m) ? R.c[x] : 1.0;
    const double z = -D * h * cx;
    double e = exp(z);
    if (deriv == 1) e = -D * cx * e;            // dE/dh
    else if (deriv == 2) e = -h * cx * e;       // dE/dD
    if (x < m) w.E[x] = e; else w.Ee = e;
    if (R.lawson) {
#pragma unroll
      for (int y = 0; y < m; ++y) {
        const double arg = D * h * (R.c[y] - cx);
        const double a = (x < m) ? R.A[x][y] : R.b[y];
        const double v = deriv == 1 ? a * exp(arg) * (1.0 + arg)
                                    : (deriv == 2 ? h * a * exp(arg) * h * (R.c[y] - cx) : h * a * exp(arg));
        if (x < m) w.W[x][y] = v; else w.We[y] = v;
      }
      continue;
    }
    if (deriv == 2) phi_all<M + 1>(z, phi);
    else phi_all<M>(z, phi);
#pragma unroll
    for (int y = 0; y < m; ++y) {
      double acc = 0.0;
#pragma unroll
      for (int k = 0; k < m; ++k) {
        const double g = R.gc[x][y][k];
        if (deriv == 1) acc += g * ((z - k) * phi[k + 1] + kInvFact.f[k]);
        else if (deriv == 2) acc += g * (phi[k + 1] - (k + 1) * phi[k + 2]);
        else acc += g * phi[k + 1];
      }
      if (deriv == 0) acc *= h;
      else if (deriv == 2) acc *= -h * h * cx;
      if (x < m) w.W[x][y] = acc; else w.We[y] = acc;
    }
  }
}

// orbital-energy difference of element e of a t1 (rank 2, [i][a]) or t2
// (rank 4, [i][j][a][b]) segment
__device__ __forceinline__ double seg_delta(const double* eps_ptr, int n, int rank, long e) {
  const gptr<const double> eps = gview(eps_ptr);
  // element offsets are below 2^32 (n <= 256)
  const unsigned un = (unsigned)n, ue = (unsigned)e;
  if (rank == 2) return eps[ue % un] - eps[ue / un];
  unsigned r = ue / un;
  const unsigned b = ue - r * un;
  unsigned q = r / un;
  const unsigned a = r - q * un;
  const unsigned i = q / un;
  const unsigned j = q - i * un;
  return eps[a] + eps[b] - eps[i] - eps[j];
}

__device__ __forceinline__ double delta_of(const TauProblem& P, long e) { return seg_delta(P.eps, P.n, P.rank, e); }

// max that propagates a NaN b as +infinity (fmax would drop it); a is not NaN
__device__ __forceinline__ double nan_max(double a, double b) {
  if (b != b) return INFINITY;
  return fmax(a, b);
}

__device__ __forceinline__ void atomic_max_pos(unsigned long long* p, double v) {
  // non-negative doubles order like their bit patterns; the maximum only grows, so a
  // block whose value is not above a (possibly old) reading of it has nothing to add
  if ((unsigned long long)__double_as_longlong(v) <= __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    return;
  atomicMax(p, (unsigned long long)__double_as_longlong(v));
}

// One element per thread (IT = 1); TAU_BETA four (IT = 4), its partial sums being one
// per 1024 elements.  A loop over a thread's elements would queue them up behind each
// other where the chip is not full, and the compiler would keep the series' 35
// coefficients in registers across it (245 VGPRs).
template <int M, int IT>
__global__ void __launch_bounds__(256) tau_kernel(const PanelRule* __restrict__ rule, int mode,
                                                  const TauProblem* __restrict__ probs,
                                                  const int* __restrict__ prefix, int n_prob) {
  int lo = 0, hi = n_prob - 1;
  const int b = blockIdx.x;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= b) lo = mid; else hi = mid - 1;
  }
  const TauProblem& P = probs[lo];
  if (P.active && *gview(P.active) == 0) return;   // converged instance of a batch: left unchanged
  const PanelRule& R = *rule;
  constexpr int m = M;
  const long base = (long)(b - prefix[lo]) * (256 * IT);
  double mchg = 0.0, mval = 0.0, acc = 0.0;
  for (int u = 0; u < IT; ++u) {
    const long ei = base + u * 256 + threadIdx.x;
    if (ei >= P.len) break;
    const long e = P.idx ? (long)gview(P.idx)[ei] : ei;   // element of the segment, and where it lies
    const long at = P.pack ? (long)((unsigned)e / P.pack) : e;
    const double sb = P.sb ? gview(P.sb)[at] : 0.0;
    double Sv[M];
    bool any = (sb != 0.0);
    for (int y = 0; y < m; ++y) {
      Sv[y] = P.S[y] ? gview(P.S[y])[at] : 0.0;
      any = any || (Sv[y] != 0.0);
    }
    if (mode == TAU_LSTEP || mode == TAU_LSWEEP) {
      for (int x = 0; x < m; ++x) {
        const double nv = -gview(P.R[x])[at];
        mchg = nan_max(mchg, fabs(nv - gview(P.s[x])[at]));
        mval = nan_max(mval, fabs(nv));
        gview(P.s[x])[at] = nv;
        Sv[x] = nv;
        any = any || nv != 0.0;
      }
      if (mode == TAU_LSTEP) continue;   // TAU_LSWEEP: lambda-tilde of the new lambda below
    }
    if ((IT == 4 && mode == TAU_BETA) || (IT == 1 && mode == TAU_DEPS)) {
      double Rv[M];
      bool anyb = any || (P.lam_a && gview(P.lam_a)[at] != 0.0);
      for (int y = 0; y < m; ++y) {
        Rv[y] = gview(P.R[y])[at];
        anyb = anyb || (Rv[y] != 0.0);
      }
      if (!anyb) continue;
      Weights<M> w;
      weights<M>(R, delta_of(P, e), P.h, w, mode == TAU_BETA ? 1 : 2, P.lam_a != nullptr);
      double val = 0.0;
      for (int x = 0; x < m; ++x) {
        double f = (sb != 0.0) ? -w.E[x] * sb : 0.0;
        for (int y = 0; y < m; ++y)
          if (Rv[y] != 0.0) f += w.W[x][y] * Rv[y];
        val += Sv[x] * f;
      }
      if (P.lam_a) {
        double f = (sb != 0.0) ? -w.Ee * sb : 0.0;
        for (int y = 0; y < m; ++y)
          if (Rv[y] != 0.0) f += w.We[y] * Rv[y];
        val += gview(P.lam_a)[at] * f;
      }
      if (mode == TAU_BETA) acc += val;
      else gview(P.out)[at] += val;
      continue;
    }
    if (IT == 4) continue;   // TAU_BETA only
    if (!any) {
      // structurally zero (dropped slots, or zero start): outputs stay zero
      if (mode == TAU_LSWEEP) {
        for (int x = 0; x < m; ++x) gview(P.lamt[x])[at] = 0.0;
      } else if (mode == TAU_INIT || mode == TAU_LAMT) {
        for (int x = 0; x < m; ++x) gview(P.s[x])[at] = 0.0;
      } else if (mode == TAU_STEP) {
        for (int x = 0; x < m; ++x) {
          mchg = nan_max(mchg, fabs(gview(P.s[x])[at]));
          gview(P.s[x])[at] = 0.0;
        }
      } else {
        gview(P.out)[at] = 0.0;
      }
      continue;
    }
    Weights<M> w;
    weights<M>(R, delta_of(P, e), P.h, w, 0, mode != TAU_INIT && mode != TAU_STEP);
    if (mode == TAU_INIT) {
      for (int x = 0; x < m; ++x) gview(P.s[x])[at] = (sb != 0.0) ? w.E[x] * sb : 0.0;
    } else if (mode == TAU_STEP) {
      for (int x = 0; x < m; ++x) {
        double v = (sb != 0.0) ? w.E[x] * sb : 0.0;
        for (int y = 0; y < m; ++y)
          if (Sv[y] != 0.0) v -= w.W[x][y] * Sv[y];
        mchg = nan_max(mchg, fabs(v - gview(P.s[x])[at]));
        mval = nan_max(mval, fabs(v));
        gview(P.s[x])[at] = v;
      }
    } else if (mode == TAU_END) {
      double v = (sb != 0.0) ? w.Ee * sb : 0.0;
      for (int y = 0; y < m; ++y)
        if (Sv[y] != 0.0) v -= w.We[y] * Sv[y];
      gview(P.out)[at] = v;
    } else if (mode == TAU_LAMT || mode == TAU_LSWEEP) {
      for (int x = 0; x < m; ++x) {
        double v = (sb != 0.0) ? w.We[x] * sb : 0.0;
        for (int y = 0; y < m; ++y)
          if (Sv[y] != 0.0) v += w.W[y][x] * Sv[y];
        gview(mode == TAU_LAMT ? P.s[x] : P.lamt[x])[at] = v;
      }
    } else if (mode == TAU_APREV) {
      double v = (sb != 0.0) ? w.Ee * sb : 0.0;
      for (int x = 0; x < m; ++x)
        if (Sv[x] != 0.0) v += w.E[x] * Sv[x];
      gview(P.out)[at] = v;
    }
  }
  // block reductions
  __shared__ double r0[256], r1[256];
  if (mode == TAU_STEP || mode == TAU_LSTEP || mode == TAU_LSWEEP) {
    r0[threadIdx.x] = mchg;
    r1[threadIdx.x] = mval;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
      if (threadIdx.x < s) {
        r0[threadIdx.x] = nan_max(r0[threadIdx.x], r0[threadIdx.x + s]);
        r1[threadIdx.x] = nan_max(r1[threadIdx.x], r1[threadIdx.x + s]);
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      atomic_max_pos(P.maxbits, r0[0]);
      atomic_max_pos(P.maxbits + 1, r1[0]);
    }
  } else if (IT == 4 && mode == TAU_BETA) {
    r0[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
      if (threadIdx.x < s) r0[threadIdx.x] += r0[threadIdx.x + s];
      __syncthreads();
    }
    if (threadIdx.x == 0) gview(P.partial)[b - prefix[lo]] = r0[0];
  }
}

void launch_tau(const PanelRule* d_rule, int m, int mode, const TauProblem* d_probs, const int* d_prefix, int n_prob,
                int total_blocks, hipStream_t s) {
  if (total_blocks <= 0) return;
#define FTCC_TAU(MM)                                                                                            \
  case MM:                                                                                                      \
    if (mode == TAU_BETA)                                                                                       \
      hipLaunchKernelGGL((tau_kernel<MM, 4>), dim3(total_blocks), dim3(256), 0, s, d_rule, mode, d_probs,       \
                         d_prefix, n_prob);                                                                     \
    else                                                                                                        \
      hipLaunchKernelGGL((tau_kernel<MM, 1>), dim3(total_blocks), dim3(256), 0, s, d_rule, mode, d_probs,       \
                         d_prefix, n_prob);                                                                     \
    break;
  switch (m) {
    FTCC_TAU(1)
    FTCC_TAU(2)
    FTCC_TAU(3)
    FTCC_TAU(4)
    FTCC_TAU(5)
    FTCC_TAU(6)
  }
#undef FTCC_TAU
}

// Runge-Kutta combinations (differential form, Algorithm alg:diff):
//   out = x0 * base + sum_l coef[l] * (-Delta Y_l + sigma S_l)
// over the (allowed) elements of one segment, one per thread: a loop over a thread's
// elements would queue their scattered loads up behind each other (33 labelled
// orbitals, up to nine states: 12.0 us with four).
__global__ void __launch_bounds__(256) rk_combine_kernel(const RKProblem* __restrict__ probs,
                                                         const int* __restrict__ prefix, int n_prob) {
  int lo = 0, hi = n_prob - 1;
  const int b = blockIdx.x;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= b) lo = mid; else hi = mid - 1;
  }
  const RKProblem& P = probs[lo];
  if (P.active && *gview(P.active) == 0) return;   // uniform per block, before the barrier
  const long ei = (long)(b - prefix[lo]) * kRKBlock + threadIdx.x;
  double vmax = 0.0;
  if (ei < P.len) {
    const long e = P.idx ? (long)gview(P.idx)[ei] : ei;
    const long at = P.pack ? (long)((unsigned)e / P.pack) : e;
    const double d = seg_delta(P.eps, P.n, P.rank, e);
    const double hx = P.h_x0 ? *gview(P.h_x0) : 1.0, hc = P.h_coef ? *gview(P.h_coef) : 1.0;
    double v = P.base ? hx * P.x0 * gview(P.base)[at] : 0.0;
    for (int l = 0; l < P.nst; ++l) {
      const double y = P.Y[l] ? gview(P.Y[l])[at] : 0.0;
      const double sv = P.S[l] ? gview(P.S[l])[at] : 0.0;
      v += hc * P.coef[l] * (-d * y + P.sigma * sv);
    }
    gview(P.out)[at] = v;
    vmax = nan_max(0.0, fabs(v));   // a NaN as infinity: nan_max below would drop one on its left
  }
  if (!P.maxbits) return;   // uniform per launch problem
  __shared__ double red[256];
  red[threadIdx.x] = vmax;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] = nan_max(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) atomic_max_pos(P.maxbits, red[0]);
}

void launch_rk_combine(const RKProblem* d_probs, const int* d_prefix, int n_prob, int total_blocks, hipStream_t s) {
  if (total_blocks <= 0) return;
  hipLaunchKernelGGL(rk_combine_kernel, dim3(total_blocks), dim3(256), 0, s, d_probs, d_prefix, n_prob);
}

__global__ void __launch_bounds__(256) expsum_kernel(const ExpSumProblem* __restrict__ probs,
                                                     const int* __restrict__ prefix, int n_prob) {
  int lo = 0, hi = n_prob - 1;
  const int b = blockIdx.x;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= b) lo = mid; else hi = mid - 1;
  }
  const ExpSumProblem& P = probs[lo];
  if (P.active && *gview(P.active) == 0) return;   // uniform per block, before the barrier
  const long first = (long)(b - prefix[lo]) * 1024;
  double vmax = 0.0, cmax = 0.0;
  for (int u = 0; u < 4; ++u) {
    const long ei = first + u * 256 + threadIdx.x;
    if (ei >= P.len) break;
    const long e = P.idx ? (long)gview(P.idx)[ei] : ei;
    const long at = P.pack ? (long)((unsigned)e / P.pack) : e;
    const double d = seg_delta(P.eps, P.n, P.rank, e);
    double acc = 0.0;
    for (int l = 0; l < P.nterms; ++l) {
      const ExpTerm t = P.terms[l];
      const double x = gview(t.X)[at];
      if (x == 0.0) continue;
      const double z = d * P.h * t.k;
      const double ex = exp(-z);
      const double f = P.mode == 0 ? P.h * t.C * ex
                                   : (P.mode == 1 ? t.C * ex * (1.0 - z) : -P.h * P.h * t.C * t.k * ex);
      acc += f * x;
    }
    if (P.prod) acc *= gview(P.prod)[at];
    const double v = (P.base ? P.x0 * gview(P.base)[at] : 0.0) + acc;
    if (P.maxbits) cmax = nan_max(cmax, fabs(v - gview(P.out)[at]));
    gview(P.out)[at] = v;
    vmax = nan_max(vmax, fabs(v));
  }
  if (!P.maxbits) return;   // uniform per launch problem
  __shared__ double r0[256], r1[256];
  r0[threadIdx.x] = cmax;
  r1[threadIdx.x] = vmax;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) {
      r0[threadIdx.x] = nan_max(r0[threadIdx.x], r0[threadIdx.x + st]);
      r1[threadIdx.x] = nan_max(r1[threadIdx.x], r1[threadIdx.x + st]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    atomic_max_pos(P.maxbits, r0[0]);
    atomic_max_pos(P.maxbits + 1, r1[0]);
  }
}

void launch_expsum(const ExpSumProblem* d_probs, const int* d_prefix, int n_prob, int total_blocks, hipStream_t s) {
  if (total_blocks <= 0) return;
  hipLaunchKernelGGL(expsum_kernel, dim3(total_blocks), dim3(256), 0, s, d_probs, d_prefix, n_prob);
}

__global__ void __launch_bounds__(256) copy_listed_kernel(const unsigned* __restrict__ a, long na,
                                                          const unsigned* __restrict__ b, long nb, long second,
                                                          const double* __restrict__ src, double* __restrict__ dst) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= na + nb) return;
  const long off = e < na ? (long)gview(a)[e] : second + (long)gview(b)[e - na];
  gview(dst)[off] = gview(src)[off];
}

void launch_copy_listed(const unsigned* a, long na, const unsigned* b, long nb, long second, const double* src,
                        double* dst, hipStream_t s) {
  const long total = na + nb;
  if (total <= 0) return;
  hipLaunchKernelGGL(copy_listed_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a, na, b, nb,
                     second, src, dst);
}

// A segment between dense storage and storage without the last index: the allowed
// elements `list`, dense element e against packed element e / n.
__global__ void __launch_bounds__(256) repack_kernel(const unsigned* __restrict__ list, long count, unsigned n,
                                                     double* __restrict__ dense, double* __restrict__ packed,
                                                     bool to_packed) {
  const long k = (long)blockIdx.x * 256 + threadIdx.x;
  if (k >= count) return;
  const unsigned e = gview(list)[k];
  if (to_packed) gview(packed)[e / n] = gview(dense)[e];
  else gview(dense)[e] = gview(packed)[e / n];
}

void launch_repack(const unsigned* list, long count, int n, double* dense, double* packed, bool to_packed,
                   hipStream_t s) {
  if (count <= 0) return;
  hipLaunchKernelGGL(repack_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, list, count, (unsigned)n,
                     dense, packed, to_packed);
}

// ------------------------------------------------------------------ thermal quantities
__global__ void __launch_bounds__(256) state_copy_kernel(const StateCopy* __restrict__ copies,
                                                         const int* __restrict__ prefix, int n) {
  int lo = 0, hi = n - 1;
  const int b = blockIdx.x;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= b) lo = mid; else hi = mid - 1;
  }
  const StateCopy& C = copies[lo];
  if (C.active && *gview(C.active) == 0) return;
  const long first = (long)(b - prefix[lo]) * kStateCopyBlock;
#pragma unroll
  for (int u = 0; u < (int)(kStateCopyBlock / 256); ++u) {
    const long e = first + u * 256 + threadIdx.x;
    if (e >= C.len) return;
    long off = e;
    if (C.a) off = e < C.na ? (long)gview(C.a)[e] : C.second + (long)gview(C.b)[e - C.na];
    double v = C.src ? gview(C.src)[off] : 0.0;
    if (C.add) v += gview(C.dst)[off];
    gview(C.dst)[off] = v;
  }
}

void launch_state_copies(const StateCopy* d_copies, const int* d_prefix, int n, int blocks, hipStream_t s) {
  if (n <= 0 || blocks <= 0) return;
  hipLaunchKernelGGL(state_copy_kernel, dim3(blocks), dim3(256), 0, s, d_copies, d_prefix, n);
}

__global__ void occ_kernel(const SetupProblem* probs, const double* mubeta, double thr) {
  const SetupProblem& P = probs[blockIdx.y];
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P.n) return;
  const double x = mubeta[2 * blockIdx.y + 1] * (P.eps[p] - mubeta[2 * blockIdx.y]);
  // n = 1 / (1 + e^x), 1 - n = 1 / (1 + e^-x), each without cancellation
  double nocc, nvir;
  if (x > 0.0) {
    const double t = exp(-x);
    nocc = t / (1.0 + t);
    nvir = 1.0 / (1.0 + t);
  } else {
    const double t = exp(x);
    nocc = 1.0 / (1.0 + t);
    nvir = t / (1.0 + t);
  }
  P.occ[p] = nocc;
  P.wo[p] = (nocc > thr) ? sqrt(nocc) : 0.0;
  P.wv[p] = (nvir > thr) ? sqrt(nvir) : 0.0;
}

// f_pq = h_pq + sum_r (g <pr|qr> - <pr|rq>) n_r, u = f - diag(eps)
__global__ void fock_kernel(const SetupProblem* probs, double g) {
  const SetupProblem& P = probs[blockIdx.z];
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  const int n = P.n;
  if (q >= n || p >= n) return;
  double acc = P.h[(long)p * n + q];
#pragma unroll 8
  for (int r = 0; r < n; ++r) {
    const double d = gview(P.eri)[(((long)p * n + r) * n + q) * n + r];
    const double x = gview(P.eri)[(((long)p * n + r) * n + r) * n + q];
    acc += (g * d - x) * gview(P.occ)[r];
  }
  P.fock[(long)p * n + q] = acc;
  P.u_raw[(long)p * n + q] = acc - (p == q ? P.eps[p] : 0.0);
}

// dn, dw along mu, beta or eps_q (dn_p/deps_q = -beta n_q (1 - n_q) delta_pq)
__global__ void occ_deriv_kernel(const SetupProblem* probs, const double* mubeta, int which, int q) {
  const SetupProblem& P = probs[blockIdx.y];
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P.n || (which == SETUP_EPS && q >= P.n)) return;
  const double mu = mubeta[2 * blockIdx.y], beta = mubeta[2 * blockIdx.y + 1];
  const double x = beta * (P.eps[p] - mu);
  const double nvir = (x > 0.0) ? 1.0 / (1.0 + exp(-x)) : exp(x) / (1.0 + exp(x));
  const double nn1 = P.occ[p] * nvir;
  const double d = which == SETUP_MU ? beta * nn1
                                     : (which == SETUP_BETA ? -(P.eps[p] - mu) * nn1 : (p == q ? -beta * nn1 : 0.0));
  P.dn[p] = d;
  P.dwo[p] = (P.wo[p] > 0.0) ? d / (2.0 * P.wo[p]) : 0.0;
  P.dwv[p] = (P.wv[p] > 0.0) ? -d / (2.0 * P.wv[p]) : 0.0;
}

// du_pq = dh_pq + sum_r (g <pr|qr> - <pr|rq>) dn_r + sum_r (g d<pr|qr> - d<pr|rq>) n_r; along
// eps_q the explicit part of u = f - diag(eps) is -e_q e_q^T
__global__ void fock_deriv_kernel(const SetupProblem* probs, const double* const* dirs, int which, int eq, double g) {
  const SetupProblem& P = probs[blockIdx.z];
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  const int n = P.n;
  if (q >= n || p >= n || (which == SETUP_EPS && eq >= n)) return;
  const double* dh = which == SETUP_DIR ? dirs[2 * blockIdx.z] : nullptr;
  const double* deri = which == SETUP_DIR ? dirs[2 * blockIdx.z + 1] : nullptr;
  double acc = dh ? dh[(long)p * n + q] : 0.0;
  if (which == SETUP_EPS && p == eq && q == eq) acc = -1.0;
  if (which != SETUP_DIR || deri) {
    const gptr<const double> v = gview(which == SETUP_DIR ? deri : P.eri);
    const gptr<const double> occ = gview((const double*)(which == SETUP_DIR ? P.occ : P.dn));
#pragma unroll 8
    for (int r = 0; r < n; ++r) {
      const long id = (((long)p * n + r) * n + q) * n + r;
      const long ix = (((long)p * n + r) * n + r) * n + q;
      acc += (g * v[id] - v[ix]) * occ[r];
    }
  }
  P.du_raw[(long)p * n + q] = acc;
}

// ------------------------------------------------------------------ weighted blocks
// Every block of every instance in one pass: an element of <pq|rs> is read once and its
// 12 weighted copies are written (one launch per block and instance before: 12 reads
// and, for a batch of 16 small instances, 256 launches per set-up).
//   out = (prod w) * dX + sum_k (prod_{j != k} w_j) dw_k * X
template <int R, bool DERIV>
__device__ __forceinline__ double weighted(int holes, const double (&wo)[R], const double (&wv)[R],
                                           const double (&dwo)[R], const double (&dwv)[R], bool has_d, double base,
                                           bool has_dx, double dx) {
  double w[R], prod = 1.0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    w[k] = (holes >> k) & 1 ? wo[k] : wv[k];
    prod *= w[k];
  }
  double v = has_dx ? prod * dx : 0.0;
  if (DERIV && has_d) {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      double pk = (holes >> k) & 1 ? dwo[k] : dwv[k];
      if (pk == 0.0) continue;
#pragma unroll
      for (int j = 0; j < R; ++j)
        if (j != k) pk *= w[j];
      v += pk * base;
    }
  }
  return v;
}

template <bool DERIV>
__global__ void __launch_bounds__(256) blocks_kernel(const SetupProblem* __restrict__ probs,
                                                     const int* __restrict__ prefix, int n_prob,
                                                     const double* const* __restrict__ dirs, int which, int eq) {
  int lo = 0, hi = n_prob - 1;
  const int b = blockIdx.x;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= b) lo = mid; else hi = mid - 1;
  }
  const SetupProblem& P = probs[lo];
  const unsigned n = (unsigned)P.n;
  if (DERIV && which == SETUP_EPS && eq >= P.n) return;
  const bool has_d = DERIV && which != SETUP_DIR;
  const long n2 = (long)n * n, cnt4 = P.idx ? P.count : n2 * n2;
  const long t = (long)(b - prefix[lo]) * 256 + threadIdx.x;
  const gptr<const double> wo = gview((const double*)P.wo), wv = gview((const double*)P.wv);
  const gptr<const double> dwo = gview((const double*)P.dwo), dwv = gview((const double*)P.dwv);
  if (t < cnt4) {
    const unsigned e = P.idx ? gview(P.idx)[t] : (unsigned)t;   // n <= 256: below 2^32
    unsigned i[4], r = e;
    i[3] = r % n;
    r /= n;
    i[2] = r % n;
    r /= n;
    i[1] = r % n;
    i[0] = r / n;
    double a[4], v[4], da[4] = {}, dv[4] = {};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a[k] = wo[i[k]];
      v[k] = wv[i[k]];
      if (has_d) {
        da[k] = dwo[i[k]];
        dv[k] = dwv[i[k]];
      }
    }
    const double* deri = DERIV && which == SETUP_DIR ? dirs[2 * lo + 1] : nullptr;
    const double base = !DERIV || has_d ? gview(P.eri)[e] : 0.0;
    const double dx = DERIV ? (deri ? gview(deri)[e] : 0.0) : base;
#pragma unroll
    for (int k = 0; k < 12; ++k)
      gview(DERIV ? P.dg[k] : P.g[k])[e] =
          weighted<4, DERIV>(kBlockHoles[k], a, v, da, dv, has_d, base, !DERIV || deri != nullptr, dx);
    return;
  }
  const long e2 = t - cnt4;
  if (e2 >= n2) return;
  const unsigned p = (unsigned)e2 / n, q = (unsigned)e2 % n;
  const double a[2] = {wo[p], wo[q]}, v[2] = {wv[p], wv[q]};
  double da[2] = {}, dv[2] = {};
  if (has_d) {
    da[0] = dwo[p];
    da[1] = dwo[q];
    dv[0] = dwv[p];
    dv[1] = dwv[q];
  }
  const double base = P.u_raw[e2];
  const double dx = DERIV ? P.du_raw[e2] : base;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    gview(DERIV ? P.du[k] : P.u[k])[e2] = weighted<2, DERIV>(kBlockHoles1[k], a, v, da, dv, has_d, base, true, dx);
}

void launch_thermal(const SetupProblem* d_probs, const double* d_mubeta, const int* d_prefix, int n_prob, int n_max,
                    int blocks, double thr, double g, hipStream_t s) {
  const unsigned c = (n_max + 63) / 64;
  hipLaunchKernelGGL(occ_kernel, dim3(c, n_prob), dim3(64), 0, s, d_probs, d_mubeta, thr);
  hipLaunchKernelGGL(fock_kernel, dim3(c, n_max, n_prob), dim3(64), 0, s, d_probs, g);
  hipLaunchKernelGGL(blocks_kernel<false>, dim3(blocks), dim3(256), 0, s, d_probs, d_prefix, n_prob,
                     (const double* const*)nullptr, 0, 0);
}

void launch_setup_deriv(const SetupProblem* d_probs, const double* d_mubeta, const double* const* d_dirs,
                        const int* d_prefix, int n_prob, int n_max, int blocks, int which, int q, double g,
                        hipStream_t s) {
  const unsigned c = (n_max + 63) / 64;
  if (which != SETUP_DIR)
    hipLaunchKernelGGL(occ_deriv_kernel, dim3(c, n_prob), dim3(64), 0, s, d_probs, d_mubeta, which, q);
  hipLaunchKernelGGL(fock_deriv_kernel, dim3(c, n_max, n_prob), dim3(64), 0, s, d_probs, d_dirs, which, q, g);
  hipLaunchKernelGGL(blocks_kernel<true>, dim3(blocks), dim3(256), 0, s, d_probs, d_prefix, n_prob, d_dirs, which, q);
}

// ------------------------------------------------------------------ DIIS (Anderson) extrapolation
// One thread per instance: minimise |sum_j c_j r_j|^2 subject to sum_j c_j = 1 over
// the `count` stored residuals (Gram matrix G, row-major with leading dimension
// ld), by Gaussian elimination with partial pivoting on the bordered system.
// A singular or non-finite system falls back to the newest iterate (plain Picard).
__global__ void diis_solve_kernel(int n_inst, const int* counts, const int* newest, const double* G, int ld,
                                  double* coef) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_inst) return;
  const int k = counts[i];
  const double* g = G + (long)i * ld * ld;
  double* c = coef + (long)i * ld;
  double A[9][10];
  double scale = 0.0;
  for (int a = 0; a < k; ++a) scale = fmax(scale, fabs(g[a * ld + a]));
  bool ok = (k > 1) && scale > 0.0 && isfinite(scale);
  if (ok) {
    for (int a = 0; a < k; ++a) {
      for (int b = 0; b < k; ++b) A[a][b] = g[a * ld + b] / scale;
      A[a][k] = -1.0;
      A[a][k + 1] = 0.0;
    }
    for (int b = 0; b < k; ++b) A[k][b] = -1.0;
    A[k][k] = 0.0;
    A[k][k + 1] = -1.0;
    const int nn = k + 1;
    for (int col = 0; col < nn && ok; ++col) {
      int piv = col;
      for (int r = col + 1; r < nn; ++r)
        if (fabs(A[r][col]) > fabs(A[piv][col])) piv = r;
      if (!(fabs(A[piv][col]) > 1e-14)) {
        ok = false;
        break;
      }
      if (piv != col)
        for (int q = 0; q <= nn; ++q) {
          const double t = A[col][q];
          A[col][q] = A[piv][q];
          A[piv][q] = t;
        }
      for (int r = 0; r < nn; ++r) {
        if (r == col) continue;
        const double f = A[r][col] / A[col][col];
        for (int q = col; q <= nn; ++q) A[r][q] -= f * A[col][q];
      }
    }
    if (ok)
      for (int a = 0; a < k; ++a) {
        c[a] = A[a][nn] / A[a][a];
        if (!isfinite(c[a])) ok = false;
      }
  }
  if (!ok)
    for (int a = 0; a < ld; ++a) c[a] = (a == newest[i]) ? 1.0 : 0.0;
}

void launch_diis_solve(int n_inst, const int* counts, const int* newest, const double* G, int ld, double* coef,
                       hipStream_t s) {
  hipLaunchKernelGGL(diis_solve_kernel, dim3((n_inst + 63) / 64), dim3(64), 0, s, n_inst, counts, newest, G, ld,
                     coef);
}

// out[e] = sum_j coef[j] * (X_j[e] + R_j[e])
__global__ void diis_combine_kernel(long len, DiisTerms t, double* out) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= len) return;
  double v = 0.0;
  for (int j = 0; j < t.k; ++j) {
    const double cj = t.coef[j];
    if (cj != 0.0) v += cj * (t.X[j][e] + t.R[j][e]);
  }
  out[e] = v;
}

void launch_diis_combine(long len, const DiisTerms& t, double* out, hipStream_t s) {
  if (len <= 0) return;
  hipLaunchKernelGGL(diis_combine_kernel, dim3((len + 255) / 256), dim3(256), 0, s, len, t, out);
}

// ------------------------------------------------------------------ small utilities
__global__ void sum_kernel(const double* x, int count, double* out) {
  __shared__ double r[256];
  double a = 0.0;
  for (int i = threadIdx.x; i < count; i += 256) a += x[i];
  r[threadIdx.x] = a;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) r[threadIdx.x] += r[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = r[0];
}

__global__ void __launch_bounds__(256) partial_sums_kernel(const double* partial, const int* off, double scale,
                                                           double* const* acc, int slot) {
  __shared__ double r[256];
  double a = 0.0;
  for (int i = off[blockIdx.x] + threadIdx.x; i < off[blockIdx.x + 1]; i += 256) a += partial[i];
  r[threadIdx.x] = a;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) r[threadIdx.x] += r[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) acc[blockIdx.x][slot] = scale * r[0] + acc[blockIdx.x][slot];
}

void launch_partial_sums(int n_inst, const double* partial, const int* off, double scale, double* const* acc, int slot,
                         hipStream_t s) {
  hipLaunchKernelGGL(partial_sums_kernel, dim3(n_inst), dim3(256), 0, s, partial, off, scale, acc, slot);
}

void launch_sum(const double* x, int count, double* out, hipStream_t s) {
  hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(256), 0, s, x, count, out);
}

__global__ void axpby_kernel(long len, double a, const double* x, double b, double* y) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= len) return;
  const double xv = (a != 0.0) ? a * x[e] : 0.0;
  y[e] = (b != 0.0) ? xv + b * y[e] : xv;
}

void launch_axpby(long len, double a, const double* x, double b, double* y, hipStream_t s) {
  if (len <= 0) return;
  hipLaunchKernelGGL(axpby_kernel, dim3((len + 255) / 256), dim3(256), 0, s, len, a, x, b, y);
}

}  // namespace ftcc
