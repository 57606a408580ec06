// Model assembly kernels: prior precision builders, the bordered Q* / b
// assembly with the likelihood terms, the kriging-system build, and the FP64
// residuals of the constrained Newton system used by mixed-precision
// refinement.
#include "device.hpp"
#include "host.hpp"
#include "model.hpp"

namespace inla {

// Sigma_ij = exp(-||p_i - p_j|| / rho) for the first n_s points, identity padded
// to ns_pad, bordered below by the identity (rows ns_pad + i = e_i).  Factoring
// the first ns_pad columns leaves -Sigma^{-1} in the Schur block.  The prior of
// the exponential-covariance models is tau Sigma^{-1}.  Always FP64.
__global__ __launch_bounds__(256) void expcov_bordered_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int c = blockIdx.x;
  const int np = t.ns_pad, N = t.Np;
  if (c >= N) return;
  const int ns = t.prior == PRIOR_EXPCOV ? t.n : t.n_s;
  double *col = t.P + (size_t)c * t.ldp;
  const double inv_rho = 1.0 / t.rho;
  double px = 0.0, py = 0.0;
  if (c < ns) { px = t.coords[2 * c]; py = t.coords[2 * c + 1]; }
  for (int r = c + threadIdx.x; r < N; r += 256) {
    double v = 0.0;
    if (c < np) {
      if (r < np) {
        if (r < ns && c < ns) {
          const double dx = t.coords[2 * r] - px, dy = t.coords[2 * r + 1] - py;
          v = exp(-sqrt(dx * dx + dy * dy) * inv_rho);
        } else if (r == c) {
          v = 1.0;
        }
      } else if (r - np == c) {
        v = 1.0;
      }
    }
    col[r] = v;
  }
}

// Q_prior from -Sigma^{-1} left in the Schur block of P:
//   EXPCOV: Q = tau Sigma^{-1};
//   KRON:   Q[t1 n_s + s1, t2 n_s + s2] = tau (R_t[t1,t2] Sigma_s^{-1}[s1,s2] + delta [i == j]),
//           R_t the unscaled first-order random walk (tridiagonal 1,2,..,2,1 / -1);
//   DENSE:  copy of the caller's matrix (its lower triangle).
// Only the lower triangle (rows r >= c of column c) is written: the assembly
// and the lower-triangle products read no more.  Identity on padded diagonal
// entries; one workgroup per column.
__global__ __launch_bounds__(256) void prior_assemble_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int c = blockIdx.x;
  if (c >= t.n_pad) return;
  double *col = t.Qp + (size_t)c * t.ldqp;
  const int n = t.n;
  if (c >= n) {
    for (int r = c + threadIdx.x; r < t.n_pad; r += 256) col[r] = (r == c) ? 1.0 : 0.0;
    return;
  }
  if (t.prior == PRIOR_DENSE) {
    for (int r = c + threadIdx.x; r < t.n_pad; r += 256) col[r] = r < n ? t.Quser[(size_t)c * t.ldquser + r] : 0.0;
  } else if (t.prior == PRIOR_EXPCOV) {
    const double *Sn = t.P + (size_t)t.ns_pad * t.ldp + t.ns_pad;  // -Sigma^{-1}, lower
    for (int r = c + threadIdx.x; r < t.n_pad; r += 256) col[r] = r < n ? -t.tau * Sn[(size_t)c * t.ldp + r] : 0.0;
  } else {
    const int ns = t.n_s, nt = t.n_t;
    const int t2 = c / ns, s2 = c % ns;
    const double *Sn = t.P + (size_t)t.ns_pad * t.ldp + t.ns_pad;  // -Sigma_s^{-1}, lower
    for (int r = c + threadIdx.x; r < t.n_pad; r += 256) {
      double v = 0.0;
      if (r < n) {
        const int t1 = r / ns, s1 = r % ns;
        double R = 0.0;
        if (t1 == t2) R = (nt == 1) ? 0.0 : ((t1 == 0 || t1 == nt - 1) ? 1.0 : 2.0);
        else if (t1 - t2 == 1 || t2 - t1 == 1) R = -1.0;
        if (R != 0.0) {
          const int a = s1 > s2 ? s1 : s2, b = s1 > s2 ? s2 : s1;
          v = -R * Sn[(size_t)b * t.ldp + a];
        }
        if (r == c) v += t.delta;
        v *= t.tau;
      }
      col[r] = v;
    }
  }
}

// --------------------------------------------------------------------------
// Structured prior pass: log|Q_prior| and S_p = C Q_prior^{-1} C^T without the
// factorisation of the n x n prior.
//
// KRON: Q_prior = tau (R_t kron Sigma_s^{-1} + delta I).  The unscaled random walk
// has the eigenvectors u_i[t] = c_i cos(pi i (2t + 1) / (2 n_t)) (c_0 =
// sqrt(1 / n_t), c_i = sqrt(2 / n_t)) and eigenvalues 4 sin^2(pi i / (2 n_t)), so in
// that basis Q_prior is block diagonal with the n_s x n_s blocks
//   M_i = tau (lambda_i Sigma_s^{-1} + delta I),
// log|Q_prior| = sum_i log|M_i| and S_p = sum_i C_i M_i^{-1} C_i^T with C_i = C (u_i
// kron I): n_t bordered factorisations of order n_s in place of one of order
// n_s n_t (0.5 against 196 GFLOP at n_s = 128, n_t = 64, k = 191).
// EXPCOV: Q_prior = tau Sigma^{-1} with Sigma = L L^T from the prior build, so
// log|Q_prior| = n log tau - log|Sigma| and S_p = (C L)(C L)^T / tau.
// --------------------------------------------------------------------------
// cos(pi m / (2 n_t)), m = 0 .. 4 n_t - 1.
__global__ __launch_bounds__(256) void kron_cosines_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int m = blockIdx.x * 256 + threadIdx.x;
  if (m < 4 * t.n_t) t.ctab[m] = cospi((double)m / (2.0 * t.n_t));
}

// C_i[a][s] = sum_t C[a][t n_s + s] u_i[t] at Ct[(i n_s + s) k + a].  Workgroup
// (s block of 64, a, theta); a wave takes eight i at a time, so that each row of C
// is read n_t / 32 times per wave and not n_t times.
__global__ __launch_bounds__(256) void kron_rows_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.z];
  const int a = blockIdx.y, s = blockIdx.x * 64 + (threadIdx.x & 63);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (a >= t.k || (int)blockIdx.x * 64 >= t.n_s) return;
  const int ns = t.n_s, nt = t.n_t, period = 4 * nt;
  const double *row = t.C + (size_t)a * t.n + min(s, ns - 1);
  constexpr int G = 8;
  for (int i0 = G * w; i0 < nt; i0 += 4 * G) {
    double acc[G];
    int m[G];   // (2 t + 1) i mod 4 n_t
#pragma unroll
    for (int q = 0; q < G; ++q) { acc[q] = 0.0; m[q] = i0 + q; }
    for (int tt = 0; tt < nt; ++tt) {
      const double c = row[(size_t)tt * ns];
#pragma unroll
      for (int q = 0; q < G; ++q) {
        if (i0 + q >= nt) continue;
        acc[q] += c * t.ctab[m[q]];
        m[q] += 2 * (i0 + q);
        if (m[q] >= period) m[q] -= period;
      }
    }
    if (s < ns) {
#pragma unroll
      for (int q = 0; q < G; ++q) {
        const int i = i0 + q;
        if (i < nt) t.Ct[((size_t)i * ns + s) * t.k + a] = acc[q] * sqrt((i == 0 ? 1.0 : 2.0) / nt);
      }
    }
  }
}

// The bordered matrices [M_i; C_i], identity padded, Schur block zero.  Workgroup
// (column, theta, i).
__global__ __launch_bounds__(256) void kron_assemble_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int c = blockIdx.x, i = blockIdx.z, N = t.kN;
  if (c >= N || i >= t.n_t) return;
  double *col = t.K + ((size_t)i * N + c) * N;
  const int ns = t.n_s, np = t.ns_pad, k = t.k;
  const double sn = sinpi((double)i / (2.0 * t.n_t)), lambda = 4.0 * sn * sn;
  const double *Sn = t.P + (size_t)np * t.ldp + np + (size_t)c * t.ldp;  // column c of -Sigma_s^{-1}
  const double *row = t.Ct + ((size_t)i * ns + c) * k;
  for (int r = c + threadIdx.x; r < N; r += 256) {
    double v = 0.0;
    if (c < ns && r < ns) v = t.tau * (t.delta * (r == c) - lambda * Sn[r]);
    else if (r == c && c < np) v = 1.0;
    else if (c < ns && r >= np && r - np < k) v = row[r - np];
    col[r] = v;
  }
}

// The kriging system of the prior (layout of kriging_build_kernel) from the Schur
// blocks -C_i M_i^{-1} C_i^T, added in the order of i.
__global__ __launch_bounds__(256) void kron_schur_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int c = blockIdx.x, kp = t.k_pad, k = t.k, N = t.kN;
  if (c >= kp) return;
  double *col = t.S + (size_t)c * t.lds;
  const double *sch = t.K + (size_t)(t.ns_pad + c) * N + t.ns_pad;
  for (int r = c + threadIdx.x; r < t.Ns; r += 256) {
    double v = 0.0;
    if (r < k && c < k) {
      for (int i = 0; i < t.n_t; ++i) v -= sch[(size_t)i * N * N + r];
    } else if (r < kp) {
      if (r == c) v = 1.0;
    } else if (r == kp && c < k) {
      v = t.e ? -t.e[c] : -0.0;
    }
    col[r] = v;
  }
}

// (C L)[a][c], L the factor of Sigma in P: one wave per (column c, row a).
__global__ __launch_bounds__(256) void expcov_rows_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.z];
  const int a = blockIdx.y, c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (a >= t.k || c >= t.n) return;
  const double *row = t.C + (size_t)a * t.n, *L = t.P + (size_t)c * t.ldp;
  double s = 0.0;
  for (int r = c + lane; r < t.n; r += 64) s += row[r] * L[r];
  s = wave_sum(s);
  if (lane == 0) t.Ct[(size_t)a * t.n_pad + c] = s;
}

// The kriging system of the prior from those rows.  Workgroup (column, theta).
__global__ __launch_bounds__(256) void expcov_schur_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int c = blockIdx.x, kp = t.k_pad, k = t.k;
  if (c >= kp) return;
  __shared__ double sh[4];
  double *col = t.S + (size_t)c * t.lds;
  for (int r = c + threadIdx.x; r < t.Ns; r += 256) {
    double v = 0.0;
    if (r < kp) v = r == c && c >= k ? 1.0 : 0.0;
    else if (r == kp && c < k) v = t.e ? -t.e[c] : -0.0;
    col[r] = v;
  }
  __syncthreads();
  if (c >= k) return;
  const double *yc = t.Ct + (size_t)c * t.n_pad;
  for (int r = c; r < k; ++r) {
    const double *yr = t.Ct + (size_t)r * t.n_pad;
    double s = 0.0;
    for (int i = threadIdx.x; i < t.n; i += 256) s += yr[i] * yc[i];
    s = block_sum256(s, sh);
    if (threadIdx.x == 0) col[r] = s / t.tau;
  }
}

// log|Q_prior| from the factors' diagonals (all M_i, or Sigma); not a number where
// Q_prior is singular to the rounding of its own factorisation, which then decides
// (the caller takes the general pass).  Cholesky of Q_prior breaks down when its
// smallest eigenvalue is within a few n eps of its largest element; the pass here
// never forms that matrix and would accept any delta above zero, or points a rounding
// apart.  In units of tau the eigenvalue is delta (KRON, by R_t's null vector) or at least
// 1 / n (EXPCOV, Sigma's elements being at most 1), and the largest element
// max R_t max (Sigma^{-1})_ii + delta.  The general pass refuses, a pivot or the rank of
// the constraints, up to 3 n eps (orders 60 to 3000); the line is at 16.
__global__ __launch_bounds__(256) void structured_logdet_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.x];
  __shared__ double sh[4];
  const bool kron = t.prior == PRIOR_KRON;
  double s = 0.0, big = 0.0;
  for (int i = threadIdx.x; i < t.n; i += 256) {
    const double *A = kron ? t.K + (size_t)(i / t.n_s) * t.kN * t.kN : t.P;
    const int c = kron ? i % t.n_s : i, ld = kron ? t.kN : t.ldp;
    s += log(A[(size_t)c * ld + c]);
    // P's Schur block: -Sigma^{-1}
    if (i < t.n_s) big = fmax(big, -t.P[(size_t)(t.ns_pad + i) * (t.ldp + 1)]);
  }
  s = block_sum256(s, sh);
  big = block_max256(big, sh);
  if (threadIdx.x != 0) return;
  const double low = kron ? t.delta : 1.0 / t.n;
  const double top = kron ? min(t.n_t - 1, 2) * big + t.delta : big;
  if (!(low > 16.0 * t.n * 2.220446049250313e-16 * top)) s = __builtin_nan("");
  t.dres[DRES_LOGDET_L] = kron ? 2.0 * s : t.n * log(t.tau) - 2.0 * s;
}

__device__ __forceinline__ void lik_point_at(const ThetaDesc &t, int i, double x, double &g, double &W, double &ll) {
  const double y = t.y[i];
  if (t.lik == LIK_GAUSSIAN) {
    const double s2 = t.lpar;
    const double r = y - x;
    g = r / s2;
    W = 1.0 / s2;
    ll = -0.5 * log(2.0 * M_PI * s2) - r * r / (2.0 * s2);
  } else {
    const double E = t.E ? t.E[i] : 1.0;
    const double eta = t.lpar + x;
    const double mu = E * exp(eta);
    g = y - mu;
    W = mu;
    ll = y * (log(E) + eta) - mu - lgamma(y + 1.0);
  }
}

// g = d log pi(y_i | eta) / d eta and W = -d^2 log pi / d eta^2 at eta(x); in a
// variational-Bayes pass their expectations over eta ~ N(eta(x), vb_var[i])
// (appendix "Variational Bayes approximation strategy": I' = -E g, I'' = E W),
// by Gauss-Hermite quadrature: E h = sum_j w_j / sqrt(pi) h(eta + sqrt(2 var) r_j).
__device__ __forceinline__ void lik_point(const ThetaDesc &t, int i, double x, double &g, double &W, double &ll) {
  lik_point_at(t, i, x, g, W, ll);
  if (!t.vb_var) return;
  const double sd = sqrt(2.0 * t.vb_var[i]);
  double eg = 0.0, ew = 0.0;
  for (int j = 0; j < t.ngh; ++j) {
    double gj, wj, lj;
    lik_point_at(t, i, x + sd * t.gh[j], gj, wj, lj);
    eg += t.gh[t.ngh + j] * gj;
    ew += t.gh[t.ngh + j] * wj;
  }
  g = eg;
  W = ew;
}

// Per observation of a model with a general design matrix: (A x)_i by the CSR
// row, then the likelihood terms at eta_i = offset + (A x)_i.
__global__ __launch_bounds__(256) void obs_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (t.m == 0 || i >= t.m) return;
  double ax = 0.0;
  for (int p = t.A_rowptr[i]; p < t.A_rowptr[i + 1]; ++p) ax += t.A_val[p] * t.x[t.A_col[p]];
  double g, W, ll;
  lik_point_at(t, i, ax, g, W, ll);
  t.obs_ax[i] = ax;
  t.obs_g[i] = g;
  t.obs_W[i] = W;
  t.obs_ll[i] = ll;
}

// The bordered posterior precision of one Newton step (algorithm "Gaussian
// Approximation": Q* = Q_prior + Q_l(x0), b = grad + Q_l x0; A = I so Q_l is the
// diagonal W), written in the factorisation's storage type T:
//   rows [0, n_pad)          Q_prior + diag(W)            (lower)
//   rows n_pad + a, a < k    constraint row C_a
//   row  n_pad + k           b^T                 (border == BORDER_CB)
//   rows n_pad + kc_pad + i  e_i^T               (border == BORDER_CI)
// Schur-block columns start at zero.  `with_lik` = 0 gives the prior pass
// (W = 0, b = 0).  Per-column partial sums of log pi(y|eta) and x^T Q_prior x go
// to t.part for a fixed-order reduction.
//
// HBM-bound.  A workgroup takes ASM_C columns, a thread two rows of them in 16-byte
// loads: with one column per workgroup most of its life went to the descriptor and
// the likelihood.  Nine of order 3000: 178 to 146 us, the 25 of order 1024 in FP32 52
// to 26, with an identity border 940 to 260 us; at order 8192 and above one column
// is as good (980 to 967 us for eight in FP64, two of 16384 in FP32 464 to 500).
// Two and eight columns: 147 and 160 us at 3000.
constexpr int ASM_C = 4;
template <typename T>
__global__ __launch_bounds__(256) void assemble_kernel(const ThetaDesc *__restrict__ td, int with_lik, int want_xqx,
                                                       int border) {
  const ThetaDesc t = td[blockIdx.y];
  const int c0 = blockIdx.x * ASM_C, N = t.Nw, tid = threadIdx.x;
  if (c0 >= t.Ncw) return;
  auto *col = gptr((T *)t.W) + (size_t)c0 * t.ldw;
  const int np = t.n_pad, n = t.n, k = t.k;
  if (c0 >= np) {
    for (int r = c0 + tid; r < N; r += 256)
#pragma unroll
      for (int q = 0; q < ASM_C; ++q)
        if (r >= c0 + q) col[(size_t)q * t.ldw + r] = (T)0;
    return;
  }
  __shared__ double sW[ASM_C], sb[ASM_C], sx[4][ASM_C];
  if (tid < ASM_C) {
    const int c = c0 + tid;
    double g = 0.0, W = 0.0, ll = 0.0, xc = 0.0;
    if (c < n) {
      xc = t.x[c];
      if (with_lik && t.m == 0) lik_point(t, c, xc, g, W, ll);
    }
    sW[tid] = W;
    sb[tid] = with_lik && t.m == 0 ? g + W * xc : 0.0;
    t.part[c] = ll;
  }
  __syncthreads();
  const auto *Q = gptr((const double *)t.Qp) + (size_t)c0 * t.ldqp;
  const auto *C = gptr(t.C) + c0;
  const int kc_pad = round_up_dev(k, PADN);
  double xq[ASM_C];
#pragma unroll
  for (int q = 0; q < ASM_C; ++q) xq[q] = 0.0;
  typedef T t2 __attribute__((ext_vector_type(2)));
  typedef __attribute__((address_space(1))) t2 gt2;
#pragma unroll 2
  for (int r = c0 + 2 * tid; r < np; r += 512) {
    d2 v[ASM_C];
#pragma unroll
    for (int q = 0; q < ASM_C; ++q) v[q] = *(gcd2 *)(Q + (size_t)q * t.ldqp + r);
    if (want_xqx) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (r + h >= n) break;
        const double xr = t.x[r + h];
#pragma unroll
        for (int q = 0; q < ASM_C; ++q)
          if (r + h >= c0 + q) xq[q] += (r + h == c0 + q ? 1.0 : 2.0) * v[q][h] * xr;
      }
    }
#pragma unroll
    for (int q = 0; q < ASM_C; ++q) {
      auto *p = col + (size_t)q * t.ldw + r;
      if (r == c0 + q) v[q][0] += sW[q];
      if (r + 1 == c0 + q) v[q][1] += sW[q];
      if (r >= c0 + q) *(gt2 *)p = t2{(T)v[q][0], (T)v[q][1]};
      else if (r + 1 == c0 + q) p[1] = (T)v[q][1];
    }
  }
  for (int r = np + tid; r < N; r += 256) {
    const int a = r - np;
    double v[ASM_C];
#pragma unroll
    for (int q = 0; q < ASM_C; ++q) {
      if (a < k) v[q] = c0 + q < n ? C[(size_t)a * n + q] : 0.0;
      else if (border == BORDER_CB) v[q] = a == k ? sb[q] : 0.0;
      else v[q] = a - kc_pad == c0 + q ? 1.0 : 0.0;
    }
#pragma unroll
    for (int q = 0; q < ASM_C; ++q) col[(size_t)q * t.ldw + r] = (T)v[q];
  }
  if (want_xqx) {
#pragma unroll
    for (int q = 0; q < ASM_C; ++q) {
      const double d = wave_sum(xq[q]);
      if ((tid & 63) == 0) sx[tid >> 6][q] = d;
    }
    __syncthreads();
    if (tid < ASM_C) {
      const int c = c0 + tid;
      t.part[t.ldw + c] = c < n ? ((sx[0][tid] + sx[1][tid]) + (sx[2][tid] + sx[3][tid])) * t.x[c] : 0.0;
    }
  }
  if (tid < ASM_C && (!isfinite(sW[tid]) || !isfinite(sb[tid]))) t.dres[DRES_NONFINITE] = 1.0;
}

// A general design matrix's share of the assembled columns: b_c = (A^T (g + W A x))_c in
// the border row and (A^T W A)_{r c} on the lower pattern.  One workgroup per column and
// a launch of its own: an intercept's or a factor level's column is a long serial walk
// over its observations, and four of them in one workgroup of the assembly follow one
// another (two of order 4807 with columns of 4000 entries: 1,680 to 805 us a pass, both
// launches together).
__global__ __launch_bounds__(256) void design_columns_kernel(const ThetaDesc *__restrict__ td, int border) {
  const ThetaDesc t = td[blockIdx.y];
  const int c = blockIdx.x, tid = threadIdx.x;
  if (t.m == 0 || c >= t.n) return;
  auto *col = gptr((double *)t.W) + (size_t)c * t.ldw;
  __shared__ double sh[4];
  // fixed-order block sum over the CSC column
  double b = 0.0;
  for (int p = t.cscp[c] + tid; p < t.cscp[c + 1]; p += 256) {
    const int i = t.csci[p];
    b += t.cscv[p] * (t.obs_g[i] + t.obs_W[i] * t.obs_ax[i]);
  }
  b = block_sum256(b, sh);
  double bad = isfinite(b) ? 0.0 : 1.0;
  if (border == BORDER_CB && tid == 0) col[t.n_pad + t.k] = b;
  for (int e = t.patp[c] + tid; e < t.patp[c + 1]; e += 256) {   // (distinct rows)
    double v = 0.0;
    for (int p = t.patt[e]; p < t.patt[e + 1]; ++p) v += t.tcoef[p] * t.obs_W[t.tobs[p]];
    if (!isfinite(v)) bad = 1.0;
    col[t.patr[e]] += v;
  }
  bad = block_sum256(bad, sh);
  if (tid == 0 && bad > 0.0) t.dres[DRES_NONFINITE] = 1.0;
}

// Kriging system from the Schur block -[[S, C x_u], [., b^T x_u]] of the big
// factorisation: S into rows/cols [0, k) (identity padded to k_pad) and the
// border row (C x_u - e)^T at row k_pad, always in FP64.  Factoring it leaves
// L_S and w^T = (C x_u - e)^T L_S^{-T} in the border row.
template <typename T>
__global__ __launch_bounds__(256) void kriging_build_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int c = blockIdx.x;
  const int kp = t.k_pad, N = t.Ns, k = t.k;
  if (c >= kp) return;   // only the k_pad factor columns exist; the border is a row
  double *col = t.S + (size_t)c * t.lds;
  const T *sch = (const T *)t.W + (size_t)(t.n_pad + c) * t.ldw + t.n_pad;
  for (int r = c + threadIdx.x; r < N; r += 256) {
    double v = 0.0;
    if (r < kp) {
      if (r < k && c < k) v = -(double)sch[r];
      else if (r == c) v = 1.0;
    } else if (r == kp && c < k) {
      const double e = t.e ? t.e[c] : 0.0;
      v = -(double)sch[k] - e;   // C x_u - e (Schur holds -C Q^{-1} b = -C x_u)
    }
    col[r] = v;
  }
}

// y = Q_prior v from the lower triangle of Q_prior alone (half the bytes of a
// whole-column product; the consumers below finish it).  A workgroup takes up to
// SYMV_TILES 64 x 64 tiles of block column J, from the diagonal down: row r of a tile
// receives sum_{c in J, c <= r} Q_rc v_c, written to P[J][r]; column c receives
// sum_{r > c} Q_rc v_r over the tiles, written to D[c] by the first workgroup of the
// block column and to P[J + s][c] by its s-th further one, rows of P that hold no row
// sums above the diagonal.  Then (Q v)_i = D[i] + the sum of P[j][i] over
// j < i / 64 + (workgroups of that block column), in a fixed order (no atomics).
// A lane keeps one row of 16 columns, so both products come from the registers that
// were loaded, and only their sums cross lanes, once per workgroup.  HBM-bound; four
// tiles, since one workgroup per block column leaves the longest to run alone: at
// order 16384, over a run's launches for two theta and for one, 724 to 279 us on average
// (two 442 us, 4.9 TB/s; 25 of order 8192 1.36 ms, 4.9 TB/s); 25 of 1024 44 to 16 us.
// src 0: v = xn (refinement residuals); 1: v = x (objective terms).
constexpr int SYMV_TILES = 4;
__device__ __forceinline__ int symv_splits(int np, int J) { return (np / 64 - J + SYMV_TILES - 1) / SYMV_TILES; }
__global__ __launch_bounds__(256) void symv_lower_part_kernel(const ThetaDesc *__restrict__ td, int src) {
  const ThetaDesc t = td[blockIdx.z];
  const int J = blockIdx.x, sp = blockIdx.y, c0 = J * 64, np = t.n_pad, n = t.n;
  const int r0 = c0 + sp * 64 * SYMV_TILES;
  if (r0 >= np) return;
  const auto *v = gptr((const double *)(src ? t.x : t.xn));
  __shared__ double red[SYMV_TILES][4][64];
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double *P = t.symv;
  const auto *Q = gptr((const double *)t.Qp) + (size_t)(c0 + 16 * w) * t.ldqp;
  double vc[16], col[16];   // the wave's columns c0 + 16 w ..
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int c = c0 + 16 * w + q;
    vc[q] = c < n ? v[c] : 0.0;
    col[q] = 0.0;
  }
#pragma unroll
  for (int i = 0; i < SYMV_TILES; ++i) {
    const int r = r0 + 64 * i;
    if (r >= np) break;
    double x[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) x[q] = (Q + (size_t)q * t.ldqp + r)[(unsigned)l];
    const double vr = r + l < n ? v[r + l] : 0.0;
    const bool diag = r == c0;
    double s[2] = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int c = 16 * w + q;
      s[q & 1] += (diag && c > l ? 0.0 : x[q]) * vc[q];
      col[q] += (diag && c >= l ? 0.0 : x[q]) * vr;
    }
    red[i][w][l] = s[0] + s[1];
  }
  __syncthreads();
  const int r = r0 + 64 * w + l;   // wave w adds up tile w
  if (r < np) P[(size_t)J * np + r] = (red[w][0][l] + red[w][1][l]) + (red[w][2][l] + red[w][3][l]);
  double *D = P + (size_t)(sp == 0 ? np / 64 : J + sp) * np + c0 + 16 * w;
#pragma unroll
  for (int q = 0; q < 16; q += 4) {
    const double d = wave_sum4(col + q);
    if ((l & 15) == 0) D[q + (l >> 4)] = d;
  }
}

// (Q_prior v)_i from the partial sums of symv_lower_part_kernel.
__device__ __forceinline__ double symv_row(const ThetaDesc &t, int i) {
  const int np = t.n_pad, nj = i / 64 + symv_splits(np, i / 64);
  double y = t.symv[(size_t)(np / 64) * np + i];
#pragma unroll 8
  for (int j = 0; j < nj; ++j) y += t.symv[(size_t)j * np + i];
  return y;
}

// FP64 residual of the constrained Newton system at the refined iterate xn:
//   r1 = b - (Q_prior + diag W) xn - C^T lambda,   b = g(x) + W(x) x
// with g, W at the linearisation point x and Q_prior xn from the lower-triangle
// partial sums, the result to t.z.  A workgroup takes 64 rows, its 16 waves a 16th of
// the partial sums and of the constraints each: one thread per row walks both alone,
// which for two of n = 16384 is 128 workgroups and 193 us (now 17).
__global__ __launch_bounds__(1024) void kkt_residual_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6, np = t.n_pad;
  const int i = blockIdx.x * 64 + l, ic = min(i, t.n - 1), nj = blockIdx.x + symv_splits(np, blockIdx.x);
  __shared__ double part[16][64];
  if ((int)blockIdx.x * 64 >= np) return;
  double s = 0.0;
#pragma unroll 4
  for (int j = w; j < nj; j += 16) s += t.symv[(size_t)j * np + i];
#pragma unroll 4
  for (int a = w; a < t.k; a += 16) s += t.C[(size_t)a * t.n + ic] * t.lam[a];
  part[w][l] = s;
  __syncthreads();
  if (w != 0) return;
  double r = 0.0;
  if (i < t.n) {
    double c[4] = {t.symv[(size_t)(np / 64) * np + i], 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 16; ++q) c[q & 3] += part[q][l];
    double g, W, ll;
    lik_point(t, i, t.x[i], g, W, ll);
    r = (g + W * t.x[i]) - W * t.xn[i] - ((c[0] + c[1]) + (c[2] + c[3]));
  }
  t.z[i] = r;
}

// Objective terms at the mode without re-assembling: x^T Q_prior x (from the
// lower-triangle partial sums of Q_prior x) and log pi(y | eta) into the
// per-column partial sums read by the finish kernel.  Used when the last Newton
// factorisation is reused for log|Q*|.
__global__ __launch_bounds__(256) void objective_terms_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= t.n_pad) return;
  double ll = 0.0, xq = 0.0;
  if (i < t.n) {
    double g, W;
    lik_point(t, i, t.x[i], g, W, ll);
    xq = t.x[i] * symv_row(t, i);
  }
  t.part[i] = ll;
  t.part[t.ldw + i] = xq;
}

// r2 = e - C xn, a workgroup per constraint row (zero on padded rows).
__global__ __launch_bounds__(256) void constraint_residual_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int a = blockIdx.x;
  __shared__ double sh[4];
  if (a >= t.k_pad) return;
  double s = 0.0;
  if (a < t.k) {
#pragma unroll 8
    for (int i = threadIdx.x; i < t.n; i += 256) s += t.C[(size_t)a * t.n + i] * t.xn[i];
  }
  s = block_sum256(s, sh);
  if (threadIdx.x == 0) t.rtwo[a] = a < t.k ? (t.e ? t.e[a] : 0.0) - s : 0.0;
}

// ------------------------------------------------------------------ launchers
void launch_expcov_bordered(Ctx &ctx, const ThetaDesc *dtd, int B, int Np_max) {
  if (B <= 0 || Np_max <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(expcov_bordered_kernel, dim3(Np_max, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_prior_assemble(Ctx &ctx, const ThetaDesc *dtd, int B, int np_max, double bytes) {
  if (B <= 0 || np_max <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, bytes, [&] {
    hipLaunchKernelGGL(prior_assemble_kernel, dim3(np_max, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_kron_rows(Ctx &ctx, const ThetaDesc *dtd, int B, int ns_max, int nt_max, int k_max) {
  if (B <= 0 || k_max <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(kron_cosines_kernel, dim3((4 * nt_max + 255) / 256, B), dim3(256), 0, ctx.stream, dtd);
  });
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(kron_rows_kernel, dim3((ns_max + 63) / 64, k_max, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_kron_assemble(Ctx &ctx, const ThetaDesc *dtd, int B, int N_max, int nt_max) {
  if (B <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(kron_assemble_kernel, dim3(N_max, B, nt_max), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_kron_schur(Ctx &ctx, const ThetaDesc *dtd, int B, int kp_max) {
  if (B <= 0 || kp_max <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(kron_schur_kernel, dim3(kp_max, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_expcov_schur(Ctx &ctx, const ThetaDesc *dtd, int B, int n_max, int k_max, int kp_max) {
  if (B <= 0 || k_max <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(expcov_rows_kernel, dim3((n_max + 3) / 4, k_max, B), dim3(256), 0, ctx.stream, dtd);
  });
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(expcov_schur_kernel, dim3(kp_max, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_structured_logdet(Ctx &ctx, const ThetaDesc *dtd, int B) {
  if (B <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(structured_logdet_kernel, dim3(B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_assemble(Ctx &ctx, const ThetaDesc *dtd, int B, int N_max, int with_lik, int want_xqx, int border,
                     double bytes, int prec, int m_max) {
  if (B <= 0 || N_max <= 0) return;
  if (with_lik && m_max > 0)
    ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
      hipLaunchKernelGGL(obs_kernel, dim3((m_max + 255) / 256, B), dim3(256), 0, ctx.stream, dtd);
    });
  ctx.launch(INLA_K_ASSEMBLE, 0.0, bytes, [&] {
    if (prec != INLA_PREC_FP64)
      hipLaunchKernelGGL(assemble_kernel<float>, dim3(N_max / ASM_C, B), dim3(256), 0, ctx.stream, dtd, with_lik, want_xqx,
                         border);
    else
      hipLaunchKernelGGL(assemble_kernel<double>, dim3(N_max / ASM_C, B), dim3(256), 0, ctx.stream, dtd, with_lik, want_xqx,
                         border);
  });
  if (with_lik && m_max > 0)   // (FP64: such models are evaluated in no other precision)
    ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
      hipLaunchKernelGGL(design_columns_kernel, dim3(N_max, B), dim3(256), 0, ctx.stream, dtd, border);
    });
}
void launch_kriging_build(Ctx &ctx, const ThetaDesc *dtd, int B, int kp_max, int prec) {
  if (B <= 0 || kp_max <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    if (prec != INLA_PREC_FP64)
      hipLaunchKernelGGL(kriging_build_kernel<float>, dim3(kp_max, B), dim3(256), 0, ctx.stream, dtd);
    else
      hipLaunchKernelGGL(kriging_build_kernel<double>, dim3(kp_max, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_objective_terms(Ctx &ctx, const ThetaDesc *dtd, int B, int np_max, double bytes) {
  if (B <= 0 || np_max <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, bytes, [&] {
    hipLaunchKernelGGL(symv_lower_part_kernel, dim3(np_max / 64, (np_max / 64 + SYMV_TILES - 1) / SYMV_TILES, B), dim3(256), 0,
                       ctx.stream, dtd, 1);
  });
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(objective_terms_kernel, dim3((np_max + 255) / 256, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_kkt_residual(Ctx &ctx, const ThetaDesc *dtd, int B, int np_max, int kp_max, double bytes) {
  if (B <= 0 || np_max <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, bytes, [&] {
    hipLaunchKernelGGL(symv_lower_part_kernel, dim3(np_max / 64, (np_max / 64 + SYMV_TILES - 1) / SYMV_TILES, B), dim3(256), 0,
                       ctx.stream, dtd, 0);
  });
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(kkt_residual_kernel, dim3(np_max / 64, B), dim3(1024), 0, ctx.stream, dtd);
  });
  if (kp_max > 0)
    ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
      hipLaunchKernelGGL(constraint_residual_kernel, dim3(kp_max, B), dim3(256), 0, ctx.stream, dtd);
    });
}

}  // namespace inla
