// Triangular solves, the kriging solve, Newton control, mixed-precision
// refinement steps and fixed-order reductions.  One workgroup per theta unless
// stated otherwise.  Factors may be stored in FP64 or FP32 (template T); every
// solve accumulates in FP64.
#include <cmath>

#include "device.hpp"
#include "host.hpp"
#include "model.hpp"

namespace inla {

// Vector selectors for the step-wise triangular solves (V_* in model.hpp).
__device__ __forceinline__ double *vsel(const ThetaDesc &t, int v) {
  return v == V_X ? t.x : v == V_R ? t.r : v == V_XN ? t.xn : v == V_Z ? t.z : t.u;
}

// v of lane l (a constant).
__device__ __forceinline__ double lane_value(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}

// --------------------------------------------------------------------------
// Triangular solves with the big factor in steps of 256 rows, one launch per step
// over every theta: a workgroup of 1024 threads updates 256 rows (forward) or
// columns (backward) by the step's solved block, and the one that holds the next
// block's also solves that block, by its 64 x 64 sub-blocks with the stored
// inverses of the diagonal ones.  A chain of n / 256 dependent launches, bound by
// latency but for large batches, where the factor's bytes bound it: steps of 256
// in place of 64 because a launch (start, loads of L and of the solved block, the
// next block's solve) takes little longer for four times the rows.
//
// In the solve of a block the 16 waves share every product by its summed index
// (forward) or its result (backward), four each, so that a sub-block costs two
// barriers, and between them one LDS read per lane and sums over lanes by DPP and
// permlane swaps; operands that all lanes need come by readlane, not by LDS reads
// that each would occupy the LDS for a whole wave.  A wave's share of the products
// with the rows (columns) still to be solved stays in its registers until their
// turn comes.  A step of 256 in FP32: 13.3 us forward, 11.9 us backward at order
// 16384, 10.4 and 8.9 us at 1024 with 25 matrices (steps of 64: 4.2 us each and
// 1.5 us between launches); FP64 backward, nine of 3000: 19.5 us (6.1 us and the gap).
// --------------------------------------------------------------------------
constexpr int TSB = 256;
constexpr int TSP = TSB + 2;   // a wave's partial sums: padded against bank conflicts

// Four consecutive values from a 16-byte aligned address.
template <typename T, typename P> __device__ __forceinline__ void load4(T (&v)[4], P p) {
  constexpr int VEC = 16 / sizeof(T);
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  typedef __attribute__((address_space(1))) const vec_t gcvec;
#pragma unroll
  for (int q = 0; q < 4; q += VEC) {
    const vec_t x = *(gcvec *)(p + q);
#pragma unroll
    for (int k = 0; k < VEC; ++k) v[q + k] = x[k];
  }
}

// A factor in lower triangular, column-major form and its stored inverses.
template <typename T> struct TriMat {
  const T *L, *X;
  int ld;
};

// Forward solve of the diagonal block at row i0 (nsub sub-blocks of 64): z to the
// global vector.  acc holds the wave's sums over earlier columns for the block's rows
// 4 l .. 4 l + 3.  Loads run AHEAD sub-blocks ahead and have no conditions: sub-blocks
// and rows are clamped to the block, and values above the diagonal are not used.
template <typename T, typename P>
__device__ __forceinline__ void solve_block_fwd(const TriMat<T> &t, int i0, int nsub, P r, double (&acc)[4], P z,
                                                double *part) {
  constexpr int AHEAD = sizeof(T) == 4 ? 3 : 1;
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q4 = l >> 4;
  const auto *L = gptr(t.L) + (size_t)(i0 + 4 * w) * t.ld + i0;
  const unsigned lr = min(4 * l, 64 * nsub - 4);
  const auto *X = gptr(t.X) + (size_t)(i0 / 64) * 4096 + 4 * w * 64;
  double *p1 = part, *p2 = part + 16 * TSP;
  double rv[4];
  T e[4][4], lo[4][4][4];   // inverses: columns 4 w .. of row l; rows 4 l .. of the sub-block's columns 4 w ..
  auto load = [&](int b) {
    const int bc = min(b, nsub - 1);
    rv[b] = r[i0 + 64 * bc + 4 * w + q4];
#pragma unroll
    for (int q = 0; q < 4; ++q) e[b][q] = X[bc * 4096 + q * 64 + (unsigned)l];
    if (b < 3) {
#pragma unroll
      for (int q = 0; q < 4; ++q) load4(lo[b][q], L + (size_t)(64 * bc + q) * t.ld + lr);
    }
  };
#pragma unroll
  for (int b = 0; b < AHEAD; ++b) load(b);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    if (b >= nsub) break;
    if (b + AHEAD < 4) load(b + AHEAD);
    if (q4 == b) {
#pragma unroll
      for (int q = 0; q < 4; ++q) p1[w * TSP + 4 * l + q] = acc[q];
    }
    __syncthreads();
    const double rb = rv[b] - row_sum16(p1[(l & 15) * TSP + 64 * b + 4 * w + q4]);
    double s = (double)e[b][0] * lane_value(rb, 0) + (double)e[b][1] * lane_value(rb, 16);
    s += (double)e[b][2] * lane_value(rb, 32) + (double)e[b][3] * lane_value(rb, 48);
    p2[w * TSP + 64 * b + l] = s;
    __syncthreads();
    const double zv = row_sum16(p2[(l & 15) * TSP + 64 * b + 4 * w + q4]);
    if ((l & 15) == 0) z[i0 + 64 * b + 4 * w + q4] = zv;
    if (b < 3) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double zq = lane_value(zv, 16 * q);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += (double)lo[b][q][k] * zq;
      }
    }
  }
}

// Back solve x = L_bb^{-T} r of the same block: acc[s][q] holds this lane's part of
// the sum over later rows for column 64 s + 4 w + q.
template <typename T, typename P>
__device__ __forceinline__ void solve_block_bwd(const TriMat<T> &t, int i0, int nsub, P r, double (&acc)[4][4], P x,
                                                double *part) {
  constexpr int AHEAD = sizeof(T) == 4 ? 3 : 1;
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q4 = l >> 4;
  const auto *L = gptr(t.L) + (size_t)(i0 + 4 * w) * t.ld + i0;
  const auto *X = gptr(t.X) + (size_t)(i0 / 64) * 4096 + 4 * w * 64;
  double *sr = part, *sz = part + TSB;
  double rv[4];
  T e[4][4], lo[4][3][4];   // inverses: row l of columns 4 w ..; row l of columns 64 s + 4 w .. of the block row
  auto load = [&](int b) {
    const int bc = min(b, nsub - 1);
    rv[b] = r[i0 + 64 * bc + 4 * w + q4];
#pragma unroll
    for (int q = 0; q < 4; ++q) e[b][q] = X[bc * 4096 + q * 64 + (unsigned)l];
#pragma unroll
    for (int s = 0; s < b; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) lo[b][s][q] = (L + (size_t)(64 * min(s, bc) + q) * t.ld + 64 * bc)[(unsigned)l];
  };
#pragma unroll
  for (int b = 3; b > 3 - AHEAD; --b) load(b);
#pragma unroll
  for (int b = 3; b >= 0; --b) {
    if (b - AHEAD >= 0) load(b - AHEAD);
    if (b >= nsub) continue;
    const double rb = rv[b] - wave_sum4(acc[b]);
    if ((l & 15) == 0) sr[64 * b + 4 * w + q4] = rb;
    __syncthreads();
    const double rl = sr[64 * b + l];
    double zs[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) zs[q] = (double)e[b][q] * rl;
    const double xv = wave_sum4(zs);
    if ((l & 15) == 0) {
      sz[64 * b + 4 * w + q4] = xv;
      x[i0 + 64 * b + 4 * w + q4] = xv;
    }
    if (b > 0) {
      __syncthreads();
      const double zl = sz[64 * b + l];
#pragma unroll
      for (int s = 0; s < b; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[s][q] += (double)lo[b][s][q] * zl;
    }
  }
}

// acc += this wave's part of L[j0 ..][i0 ..] z for rows j0 + 4 l .. (nn rows): its
// columns are i0 + 16 w .., its lanes take four rows each in 16-byte loads.
template <typename T, typename P>
__device__ __forceinline__ void update_fwd(const TriMat<T> &t, int i0, int j0, int nn, P z, double (&acc)[4]) {
  constexpr int U = sizeof(T) == 4 ? 16 : 8;   // loads in flight before the first product
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double zv = z[i0 + 16 * w + (l & 15)];
  const auto *L = gptr(t.L) + (size_t)(i0 + 16 * w) * t.ld + j0;
  const unsigned lr = min(4 * l, nn - 4);
#pragma unroll
  for (int c0 = 0; c0 < 16; c0 += U) {
    T lv[U][4];
#pragma unroll
    for (int c = 0; c < U; ++c) load4(lv[c], L + (size_t)(c0 + c) * t.ld + lr);
#pragma unroll
    for (int c = 0; c < U; ++c) {
      const double zc = lane_value(zv, c0 + c);
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[k] += (double)lv[c][k] * zc;
    }
  }
}

// acc[s][q] += this lane's part (rows i0 + 4 l .., nb rows) of (L^T x)_c for the
// columns c = j0 + 64 s + 4 w + q.
template <typename T, typename P>
__device__ __forceinline__ void update_bwd(const TriMat<T> &t, int i0, int j0, int nb, P x, double (&acc)[4][4]) {
  constexpr int U = sizeof(T) == 4 ? 4 : 2;   // groups of four columns in flight
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned m = min(4 * l, nb - 4);
  double xv[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) xv[k] = 4 * l < nb ? x[i0 + m + k] : 0.0;
  const auto *L = gptr(t.L) + (size_t)(j0 + 4 * w) * t.ld + i0;
#pragma unroll
  for (int s0 = 0; s0 < 4; s0 += U) {
    T lv[U][4][4];
#pragma unroll
    for (int s = 0; s < U; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) load4(lv[s][q], L + (size_t)(64 * (s0 + s) + q) * t.ld + m);
#pragma unroll
    for (int s = 0; s < U; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[s0 + s][q] += ((double)lv[s][q][0] * xv[0] + (double)lv[s][q][1] * xv[1]) +
                          ((double)lv[s][q][2] * xv[2] + (double)lv[s][q][3] * xv[3]);
    __builtin_amdgcn_sched_barrier(0);   // the next group's loads stay behind: registers
  }
}

// x <- L^{-1} x and x <- L^{-T} x by one workgroup of 1024 threads, for the kriging
// factor: the same blocks one after the other, x in global memory.
template <typename T, typename P>
__device__ __forceinline__ void solve_fwd_wg(const TriMat<T> &t, int np, P x, double *part) {
  for (int j0 = 0; j0 < np; j0 += TSB) {
    const int nn = min(TSB, np - j0);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i0 = 0; i0 < j0; i0 += TSB) update_fwd<T>(t, i0, j0, nn, x, acc);
    solve_block_fwd<T>(t, j0, nn / 64, x, acc, x, part);
    __syncthreads();
  }
}
template <typename T, typename P>
__device__ __forceinline__ void solve_bwd_wg(const TriMat<T> &t, int np, P x, double *part) {
  const int last = (np - 1) / TSB * TSB;
  for (int j0 = last; j0 >= 0; j0 -= TSB) {
    double acc[4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[s][q] = 0.0;
    for (int i0 = j0 + TSB; i0 < np; i0 += TSB) update_bwd<T>(t, i0, j0, min(TSB, np - i0), x, acc);
    solve_block_bwd<T>(t, j0, min(TSB, np - j0) / 64, x, acc, x, part);
    __syncthreads();
  }
}

// One step of the forward solve L z = r (blocks from the top); i0 < 0: only the first
// block's solve.  On entry the block's solution is in z.  The rows below are updated,
// r_j -= sum_c L[j][i0 + c] z_c.
template <typename T>
__global__ __launch_bounds__(1024) void trsv_fwd_step_kernel(const ThetaDesc *__restrict__ td, int i0, int src, int dst) {
  const ThetaDesc t = td[blockIdx.y];
  const int np = t.n_pad, j0 = i0 + TSB + blockIdx.x * TSB;
  if (j0 >= np) return;
  const int tid = threadIdx.x, l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nn = min(TSB, np - j0);
  __shared__ __align__(16) double part[(16 + 16) * TSP];
  auto *r = gptr(vsel(t, src));
  auto *z = gptr(vsel(t, dst));
  const TriMat<T> f = {(const T *)t.W, (const T *)t.linv, t.ldw};
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (i0 >= 0) update_fwd<T>(f, i0, j0, nn, z, acc);
  if (blockIdx.x == 0) {   // the next block
    solve_block_fwd<T>(f, j0, nn / 64, r, acc, z, part);
    return;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) part[w * TSP + 4 * l + k] = acc[k];
  __syncthreads();
  if (tid < nn) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 16; ++k) s[k & 3] += part[k * TSP + tid];
    r[j0 + tid] -= (s[0] + s[1]) + (s[2] + s[3]);
  }
}

// One step of the back solve L^T x = r (blocks from the bottom; block starts are
// multiples of 256).  i0 is the step's block; the columns above are updated,
// r_j -= sum_m L[i0 + m][j] x_m.  A matrix whose last block is the
// one above (i0 >= n_pad) starts with that block's solve.
template <typename T>
__global__ __launch_bounds__(1024) void trsv_bwd_step_kernel(const ThetaDesc *__restrict__ td, int i0, int src, int dst) {
  const ThetaDesc t = td[blockIdx.y];
  const int np = t.n_pad, j0 = i0 - TSB - (int)blockIdx.x * TSB;
  if (j0 < 0 || j0 >= np || (i0 >= np && blockIdx.x != 0)) return;
  const int tid = threadIdx.x, l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = min(TSB, np - i0), nn = min(TSB, np - j0);
  __shared__ double part[2 * TSB];
  auto *r = gptr(vsel(t, src));
  auto *x = gptr(vsel(t, dst));
  const TriMat<T> f = {(const T *)t.W, (const T *)t.linv, t.ldw};
  double acc[4][4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[s][q] = 0.0;
  if (nb > 0) update_bwd<T>(f, i0, j0, nb, x, acc);
  if (blockIdx.x == 0) {   // the block above
    solve_block_bwd<T>(f, j0, nn / 64, r, acc, x, part);
    return;
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const double v = wave_sum4(acc[s]);
    if ((l & 15) == s) {
      const int j = j0 + 64 * s + 4 * w + (l >> 4);
      r[j] -= v;
    }
  }
}

// Maxima of three values over a workgroup of 1024 threads, valid in thread 0.
__device__ __forceinline__ void block_max3(double &a, double &b, double &c, double (*sh)[16]) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  a = wave_max(a);
  b = wave_max(b);
  c = wave_max(c);
  if (l == 0) {
    sh[0][w] = a;
    sh[1][w] = b;
    sh[2][w] = c;
  }
  __syncthreads();
  if (w == 0) {
    a = wave_max(sh[0][l & 15]);
    b = wave_max(sh[1][l & 15]);
    c = wave_max(sh[2][l & 15]);
  }
}

// A Newton step taken in correction form starts its new iterate at the current
// one (xn <- x); one refinement step then adds the constrained correction.
__global__ __launch_bounds__(256) void restart_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < t.n_pad) t.xn[i] = t.x[i];
}

// Accept the refined iterate: Newton stopping quantities and x <- xn.
__global__ __launch_bounds__(1024) void newton_accept_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.x];
  __shared__ double sh[3][16];
  double st = 0.0, sc = 0.0, bad = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < t.n; i += 1024) {
    const double xn = t.xn[i], xo = t.x[i];
    if (!isfinite(xn)) bad = 1.0;
    st = fmax(st, fabs(xn - xo));
    sc = fmax(sc, fabs(xn));
  }
  block_max3(st, sc, bad, sh);
#pragma unroll 4
  for (int i = threadIdx.x; i < t.n_pad; i += 1024) t.x[i] = i < t.n ? t.xn[i] : 0.0;
  if (threadIdx.x == 0) {
    t.dres[DRES_STEP] = st;
    t.dres[DRES_SCALE] = fmax(1.0, sc);
    if (bad > 0.0) t.dres[DRES_NONFINITE] = 1.0;
  }
}

// Kriging solve after the small (FP64) factorisation: w from the border row,
// then lambda = L_S^{-T} w; also log|S| = 2 sum log (L_S)_ii, ||w||^2 and the
// numerical-rank flag.  Latency-bound; the diagonal blocks' stored inverses and 16
// waves in place of a 64-step substitution by one: 86 to 13 us at
// k_pad = 128, 39 to 10 us at smaller borders (the residual's two solves 60 to 13 us).
__global__ __launch_bounds__(1024) void kriging_solve_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.x];
  __shared__ double sh[4][16];
  __shared__ __align__(16) double part[2 * 16 * TSP];
  const int kp = t.k_pad, k = t.k, tid = threadIdx.x;
  double lds_ = 0.0, w2 = 0.0, dmin = INFINITY, dmax = 0.0;
  for (int i = tid; i < kp; i += 1024) {
    const double wv = i < k ? t.S[(size_t)i * t.lds + kp] : 0.0;
    t.lam[i] = wv;
    w2 += wv * wv;
    if (i < k) {
      const double d = t.S[(size_t)i * t.lds + i];
      lds_ += log(d);
      dmin = fmin(dmin, d * d);
      dmax = fmax(dmax, d * d);
    }
  }
  lds_ = wave_sum(lds_);
  w2 = wave_sum(w2);
  dmin = -wave_max(-dmin);
  dmax = wave_max(dmax);
  if ((tid & 63) == 0) {
    sh[0][tid >> 6] = lds_;
    sh[1][tid >> 6] = w2;
    sh[2][tid >> 6] = dmin;
    sh[3][tid >> 6] = dmax;
  }
  __syncthreads();
  if (tid == 0) {
    lds_ = w2 = 0.0;
    for (int i = 0; i < 16; ++i) {
      lds_ += sh[0][i];
      w2 += sh[1][i];
      dmin = fmin(dmin, sh[2][i]);
      dmax = fmax(dmax, sh[3][i]);
    }
    t.dres[DRES_LOGDET_S] = 2.0 * lds_;
    t.dres[DRES_WNORM2] = w2;
    // squared pivot below 1e-13 of the largest: numerically dependent constraints
    t.dres[DRES_RANK] = (k > 0 && !(dmin >= 1e-13 * dmax)) ? 1.0 : 0.0;
  }
  if (kp > 0) solve_bwd_wg<double>({t.S, t.linv_s, t.lds}, kp, gptr(t.lam), part);
}

// r_c = z_c - sum_a lambda_a (G L^{-T})_{a,c}.  Newton (from_z = 0): z is the
// factored b row and lambda the kriging multipliers, giving the corrected
// right-hand side of x = L^{-T}(L^{-1} b - L^{-1} C^T lambda).  Refinement
// (from_z = 1): u = L^{-1} r1 and lambda = dlambda.  A wave takes four columns, all
// of their loads in flight together: nine of order 3000, 32 to 8 us.
template <typename T>
__global__ __launch_bounds__(256) void rhs_kernel(const ThetaDesc *__restrict__ td, int from_z) {
  const ThetaDesc t = td[blockIdx.y];
  const int l = threadIdx.x & 63, c0 = blockIdx.x * 16 + (threadIdx.x >> 6) * 4;
  if (c0 >= t.n_pad) return;
  const int k = t.k, np = t.n_pad;
  const auto *lam = gptr((const double *)(from_z ? t.dlam : t.lam));
  const auto *W = gptr((const T *)t.W) + (size_t)c0 * t.ldw + np;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int a = l; a < k; a += 64) {
    const double la = lam[a];
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] += la * (double)W[(size_t)q * t.ldw + a];
  }
  const int c = c0 + (l >> 4);
  const double v = from_z ? t.u[c] : (double)W[(size_t)(l >> 4) * t.ldw + k];
  const double dot = wave_sum4(s);
  if ((l & 15) == 0) t.r[c] = v - dot;
}

// Refinement, constrained part 1: partial sums of (L^{-1} C^T)^T u, u = L^{-1} r1,
// into t.symv (whose residual sums have been used): a workgroup takes 64 border rows
// and 256 columns (BG_COLS), each column read 64 contiguous border values; splits
// because the border's few row blocks alone would leave the chip idle, each a serial
// walk over every column: a batch of order 8192, 164 to 33 us.
constexpr int BG_COLS = 256;
template <typename T>
__global__ __launch_bounds__(256) void border_gemv_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.z];
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int a = blockIdx.x * 64 + l, c0 = blockIdx.y * BG_COLS + 64 * w, np = t.n_pad;
  __shared__ double part[4][64];
  if ((int)blockIdx.x * 64 >= t.k_pad || (int)blockIdx.y * BG_COLS >= np) return;
  double s = 0.0;
  if (c0 < np) {
    const auto *row = gptr((const T *)t.W) + (size_t)c0 * t.ldw + np;
    const double uv = gptr((const double *)t.u)[c0 + l];
#pragma unroll
    for (int c1 = 0; c1 < 64; c1 += 16) {
      T v[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) v[c] = (row + (size_t)(c1 + c) * t.ldw)[(unsigned)min(a, t.k - 1)];
#pragma unroll
      for (int c = 0; c < 16; ++c) s += (double)v[c] * lane_value(uv, c1 + c);
    }
  }
  part[w][l] = s;
  __syncthreads();
  if (w == 0) t.symv[(size_t)blockIdx.y * t.k_pad + a] = (part[0][l] + part[1][l]) + (part[2][l] + part[3][l]);
}

// Refinement, constrained part 2: t = C Q~^{-1} r1 - r2 from the partial sums, then
// dlambda = S~^{-1} t with the FP64 kriging factor.
__global__ __launch_bounds__(1024) void kriging_correct_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.x];
  __shared__ __align__(16) double part[2 * 16 * TSP];
  const int kp = t.k_pad, tid = threadIdx.x, l = tid & 255, p = tid >> 8;
  const int ns = (t.n_pad + BG_COLS - 1) / BG_COLS;
  if (kp == 0) return;
  for (int a0 = 0; a0 < kp; a0 += 256) {   // thread (row, quarter of the splits)
    const int a = a0 + l;
    double s = 0.0;
    if (a < t.k) {
#pragma unroll 8
      for (int j = p; j < ns; j += 4) s += t.symv[(size_t)j * kp + a];
    }
    part[p * 256 + l] = s;
    __syncthreads();
    if (p == 0 && a < kp)
      t.dlam[a] = a < t.k ? ((part[l] + part[256 + l]) + (part[512 + l] + part[768 + l])) - t.rtwo[a] : 0.0;
    __syncthreads();
  }
  const TriMat<double> f = {t.S, t.linv_s, t.lds};
  solve_fwd_wg<double>(f, kp, gptr(t.dlam), part);
  solve_bwd_wg<double>(f, kp, gptr(t.dlam), part);
}

// Refinement, update: xn += dx (dx in u), lambda += dlambda, and the
// quantities of the refinement stopping test.
__global__ __launch_bounds__(1024) void ir_update_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.x];
  __shared__ double sh[3][16];
  double dm = 0.0, xm = 0.0, bad = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < t.n_pad; i += 1024) {
    double v = 0.0;
    if (i < t.n) {
      const double dx = t.u[i];
      v = t.xn[i] + dx;
      if (!isfinite(v)) bad = 1.0;
      dm = fmax(dm, fabs(dx));
      xm = fmax(xm, fabs(v));
    }
    t.xn[i] = v;
  }
  for (int a = threadIdx.x; a < t.k; a += 1024) t.lam[a] += t.dlam[a];
  block_max3(dm, xm, bad, sh);
  if (threadIdx.x == 0) {
    t.dres[DRES_IR_DX] = bad > 0.0 ? INFINITY : dm;
    t.dres[DRES_IR_X] = fmax(1.0, xm);
  }
}

// log|Q| = 2 sum_{i<n} log L_ii of the big factor, and the fixed-order sums of
// the per-column partials (log-likelihood, x^T Q_prior x).
template <typename T>
__global__ __launch_bounds__(256) void finish_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.x];
  __shared__ double sh[4];
  double ld = 0.0, ll = 0.0, xq = 0.0;
  const T *W = (const T *)t.W;
  for (int i = threadIdx.x; i < t.n; i += 256) {
    ld += log((double)W[(size_t)i * t.ldw + i]);
    ll += t.part[i];
    xq += t.part[t.ldw + i];
  }
  for (int i = threadIdx.x; i < t.m; i += 256) ll += t.obs_ll[i];   // general design matrix
  ld = block_sum256(ld, sh);
  ll = block_sum256(ll, sh);
  xq = block_sum256(xq, sh);
  if (threadIdx.x == 0) {
    t.dres[DRES_LOGDET_L] = 2.0 * ld;
    t.dres[DRES_LOGLIK] = ll;
    t.dres[DRES_XQX] = xq;
  }
}

// Start vectors, modes and cleared vectors of a whole batch in one launch.
__global__ __launch_bounds__(256) void copy_vectors_kernel(const VecCopy *__restrict__ v) {
  const VecCopy c = v[blockIdx.y];
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < c.m) c.dst[i] = i < c.n && c.src ? c.src[i] : 0.0;
}

// Caller matrix (t.Quser, ld t.ldquser, order n) -> working matrix (storage T),
// identity padded.
template <typename T>
__global__ __launch_bounds__(256) void copy_in_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int c = blockIdx.x;
  if (c >= t.Nw) return;
  T *col = (T *)t.W + (size_t)c * t.ldw;
  const double *src = t.Quser + (size_t)c * t.ldquser;
  for (int r = c + threadIdx.x; r < t.Nw; r += 256) col[r] = (T)((r < t.n && c < t.n) ? src[r] : (r == c ? 1.0 : 0.0));
}
// Factor -> caller matrix (lower triangle only, as FP64).
template <typename T>
__global__ __launch_bounds__(256) void copy_out_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int c = blockIdx.x;
  if (c >= t.n) return;
  const T *col = (const T *)t.W + (size_t)c * t.ldw;
  double *dst = (double *)t.Quser + (size_t)c * t.ldquser;
  for (int r = c + threadIdx.x; r < t.n; r += 256) dst[r] = (double)col[r];
}

// Marginal variances, small system: S = -Schur(C, C) with the border rows
// V_i = -Schur(I_i, C) (V = Q^{-1} C^T) below it, k_pad columns to factor.
__global__ __launch_bounds__(256) void var_small_build_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int c = blockIdx.x;
  const int kp = t.k_pad, k = t.k, np = t.n_pad;
  if (c >= kp) return;
  double *col = t.S + (size_t)c * t.lds;
  const double *sch = (const double *)t.W + (size_t)(np + c) * t.ldw + np;   // column np + c, from row np
  for (int r = c + threadIdx.x; r < t.Ns; r += 256) {
    double v = 0.0;
    if (r < kp) {
      if (r < k && c < k) v = -sch[r];
      else if (r == c) v = 1.0;
    } else if (c < k) {
      v = -sch[kp + (r - kp)];     // row np + kp + i of the big matrix: identity-border row i
    }
    col[r] = v;
  }
}

// var_i = ||row i of L^{-T}||^2 - ||row i of V L_S^{-T}||^2 (i < n), written to t.out.
// A workgroup takes 64 rows, coalesced, its 16 waves share the columns; L^{-T} is
// upper triangular, so its rows start at their own 64-wide block column.  One thread
// per row over all columns was a serial walk by n / 256 workgroups: nine of
// order 3000, 1265 to 89 us.
__global__ __launch_bounds__(1024) void var_norms_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6, i0 = blockIdx.x * 64, i = i0 + l;
  __shared__ double part[2][16][64];
  if (i0 >= t.n) return;
  const int np = t.n_pad, kp = t.k_pad;
  const auto *row = gptr((const double *)t.W) + np + kp + i;
  double s = 0.0, s2 = 0.0;
#pragma unroll 8
  for (int c = i0 + w; c < np; c += 16) { const double v = row[(size_t)c * t.ldw]; s += v * v; }
  if (t.k > 0) {
    const auto *row2 = gptr((const double *)t.S) + kp + i;
#pragma unroll 4
    for (int c = w; c < t.k; c += 16) { const double v = row2[(size_t)c * t.lds]; s2 += v * v; }
  }
  part[0][w][l] = s;
  part[1][w][l] = s2;
  __syncthreads();
  if (w != 0 || i >= t.n) return;
  double c[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 16; ++q) c[q & 1] += part[0][q][l], c[2 + (q & 1)] += part[1][q][l];
  t.out[i] = (c[0] + c[1]) - (c[2] + c[3]);
}

// ------------------------------------------------------------------ launchers
int copy_vectors(Ctx &ctx, const std::vector<VecCopy> &v) {
  if (v.empty()) return INLA_OK;
  const VecCopy *d = (const VecCopy *)ctx.upload(v.data(), sizeof(VecCopy) * v.size());
  if (!d) return INLA_ERR_NOMEM;
  int m = 0;
  for (const VecCopy &c : v) m = std::max(m, c.m);
  if (m > 0)
    ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
      hipLaunchKernelGGL(copy_vectors_kernel, dim3((m + 255) / 256, v.size()), dim3(256), 0, ctx.stream, d);
    });
  return ctx.check();
}
#define INLA_DISPATCH_T(prec, KERNEL, ...)                                        \
  do {                                                                            \
    if ((prec) != INLA_PREC_FP64) hipLaunchKernelGGL(KERNEL<float>, __VA_ARGS__); \
    else hipLaunchKernelGGL(KERNEL<double>, __VA_ARGS__);                        \
  } while (0)

void launch_kriging_solve(Ctx &ctx, const ThetaDesc *dtd, int B) {
  if (B <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] { hipLaunchKernelGGL(kriging_solve_kernel, dim3(B), dim3(1024), 0, ctx.stream, dtd); });
}
void launch_rhs(Ctx &ctx, const ThetaDesc *dtd, int B, int np_max, int from_z, int prec) {
  if (B <= 0 || np_max <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
    INLA_DISPATCH_T(prec, rhs_kernel, dim3((np_max + 15) / 16, B), dim3(256), 0, ctx.stream, dtd, from_z);
  });
}
void launch_trsv_fwd(Ctx &ctx, const std::vector<ThetaDesc> &htd, int np_max, int src, int dst, double bytes,
                     int prec) {
  const int B = (int)htd.size();
  if (B <= 0 || np_max <= 0) return;
  const std::vector<int64_t> key = {0x54525346, prec != INLA_PREC_FP64, B, np_max, src, dst,
                                    (int64_t)std::llround(bytes)};
  (void)ctx.sequence(INLA_K_SOLVE, key, htd.data(), sizeof(ThetaDesc) * B, [&](const void *dv) {
    const ThetaDesc *dtd = (const ThetaDesc *)dv;
    for (int i0 = -TSB; i0 + TSB < np_max; i0 += TSB) {
      const int gx = i0 < 0 ? 1 : (np_max - i0 - 1) / TSB;
      ctx.launch(INLA_K_SOLVE, 0.0, bytes * (double)(np_max - i0) / np_max * 2.0 * TSB / np_max, [&] {
        INLA_DISPATCH_T(prec, trsv_fwd_step_kernel, dim3(gx, B), dim3(1024), 0, ctx.stream, dtd, i0, src, dst);
      });
    }
  });
}
void launch_trsv_bwd(Ctx &ctx, const std::vector<ThetaDesc> &htd, int np_max, int src, int dst, double bytes,
                     int prec) {
  const int B = (int)htd.size();
  if (B <= 0 || np_max <= 0) return;
  const std::vector<int64_t> key = {0x54525342, prec != INLA_PREC_FP64, B, np_max, src, dst,
                                    (int64_t)std::llround(bytes)};
  (void)ctx.sequence(INLA_K_SOLVE, key, htd.data(), sizeof(ThetaDesc) * B, [&](const void *dv) {
    const ThetaDesc *dtd = (const ThetaDesc *)dv;
    const int top = (np_max + TSB - 1) / TSB * TSB;
    for (int i0 = top; i0 > 0; i0 -= TSB) {
      const int gx = i0 == top ? 1 : i0 / TSB;
      ctx.launch(INLA_K_SOLVE, 0.0, bytes * (double)std::min(i0, np_max) / np_max * 2.0 * TSB / np_max, [&] {
        INLA_DISPATCH_T(prec, trsv_bwd_step_kernel, dim3(gx, B), dim3(1024), 0, ctx.stream, dtd, i0, src, dst);
      });
    }
  });
}
void launch_restart(Ctx &ctx, const ThetaDesc *dtd, int B, int np_max) {
  if (B <= 0 || np_max <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(restart_kernel, dim3((np_max + 255) / 256, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_newton_accept(Ctx &ctx, const ThetaDesc *dtd, int B) {
  if (B <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] { hipLaunchKernelGGL(newton_accept_kernel, dim3(B), dim3(1024), 0, ctx.stream, dtd); });
}
void launch_ir_correct(Ctx &ctx, const ThetaDesc *dtd, int B, int np_max, int kp_max, int prec) {
  if (B <= 0) return;
  if (kp_max > 0)
    ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
      INLA_DISPATCH_T(prec, border_gemv_kernel, dim3(kp_max / 64, (np_max + BG_COLS - 1) / BG_COLS, B), dim3(256), 0, ctx.stream, dtd);
    });
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] { hipLaunchKernelGGL(kriging_correct_kernel, dim3(B), dim3(1024), 0, ctx.stream, dtd); });
}
void launch_ir_update(Ctx &ctx, const ThetaDesc *dtd, int B) {
  if (B <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] { hipLaunchKernelGGL(ir_update_kernel, dim3(B), dim3(1024), 0, ctx.stream, dtd); });
}
void launch_finish(Ctx &ctx, const ThetaDesc *dtd, int B, int prec) {
  if (B <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
    INLA_DISPATCH_T(prec, finish_kernel, dim3(B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_copy_in(Ctx &ctx, const ThetaDesc *dtd, int B, int np_max, int prec) {
  if (B <= 0 || np_max <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    INLA_DISPATCH_T(prec, copy_in_kernel, dim3(np_max, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_copy_out(Ctx &ctx, const ThetaDesc *dtd, int B, int n_max, int prec) {
  if (B <= 0 || n_max <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    INLA_DISPATCH_T(prec, copy_out_kernel, dim3(n_max, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_var_small_build(Ctx &ctx, const ThetaDesc *dtd, int B, int kp_max) {
  if (B <= 0 || kp_max <= 0) return;
  ctx.launch(INLA_K_ASSEMBLE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(var_small_build_kernel, dim3(kp_max, B), dim3(256), 0, ctx.stream, dtd);
  });
}
void launch_var_norms(Ctx &ctx, const ThetaDesc *dtd, int B, int np_max) {
  if (B <= 0 || np_max <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
    hipLaunchKernelGGL(var_norms_kernel, dim3((np_max + 63) / 64, B), dim3(1024), 0, ctx.stream, dtd);
  });
}

}  // namespace inla
