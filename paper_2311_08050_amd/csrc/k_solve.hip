// Triangular solves, the kriging solve, Newton control, mixed-precision
// refinement steps and fixed-order reductions.  One workgroup per theta unless
// stated otherwise.  Factors may be stored in FP64 or FP32 (template T); every
// solve accumulates in FP64.
#include <cmath>

#include "device.hpp"
#include "host.hpp"
#include "model.hpp"

namespace inla {

// Solve L^T x = x in place for a lower-triangular L (column-major, order np, a
// multiple of 64) in 64-row blocks from the bottom.  For each block: the 64
// dot products with the already solved tail (coalesced column reads, 16 columns
// per wave), then a 64-step substitution in wave 0 against the block staged in
// LDS (D, 64 x 65 doubles).  Global writes to x are made visible to the other
// waves of the workgroup by the barriers.
template <typename T>
__device__ void trsv_lt_block(const T *__restrict__ L, int ld, int np, double *x, double *sred, double (*D)[65]) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int i0 = np - 64; i0 >= 0; i0 -= 64) {
    double acc[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = 0.0;
    const T *Lc = L + (size_t)(i0 + 16 * w) * ld;
    for (int j = i0 + 64 + lane; j < np; j += 64) {
      const double xj = x[j];
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[q] += (double)Lc[(size_t)q * ld + j] * xj;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const double s = wave_sum(acc[q]);
      if (lane == 0) sred[16 * w + q] = s;
    }
    for (int e = tid; e < 64 * 64; e += 256) {
      const int r = e & 63, c = e >> 6;
      D[r][c] = (double)L[(size_t)(i0 + c) * ld + i0 + r];
    }
    __syncthreads();
    if (w == 0) {
      double rhs = x[i0 + lane] - sred[lane];
      double xm = 0.0;
      for (int i = 63; i >= 0; --i) {
        const double xi = __shfl(rhs, i, 64) / D[i][i];
        if (lane == i) xm = xi;
        if (lane < i) rhs -= D[i][lane] * xi;
      }
      x[i0 + lane] = xm;
    }
    __syncthreads();
  }
}

// Solve L x = x in place (forward substitution), same blocking from the top.
// The block's rows against the solved head: thread (row i, column phase p)
// sums columns j = p, p+4, ... (each column read is 64 contiguous values).
template <typename T>
__device__ void trsv_l_block(const T *__restrict__ L, int ld, int np, double *x, double *sred4, double (*D)[65]) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int i0 = 0; i0 < np; i0 += 64) {
    double s = 0.0;
#pragma unroll 8
    for (int j = w; j < i0; j += 4) s += (double)L[(size_t)j * ld + i0 + lane] * x[j];
    sred4[w * 64 + lane] = s;
    for (int e = tid; e < 64 * 64; e += 256) {
      const int r = e & 63, c = e >> 6;
      D[r][c] = (double)L[(size_t)(i0 + c) * ld + i0 + r];
    }
    __syncthreads();
    if (w == 0) {
      double rhs = x[i0 + lane] - ((sred4[lane] + sred4[64 + lane]) + (sred4[128 + lane] + sred4[192 + lane]));
      double xm = 0.0;
      for (int c = 0; c < 64; ++c) {
        const double xc = __shfl(rhs, c, 64) / D[c][c];
        if (lane == c) xm = xc;
        if (lane > c) rhs -= D[lane][c] * xc;
      }
      x[i0 + lane] = xm;
    }
    __syncthreads();
  }
}

// Vector selectors for the step-wise triangular solves (V_* in model.hpp).
__device__ __forceinline__ double *vsel(const ThetaDesc &t, int v) {
  return v == V_X ? t.x : v == V_R ? t.r : v == V_XN ? t.xn : v == V_Z ? t.z : t.u;
}

// y = M v or y = M^T v for a 64 x 64 block M stored column-major at Mg
// (element (m, c) at Mg[c * 64 + m]).  block64_load reads the block into
// registers, lane m of wave w holding row m of columns 16w .. 16w + 15 (each
// load 64 contiguous elements of one column), so that the caller can issue it
// ahead of other work; neither product stages the block in LDS, which keeps
// the solve steps' LDS at a few KB.
template <typename T>
__device__ __forceinline__ void block64_load(const T *__restrict__ Mg, T (&e)[16]) {
  const auto *g = gptr(Mg);
  const int m = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < 16; ++q) e[q] = g[(16 * w + q) * 64 + m];
}

// The lanes of a double moved by a DPP control (within rows of 16 lanes).
template <int CTRL> __device__ __forceinline__ double dpp64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
// Sum over each row of 16 lanes, in all of them (rotations by 8, 4, 2 and 1).
__device__ __forceinline__ double row_sum16(double v) {
  v += dpp64<0x128>(v);
  v += dpp64<0x124>(v);
  v += dpp64<0x122>(v);
  v += dpp64<0x121>(v);
  return v;
}
// Sums of a and b over lanes l and l ^ 32 (H = 32) or l ^ 16: a's in the rows of 16
// lanes whose bit H is clear, b's in the others.
template <int H> __device__ __forceinline__ double fold2(double a, double b) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  u2 lo, hi;
  if (H == 32) {
    lo = __builtin_bit_cast(u2, __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false));
    hi = __builtin_bit_cast(u2, __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false));
  } else {
    lo = __builtin_bit_cast(u2, __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false));
    hi = __builtin_bit_cast(u2, __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false));
  }
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// Sums of a[0..3] over the 64 lanes: lane l returns the total of a[l >> 4].
__device__ __forceinline__ double wave_sum4(const double *a) {
  return row_sum16(fold2<16>(fold2<32>(a[0], a[2]), fold2<32>(a[1], a[3])));
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
// 16384, 10.4 and 8.9 us at 1024 with six matrices (steps of 64: 4.2 us each and
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

// Forward solve of the diagonal block at row i0 (nsub sub-blocks of 64): z to the
// global vector.  acc holds the wave's sums over earlier columns for the block's rows
// 4 l .. 4 l + 3.  Loads run AHEAD sub-blocks ahead and have no conditions: sub-blocks
// and rows are clamped to the block, and values above the diagonal are not used.
template <typename T, typename P>
__device__ __forceinline__ void solve_block_fwd(const ThetaDesc &t, int i0, int nsub, P r, double (&acc)[4], P z,
                                                double *part) {
  constexpr int AHEAD = sizeof(T) == 4 ? 3 : 1;
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q4 = l >> 4;
  const auto *L = gptr((const T *)t.W) + (size_t)(i0 + 4 * w) * t.ldw + i0;
  const unsigned lr = min(4 * l, 64 * nsub - 4);
  const auto *X = gptr((const T *)t.linv) + (size_t)(i0 / 64) * 4096 + 4 * w * 64;
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
      for (int q = 0; q < 4; ++q) load4(lo[b][q], L + (size_t)(64 * bc + q) * t.ldw + lr);
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
__device__ __forceinline__ void solve_block_bwd(const ThetaDesc &t, int i0, int nsub, P r, double (&acc)[4][4], P x,
                                                double *part) {
  constexpr int AHEAD = sizeof(T) == 4 ? 3 : 1;
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q4 = l >> 4;
  const auto *L = gptr((const T *)t.W) + (size_t)(i0 + 4 * w) * t.ldw + i0;
  const auto *X = gptr((const T *)t.linv) + (size_t)(i0 / 64) * 4096 + 4 * w * 64;
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
      for (int q = 0; q < 4; ++q) lo[b][s][q] = (L + (size_t)(64 * min(s, bc) + q) * t.ldw + 64 * bc)[(unsigned)l];
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

// One step of the forward solve L z = r (blocks from the top); i0 < 0: only the first
// block's solve.  On entry the block's solution is in z.  The rows below are updated,
// r_j -= sum_c L[j][i0 + c] z_c: wave w takes the columns 16 w .., its lanes four rows
// each in 16-byte loads.
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
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (i0 >= 0) {
    constexpr int U = sizeof(T) == 4 ? 16 : 8;   // loads in flight before the first product
    const double zv = z[i0 + 16 * w + (l & 15)];
    const auto *L = gptr((const T *)t.W) + (size_t)(i0 + 16 * w) * t.ldw + j0;
    const unsigned lr = min(4 * l, nn - 4);
#pragma unroll
    for (int c0 = 0; c0 < 16; c0 += U) {
      T lv[U][4];
#pragma unroll
      for (int c = 0; c < U; ++c) load4(lv[c], L + (size_t)(c0 + c) * t.ldw + lr);
#pragma unroll
      for (int c = 0; c < U; ++c) {
        const double zc = lane_value(zv, c0 + c);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += (double)lv[c][k] * zc;
      }
    }
  }
  if (blockIdx.x == 0) {   // the next block
    solve_block_fwd<T>(t, j0, nn / 64, r, acc, z, part);
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
// r_j -= sum_m L[i0 + m][j] x_m: wave w takes columns 64 s + 4 w + q of a workgroup's
// 256 with its lanes on four contiguous rows each.  A matrix whose last block is the
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
  double acc[4][4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[s][q] = 0.0;
  if (nb > 0) {
    constexpr int U = sizeof(T) == 4 ? 4 : 2;   // groups of four columns in flight
    const unsigned m = min(4 * l, nb - 4);
    double xv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) xv[k] = 4 * l < nb ? x[i0 + m + k] : 0.0;
    const auto *L = gptr((const T *)t.W) + (size_t)(j0 + 4 * w) * t.ldw + i0;
#pragma unroll
    for (int s0 = 0; s0 < 4; s0 += U) {
      T lv[U][4][4];
#pragma unroll
      for (int s = 0; s < U; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q) load4(lv[s][q], L + (size_t)(64 * (s0 + s) + q) * t.ldw + m);
#pragma unroll
      for (int s = 0; s < U; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc[s0 + s][q] = ((double)lv[s][q][0] * xv[0] + (double)lv[s][q][1] * xv[1]) +
                           ((double)lv[s][q][2] * xv[2] + (double)lv[s][q][3] * xv[3]);
      __builtin_amdgcn_sched_barrier(0);   // the next group's loads stay behind: registers
    }
  }
  if (blockIdx.x == 0) {   // the block above
    solve_block_bwd<T>(t, j0, nn / 64, r, acc, x, part);
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

// A Newton step taken in correction form starts its new iterate at the current
// one (xn <- x); one refinement step then adds the constrained correction.
__global__ __launch_bounds__(256) void restart_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < t.n_pad) t.xn[i] = t.x[i];
}

// Accept the refined iterate: Newton stopping quantities and x <- xn.
__global__ __launch_bounds__(256) void newton_accept_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.x];
  __shared__ double sh[4];
  double st = 0.0, sc = 0.0, bad = 0.0;
  for (int i = threadIdx.x; i < t.n; i += 256) {
    const double xn = t.xn[i], xo = t.x[i];
    if (!isfinite(xn)) bad = 1.0;
    st = fmax(st, fabs(xn - xo));
    sc = fmax(sc, fabs(xn));
  }
  st = block_max256(st, sh);
  sc = block_max256(sc, sh);
  bad = block_sum256(bad, sh);
  for (int i = threadIdx.x; i < t.n_pad; i += 256) t.x[i] = i < t.n ? t.xn[i] : 0.0;
  if (threadIdx.x == 0) {
    t.dres[DRES_STEP] = st;
    t.dres[DRES_SCALE] = fmax(1.0, sc);
    if (bad > 0.0) t.dres[DRES_NONFINITE] = 1.0;
  }
}

// Kriging solve after the small (FP64) factorisation: w from the border row,
// then lambda = L_S^{-T} w; also log|S| = 2 sum log (L_S)_ii, ||w||^2 and the
// numerical-rank flag.
__global__ __launch_bounds__(256) void kriging_solve_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.x];
  __shared__ double sred[64];
  __shared__ double sh[4];
  __shared__ double D[64][65];
  const int kp = t.k_pad, k = t.k;
  double lds_ = 0.0, w2 = 0.0, dmin = INFINITY, dmax = 0.0;
  for (int i = threadIdx.x; i < kp; i += 256) {
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
  lds_ = block_sum256(lds_, sh);
  w2 = block_sum256(w2, sh);
  dmin = -block_max256(-dmin, sh);
  dmax = block_max256(dmax, sh);
  trsv_lt_block<double>(t.S, t.lds, kp, t.lam, sred, D);
  if (threadIdx.x == 0) {
    t.dres[DRES_LOGDET_S] = 2.0 * lds_;
    t.dres[DRES_WNORM2] = w2;
    // squared pivot below 1e-13 of the largest: numerically dependent constraints
    t.dres[DRES_RANK] = (k > 0 && !(dmin >= 1e-13 * dmax)) ? 1.0 : 0.0;
  }
}

// r_c = z_c - sum_a lambda_a (G L^{-T})_{a,c}.  Newton (from_z = 0): z is the
// factored b row and lambda the kriging multipliers, giving the corrected
// right-hand side of x = L^{-T}(L^{-1} b - L^{-1} C^T lambda).  Refinement
// (from_z = 1): u = L^{-1} r1 and lambda = dlambda.
template <typename T>
__global__ __launch_bounds__(256) void rhs_kernel(const ThetaDesc *__restrict__ td, int from_z) {
  const ThetaDesc t = td[blockIdx.y];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c0 = blockIdx.x * 64 + w * 16;
  if (c0 >= t.n_pad) return;
  const int k = t.k, np = t.n_pad;
  const double *lam = from_z ? t.dlam : t.lam;
  for (int q = 0; q < 16; ++q) {
    const int c = c0 + q;
    const T *col = (const T *)t.W + (size_t)c * t.ldw + np;
    double s = 0.0;
    for (int a = lane; a < k; a += 64) s += lam[a] * (double)col[a];
    s = wave_sum(s);
    if (lane == 0) t.r[c] = (from_z ? t.u[c] : (double)col[k]) - s;
  }
}

// Refinement, constrained part 1: t = (L^{-1} C^T)^T u - r2 = C Q~^{-1} r1 - r2 with
// u = L^{-1} r1, into dlam.  A workgroup per 64 border rows; the four waves split
// the columns, each column read is 64 contiguous border values.
template <typename T>
__global__ __launch_bounds__(256) void border_gemv_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int a = blockIdx.x * 64 + (threadIdx.x & 63), w = threadIdx.x >> 6;
  __shared__ double part[4][64];
  if ((int)blockIdx.x * 64 >= t.k_pad) return;
  const int np = t.n_pad;
  double s = 0.0;
  if (a < t.k) {
    const T *row = (const T *)t.W + np + a;
#pragma unroll 8
    for (int c = w; c < np; c += 4) s += (double)row[(size_t)c * t.ldw] * t.u[c];
  }
  part[w][threadIdx.x & 63] = s;
  __syncthreads();
  if (w == 0) {
    const int l = threadIdx.x;
    t.dlam[a] = a < t.k ? ((part[0][l] + part[1][l]) + (part[2][l] + part[3][l])) - t.rtwo[a] : 0.0;
  }
}

// Refinement, constrained part 2: dlambda = S~^{-1} t with the FP64 kriging factor.
__global__ __launch_bounds__(256) void kriging_correct_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.x];
  __shared__ double sred4[256];
  __shared__ double D[64][65];
  if (t.k_pad > 0) {
    trsv_l_block<double>(t.S, t.lds, t.k_pad, t.dlam, sred4, D);
    trsv_lt_block<double>(t.S, t.lds, t.k_pad, t.dlam, sred4, D);
  }
}

// Refinement, update: xn += dx (dx in u), lambda += dlambda, and the
// quantities of the refinement stopping test.
__global__ __launch_bounds__(256) void ir_update_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.x];
  __shared__ double sh[4];
  double dm = 0.0, xm = 0.0, bad = 0.0;
  for (int i = threadIdx.x; i < t.n_pad; i += 256) {
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
  for (int a = threadIdx.x; a < t.k; a += 256) t.lam[a] += t.dlam[a];
  dm = block_max256(dm, sh);
  xm = block_max256(xm, sh);
  bad = block_sum256(bad, sh);
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
__global__ __launch_bounds__(256) void var_norms_kernel(const ThetaDesc *__restrict__ td) {
  const ThetaDesc t = td[blockIdx.y];
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= t.n) return;
  const int np = t.n_pad, kp = t.k_pad;
  const double *row = (const double *)t.W + np + kp + i;
  double s = 0.0;
  for (int c = 0; c < np; ++c) { const double v = row[(size_t)c * t.ldw]; s += v * v; }
  double s2 = 0.0;
  if (t.k > 0) {
    const double *row2 = t.S + kp + i;
    for (int c = 0; c < t.k; ++c) { const double v = row2[(size_t)c * t.lds]; s2 += v * v; }
  }
  t.out[i] = s - s2;
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
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] { hipLaunchKernelGGL(kriging_solve_kernel, dim3(B), dim3(256), 0, ctx.stream, dtd); });
}
void launch_rhs(Ctx &ctx, const ThetaDesc *dtd, int B, int np_max, int from_z, int prec) {
  if (B <= 0 || np_max <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
    INLA_DISPATCH_T(prec, rhs_kernel, dim3((np_max + 63) / 64, B), dim3(256), 0, ctx.stream, dtd, from_z);
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
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] { hipLaunchKernelGGL(newton_accept_kernel, dim3(B), dim3(256), 0, ctx.stream, dtd); });
}
void launch_ir_correct(Ctx &ctx, const ThetaDesc *dtd, int B, int kp_max, int prec) {
  if (B <= 0) return;
  if (kp_max > 0)
    ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] {
      INLA_DISPATCH_T(prec, border_gemv_kernel, dim3(kp_max / 64, B), dim3(256), 0, ctx.stream, dtd);
    });
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] { hipLaunchKernelGGL(kriging_correct_kernel, dim3(B), dim3(256), 0, ctx.stream, dtd); });
}
void launch_ir_update(Ctx &ctx, const ThetaDesc *dtd, int B) {
  if (B <= 0) return;
  ctx.launch(INLA_K_SOLVE, 0.0, 0.0, [&] { hipLaunchKernelGGL(ir_update_kernel, dim3(B), dim3(256), 0, ctx.stream, dtd); });
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
    hipLaunchKernelGGL(var_norms_kernel, dim3((np_max + 255) / 256, B), dim3(256), 0, ctx.stream, dtd);
  });
}

}  // namespace inla
