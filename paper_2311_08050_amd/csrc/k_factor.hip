// Bordered, batched, blocked Cholesky for gfx950.
//
// Dense Cholesky is the step the paper names as the bottleneck of every
// hyperparameter evaluation (section "Implementation of INLA+: OpenMP and MPI
// parallelization"; 3-5 factorisations per evaluation in section "Running INLA+
// on multiple nodes").  Here each theta of a batch owns one column-major matrix;
// every launch processes the same step of all of them.
//
// A matrix is [[Q, .], [G, D]] with G the border rows; factoring the first nf
// columns leaves L (Q = L L^T), G L^{-T} in the border rows and D - G Q^{-1} G^T
// in the Schur block.  Border rows carry the constraint rows C and the Newton
// right-hand side b, so C Q^{-1} C^T, C Q^{-1} b and L^{-1} b fall out of the
// factorisation's own MFMA updates.
//
// Per outer panel [p0, pend = p0 + nb), left-looking inside the panel and
// right-looking across panels:
//   potf2_inv  : L_pp = chol(A_pp) and X = L_pp^{-1} in FP64 in LDS for the first
//                diagonal block (one workgroup per theta)
//   panel step : per 64-wide block column j, per 64-row tile I below it
//                L[I,j] = (A[I,j] - L[I,p0:j] L[j,p0:j]^T) X_j^T, the SYRK of the
//                in-panel diagonal block A[I,I], and chol / inverse of the next
//                diagonal block by the tile just below (MFMA, one launch per j)
//   TRAIL      : A[pend:, pend:ncols] -= A[pend:, p0:pend] A[pend:ncols, p0:pend]^T
// Blocked right-looking Cholesky is the textbook form; the left-looking panel
// and the fused diagonal factorisation are this implementation's choice.
//
// Storage and MFMA precision are template parameters: FP64 storage with
// v_mfma_f64_16x16x4f64, or FP32 storage with v_mfma_f32_16x16x4f32 (FP32
// accumulate).  Operands are LDS-staged in double-buffered K chunks.
#include <limits>
#include <type_traits>

#include "device.hpp"
#include "host.hpp"

namespace inla {

// TRAIL updates everything right of the panel; with lookahead it is split into
// TRAIL_A (the next panel's columns) and TRAIL_B (the columns after it), so
// that the next panel can be factored while TRAIL_B runs.
enum { KIND_TRAIL = 0, KIND_TRAIL_A = 1, KIND_TRAIL_B = 2 };

typedef float f4 __attribute__((ext_vector_type(4)));

// --------------------------------------------------------------------------
// Diagonal block: Cholesky of the 64 x 64 block A_jj and its inverse in one
// LDS-resident FP64 pass of 34 KB: L_jj overwrites the lower triangle and
// X = L_jj^{-1} (lower triangular) is built in the strict upper triangle,
// transposed, with its diagonal 1 / L_cc kept apart.
//
// Bound by a serial chain (64 pivots), so everything that is not the chain is
// taken off it.  By 16-wide sub-panels J:
//  1. Wave 0 eliminates in registers.  Lane p stands for row p of the block; its
//     column b[] of 16 values is what the row operations on the sub-panel's
//     diagonal block turn into a result: for rows below the block their L, for
//     rows above it the inverse's entries of the sub-panel, for the block's own
//     rows (identity columns) its inverse.  Every group of 16 lanes also holds
//     the diagonal block itself (column q in lane q), so that a multiplier is one
//     broadcast inside the group.  Per pivot one reciprocal; the column scalings
//     1 / sqrt(d_c) follow after the last pivot.
//  2. The rank-16 update of everything below, of the matrix and of the inverse's
//     rows alike: the lower 16 x 16 blocks (I, C), I > J, as FP64 MFMA products
//     of the sub-panel's rows; block (I, C) with C <= J is the inverse's.  The
//     four blocks that the next sub-panel reads come first, one per wave; waves
//     1 .. 3 do the others while wave 0 eliminates the next sub-panel.
// One block of potf2_inv_kernel takes 14.5 us (35.4 us with substitution per
// column, rank-16 updates in vector arithmetic and the inverse by blocks after the
// factor); about 5,700 cycles per sub-panel, 2,300 of them the elimination.
// --------------------------------------------------------------------------
struct Potf2Lds {
  double M[NBI][NBI + 1];   // lower: the block, then L; strict upper: X[a][b] at M[b][a] (a > b).  On entry
                            // the 16 x 16 diagonal blocks are whole (symmetric), the rest above zero
  double rd[NBI];           // reciprocal pivots 1 / L_cc = X[c][c]
  int fail;
};

// Lane C of each group of 16 lanes, broadcast in the group.
template <int C> __device__ __forceinline__ double row_lane(double v) {
  const long long b = __double_as_longlong(v);
  return __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, b, 0x150 + C, 0xf, 0xf, true));
}

// X = L^{-1} element (a, b), a >= b, from its packed place.
__device__ __forceinline__ double xinv(const Potf2Lds &S, int a, int b) {
  return a == b ? S.rd[a] : S.M[b][a];
}

// Elimination of the diagonal block d[] (column q in lane q of each 16-lane
// group), applied to the columns b[] as well; dv receives pivot c in lane c of
// each group.  With u = -column / pivot, row r is updated by (row r of column c) u.
// 1 / pivot is the hardware estimate x (relative error e below 2^-20) corrected
// to x (1 + e + e^2).  SAFE scales each pivot into range first (where 1 / pivot
// would overflow or lose bits).  Step C updates the rows below C with ud, ub and
// forms the next pivot's from row C + 1 as soon as that is done, so that the
// reciprocal's latency is covered by the other rows.
template <int C, bool SAFE>
__device__ __forceinline__ void potf2_ratio(const double (&d)[16], const double (&b)[16], double &dv, double &ud,
                                            double &ub) {
  double pv = row_lane<C>(d[C]), dc = d[C], bc = b[C];
  if ((threadIdx.x & 15) == C) dv = pv;
  if constexpr (SAFE) {
    const double sc = pv < 1.0 ? 0x1p600 : 0x1p-600;
    pv *= sc;
    dc *= sc;
    bc *= sc;
  }
  const double x = __builtin_amdgcn_rcp(pv);
  const double e = fma(-pv, x, 1.0), dx = -dc * x, bx = -bc * x, t = fma(e, e, e);
  ud = fma(dx, t, dx);
  ub = fma(bx, t, bx);
}
template <int C, bool SAFE>
__device__ __forceinline__ void potf2_step(double (&d)[16], double (&b)[16], double &dv, double ud, double ub) {
  if constexpr (C < 15) {
    const double m = row_lane<C>(d[C + 1]);
    d[C + 1] = fma(m, ud, d[C + 1]);
    b[C + 1] = fma(m, ub, b[C + 1]);
    double udn, ubn;
    potf2_ratio<C + 1, SAFE>(d, b, dv, udn, ubn);
#pragma unroll
    for (int r = C + 2; r < 16; ++r) {
      const double mr = row_lane<C>(d[r]);
      d[r] = fma(mr, ud, d[r]);
      b[r] = fma(mr, ub, b[r]);
      asm volatile("" : "+v"(b[r]));   // here and not after the last pivot, with every multiplier kept until then
      if (r == 8) __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_sched_barrier(0);   // one step's multipliers in registers at a time
    potf2_step<C + 1, SAFE>(d, b, dv, udn, ubn);
  }
}
template <bool SAFE> __device__ __forceinline__ void potf2_eliminate(double (&d)[16], double (&b)[16], double &dv) {
  double ud, ub;
  potf2_ratio<0, SAFE>(d, b, dv, ud, ub);
  potf2_step<0, SAFE>(d, b, dv, ud, ub);
}

// Rows c of both column sets scaled by 1 / sqrt(pivot c) (rs of lane c).
template <int C> __device__ __forceinline__ void potf2_scale(double (&d)[16], double (&b)[16], double rs) {
  if constexpr (C < 16) {
    const double f = row_lane<C>(rs);
    d[C] *= f;
    b[C] *= f;
    potf2_scale<C + 1>(d, b, rs);
  }
}

// Block (I, C) of the update by sub-panel J: block -= P_I P_C^T over its 16
// columns, P_p = M[p][16 J ..] (for the sub-panel's own rows: its diagonal
// block's inverse).  One wave; I, C and J are uniform.
__device__ __forceinline__ void potf2_block(Potf2Lds &S, int I, int C, int J, int lane) {
  constexpr int W = 16, LD = NBI + 1;
  const int q = lane & (W - 1), g = lane >> 4, jb = W * J;
  double *M = &S.M[0][0];
  // element v of a lane: row g + 4 v of block row I, column q of block column C;
  // a block of the inverse is stored transposed
  const bool tr = C <= J;
  double *at = M + (tr ? (W * C + q) * LD + W * I + g : (W * I + g) * LD + W * C + q);
  const int step = tr ? 4 : 4 * LD;
  const double *PI = M + (W * I + q) * LD + jb + g, *PC = M + (W * C + q) * LD + jb + g;
  double pi[4], pc[4];
  d4 acc;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    pi[s] = PI[4 * s];
    pc[s] = PC[4 * s];
  }
  const double xd = S.rd[jb + q];
#pragma unroll
  for (int v = 0; v < 4; ++v) acc[v] = at[v * step];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = 4 * s + g;
    const double own = k > q ? pc[s] : k == q ? xd : 0.0;
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-pi[s], C == J ? own : pc[s], acc, 0, 0, 0);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) at[v * step] = acc[v];
}

// Element (r, c) of the block to factor into its place (and its mirror image
// inside a diagonal 16 x 16 block); elements above the diagonal are ignored.
__device__ __forceinline__ void potf2_put(Potf2Lds &S, int r, int c, double v) {
  if (r >= c) {
    S.M[r][c] = v;
    if ((r ^ c) < 16) S.M[c][r] = v;
  } else if ((r ^ c) >= 16) {
    S.M[r][c] = 0.0;
  }
}

// Sub-panel J of the factored block: columns 16 J .. of L over the lower triangle
// at Ad (column-major, ld), rows 16 J .. of the inverse into its slot Li.  Threads
// [0, nthr).
template <typename T>
__device__ __forceinline__ void potf2_store(const Potf2Lds &S, int J, __attribute__((address_space(1))) T *Ad, int ld,
                                            __attribute__((address_space(1))) T *Li, int thr, int nthr) {
  constexpr int W = 16;
#pragma unroll 1
  for (int e = thr; e < W * NBI; e += nthr) {
    const int r = e & (NBI - 1), c = W * J + (e >> 6);
    if (r >= c) Ad[(size_t)c * ld + r] = (T)S.M[r][c];
    const int xr = W * J + (e & (W - 1)), xc = e >> 4;
    Li[xc * NBI + xr] = (T)(xr >= xc ? xinv(S, xr, xc) : 0.0);   // column-major (L^{-1})[r][c]
  }
}

// The block is in S.M (potf2_put), S.fail is 0; all of it visible to the block.
// On return the lower triangle holds L_jj, the upper triangle and S.rd the
// inverse, S.fail the first failing pivot (1-based) or 0; L_jj and the inverse are
// written to their places (j: the block's first column) and a failing pivot to
// d.info.  Waves 1 .. 3 store a finished sub-panel while wave 0 eliminates the next.
template <typename T>
__device__ __forceinline__ void potf2_factor_invert(Potf2Lds &S, const FactorDesc &d, int j,
                                                    __attribute__((address_space(1))) T *Ad, int tid) {
  constexpr int W = 16, NJ = NBI / W, LD = NBI + 1;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  __attribute__((address_space(1))) T *Li = gptr((T *)d.linv) + (size_t)(j / NBI) * NBI * NBI;
  double *M = &S.M[0][0];
#pragma unroll 1
  for (int J = 0; J < NJ; ++J) {
    const int jb = J * W;
    int lane = tid & 63;
    asm volatile("" : "+v"(lane));   // addresses are formed again for each J: kept, they would be spilled
    const int q = lane & (W - 1);
    if (w == 0) {
      const bool own = (lane >> 4) == J;   // the diagonal block's rows
      double d[W], b[W], dv = 1.0;
      auto load = [&] {
#pragma unroll
        for (int r = 0; r < W; ++r) {
          d[r] = M[(jb + q) * LD + jb + r];
          const double m = M[lane * LD + jb + r];
          b[r] = own ? (r == q ? 1.0 : 0.0) : m;
        }
      };
      load();
      potf2_eliminate<false>(d, b, dv);
      if (__any(!(dv > 0x1p-900 && dv < 0x1p900))) {
        load();
        potf2_eliminate<true>(d, b, dv);
        // (an infinite pivot shows in the pivots after it, the block's last in none)
        const bool inf_last = J == NJ - 1 && q == W - 1 && dv > 0x1.fffffffffffffp1023;
        const unsigned long long neg = __ballot(!(dv > 0.0) || inf_last);
        if (neg && lane == 0 && S.fail == 0) S.fail = jb + __ffsll(neg);
      }
      double sq, rs;
      sqrt_rsqrt(dv, sq, rs);   // not a number for a negative pivot
      potf2_scale<0>(d, b, rs);
      // the block's own rows hold L up to their diagonal and the inverse beyond it
      const int upto = own ? q : -1;
#pragma unroll
      for (int r = 0; r < W; ++r) M[lane * LD + jb + r] = r <= upto ? d[r] : b[r];
      if (own) S.rd[lane] = rs;
    } else {
      if (J == 1) {
        if (w == 3) {
          potf2_block(S, 3, 3, 0, lane);
        } else {
          potf2_block(S, w + 1, 0, 0, lane);
          potf2_block(S, w + 1, 2, 0, lane);
        }
      } else if (J == 2) {
        potf2_block(S, 3, w == 3 ? 3 : w - 1, 1, lane);
      }
      if (J > 0) potf2_store<T>(S, J - 1, Ad, d.ld, Li, 64 * (w - 1) + lane, 192);
    }
    __syncthreads();
    if (J + 1 < NJ) {
      potf2_block(S, max(w, J + 1), min(w, J + 1), J, lane);
      __syncthreads();
    }
  }
  potf2_store<T>(S, NJ - 1, Ad, d.ld, Li, tid, 256);
  if (tid == 0 && S.fail != 0 && *d.info == 0) *d.info = j + S.fail;
}

// Block column j is padding: its diagonal block is the identity, and so is the inverse.
template <typename T> __device__ __forceinline__ void identity_inverse(const FactorDesc &d, int j, int tid) {
  auto *Li = gptr((T *)d.linv) + (size_t)(j / NBI) * NBI * NBI;
  for (int e = tid; e < NBI * NBI; e += 256) Li[e] = (T)(e / NBI == e % NBI ? 1 : 0);
}

template <typename T>
__global__ __launch_bounds__(256) void potf2_inv_kernel(const FactorDesc *__restrict__ descs, int j) {
  const FactorDesc d = descs[blockIdx.x];
  if (j >= d.nf) return;
  __shared__ Potf2Lds S;
  const int tid = threadIdx.x;
  __attribute__((address_space(1))) T *Ad = gptr((T *)d.A) + (size_t)j * d.ld + j;
  // all 16 loads in flight before the first LDS store
  T v[NBI * NBI / 256];
#pragma unroll
  for (int i = 0; i < NBI * NBI / 256; ++i) {
    const int e = tid + 256 * i;
    v[i] = Ad[(size_t)(e >> 6) * d.ld + (e & (NBI - 1))];
  }
#pragma unroll
  for (int i = 0; i < NBI * NBI / 256; ++i) {
    const int e = tid + 256 * i, r = e & (NBI - 1), c = e >> 6;
    potf2_put(S, r, c, (double)v[i]);
  }
  if (tid == 0) S.fail = 0;
  __syncthreads();
  potf2_factor_invert<T>(S, d, j, Ad, tid);
}

// XCD-aware workgroup order.  The hardware hands the workgroup with linear id
// L to XCD L % 8, and each XCD has its own L2; remapped, XCD k walks the
// contiguous range [k N/8, (k+1) N/8) of (theta, tile) pairs, so workgroups
// that run side by side on one XCD work on neighbouring tiles of one theta and
// share panel blocks in its L2.  The grid size N must be a multiple of 8.
__device__ __forceinline__ void xcd_order(int &bx, int &by) {
  const int N = gridDim.x * gridDim.y;
  const int L = blockIdx.y * gridDim.x + blockIdx.x;
  const int G = (L & 7) * (N >> 3) + (L >> 3);
  by = G / gridDim.x;
  bx = G - by * gridDim.x;
}

// Tile t of a lower trapezoid of nr tile rows and nc <= nr tile columns (tile
// (I, J) present when J <= I), in groups of GR tile rows, column by column
// within a group: consecutive tiles share their column block, and a group's GR
// row blocks stay in L2 while its columns go by.  Returns false past the end.
__device__ __forceinline__ bool trap_grouped(int t, int nr, int nc, int &I, int &J) {
  constexpr int GR = 8;
  auto before = [&](int r) {   // tiles in rows [0, r)
    const int m = min(r, nc);
    return m * (m + 1) / 2 + max(0, r - nc) * nc;
  };
  if (t >= before(nr)) return false;
  int lo = 0, hi = (nr + GR - 1) / GR - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (before(mid * GR) <= t) lo = mid;
    else hi = mid - 1;
  }
  const int r0 = lo * GR, gh = min(GR, nr - r0);
  int u = t - before(r0);
  const int full = min(r0, nc);   // columns left of the group's diagonal: gh tiles each
  if (u < full * gh) {
    J = u / gh;
    I = r0 + u % gh;
    return true;
  }
  u -= full * gh;
  J = r0;                         // column J >= r0 holds rows J .. r0 + gh - 1
  while (u >= r0 + gh - J) {
    u -= r0 + gh - J;
    ++J;
  }
  I = J + u;
  return true;
}

// Tile bx of one trailing-update launch: rows/columns of the C tile and the K
// range [ks, ke) = [p0, pend), the lower-triangular tiles of the updated block
// in the grouped order of trap_grouped.  Returns false when the workgroup has
// no tile, its tile reads identity border rows (or columns) that are still
// zero over [ks, ke), or the row selection excludes it (sel: 0 every tile,
// 1 tiles of the factored rows (row < nf), 2 tiles of the border rows
// (row >= nf)).
__device__ __forceinline__ bool update_tile(const FactorDesc &d, int kind, int p0, int nb, int TM, int TN, int sel,
                                            int bx, int &row0, int &col0, int &ks, int &ke) {
  if (p0 >= d.nf) return false;
  const int pend = min(p0 + nb, d.nf);
  int r0, c0, cend;
  ks = p0; ke = pend;
  if (kind == KIND_TRAIL) {
    r0 = pend; c0 = pend; cend = d.ncols;
  } else if (kind == KIND_TRAIL_A) {
    r0 = pend; c0 = pend; cend = min(pend + nb, d.nf);
  } else {
    c0 = min(pend + nb, d.nf); r0 = c0; cend = d.ncols;
  }
  if (r0 >= d.nrows || c0 >= cend) return false;
  // (the border rows' tiles are numbered by themselves: as the last of all tiles they
  // were one XCD's work per theta, 178 us where 64 do for two of order 16384)
  if (sel == 2) {
    const int nb_rows = (d.nrows - d.nf) / TM, nc = (cend - c0) / TN;
    if (bx >= nb_rows * nc) return false;
    row0 = d.nf + bx % nb_rows * TM;
    col0 = c0 + bx / nb_rows * TN;
    if (col0 > row0) return false;
  } else {
    const int nr = (d.nrows - r0) / TM;
    int I, J;
    if (!trap_grouped(bx, nr, (cend - c0) / TN, I, J)) return false;
    row0 = r0 + I * TM;
    col0 = c0 + J * TN;
    if (sel == 1 && row0 >= d.nf) return false;
  }
  if (row0 >= d.id_row0 && row0 - d.id_row0 >= ke) return false;
  if (col0 >= d.id_row0 && col0 - d.id_row0 >= ke) return false;
  return true;
}

// C -= acc for one wave's BM x BN accumulator blocks (tile coordinates from rl,
// cl).  A tile that straddles the diagonal touches only its lower triangle.
template <typename T, int BM, int BN, typename Acc, typename RL, typename CL>
__device__ __forceinline__ void subtract_tile(__attribute__((address_space(1))) T *Cg, int ld, Acc (&acc)[BM][BN],
                                              RL rl, CL cl, bool diag_tile, int row0, int col0) {
  if (!diag_tile) {
#pragma unroll
    for (int a = 0; a < BM; ++a) {
      T cv[BN][4];
#pragma unroll
      for (int b = 0; b < BN; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) cv[b][v] = Cg[(size_t)cl(b, v) * ld + rl(a, v)];
#pragma unroll
      for (int b = 0; b < BN; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) Cg[(size_t)cl(b, v) * ld + rl(a, v)] = cv[b][v] - acc[a][b][v];
    }
  } else {
#pragma unroll
    for (int a = 0; a < BM; ++a)
#pragma unroll
      for (int b = 0; b < BN; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (row0 + rl(a, v) >= col0 + cl(b, v)) {
            __attribute__((address_space(1))) T *p = Cg + (size_t)cl(b, v) * ld + rl(a, v);
            *p = *p - acc[a][b][v];
          }
        }
  }
}

// --------------------------------------------------------------------------
// MFMA tile update.  C(TM x TN) = or -= A(TM x K) B(TN x K)^T, A and B read from
// column-major storage (element (r, k) at base[k*ld + r]).
//
// FP64: v_mfma_f64_16x16x4f64 puts D row (l/16 + 4v), column (l%16) in lane l;
// the operands are swapped (x from B, y from A) so that a lane's four results
// are C row (l%16) of columns (l/16 + 4v) and every store covers four whole
// 128-byte column segments.
// FP32: v_mfma_f32_16x16x4f32 puts D rows (4(l/16) + v), column (l%16) in lane
// l; operands are not swapped, so a lane's four results are four consecutive
// rows of one column.
// Lane group g = l/16 supplies k = 4g + s at MFMA step s of each 16-deep
// sub-chunk.  LDS rows are padded by 4 elements so that each read is free of
// bank conflicts.
// --------------------------------------------------------------------------
// Elements of a tile through a buffer resource: a uniform base, one 32-bit lane
// offset for the whole tile and a scalar offset per access (both in bytes), where
// 64-bit addresses would hold two registers per element over the kernel's length.
// The resource spans 2 GB from the base (a 64-column tile ends well before that).
template <typename T> struct TileBuf {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ explicit TileBuf(const void *base)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, 0x7fffffff, 0x00020000)) {}
  __device__ __forceinline__ T load(unsigned lane_off, unsigned off) const {
    if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, lane_off, off, 0));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, lane_off, off, 0));
  }
  template <typename V> __device__ __forceinline__ V load16(unsigned lane_off, unsigned off) const {
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, 0));
  }
  __device__ __forceinline__ void store(T v, unsigned lane_off, unsigned off) const {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    if constexpr (sizeof(T) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, lane_off, off, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, lane_off, off, 0);
  }
};

// SEL (row selection of update_tile) is a template parameter so that the
// border-row launch beside a BF16 trailing update is a kernel of its own; the
// trailing update of every row is trail_update_kernel (below), so that each
// launch class has its own kernel symbol.
template <typename T, int TM, int TN, int SEL, int NBUF>
__device__ __forceinline__ void gemm_update_body(const FactorDesc *__restrict__ descs, int kind, int p0, int nb) {
  constexpr bool F64 = sizeof(T) == 8;
  // K chunk staged per LDS buffer: 16 deep in both precisions, which keeps a
  // 128 x 128 FP32 tile's buffers at 34 KB (up to four workgroups per CU)
  constexpr int KCH = 16;
  constexpr int VEC = 16 / sizeof(T);           // elements per 16-byte global load
  constexpr int WM = 2, WN = 2;                 // 2 x 2 waves
  constexpr int WTM = TM / WM, WTN = TN / WN;   // wave tile
  constexpr int BM = WTM / 16, BN = WTN / 16;   // MFMA blocks per wave
  constexpr int PAD = 4;
  constexpr int LA = KCH * TM / VEC / 256, LB = KCH * TN / VEC / 256;
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  typedef __attribute__((address_space(1))) T gT;
  typedef __attribute__((address_space(1))) const T gcT;
  typedef __attribute__((address_space(1))) const vec_t gcvec;
  typedef typename std::conditional<F64, d4, f4>::type acc_t;
  static_assert(NBUF == 1 || NBUF == 2, "one or two LDS buffers");
  __shared__ __attribute__((aligned(16))) T As[NBUF][KCH][TM + PAD];
  __shared__ __attribute__((aligned(16))) T Bs[NBUF][KCH][TN + PAD];

  int bx, by;
  xcd_order(bx, by);
  const FactorDesc d = descs[by];
  int row0, col0, ks, ke;
  if (!update_tile(d, kind, p0, nb, TM, TN, SEL, bx, row0, col0, ks, ke)) return;

  const int ld = d.ld;
  const T *Ap = (const T *)d.A + (size_t)ks * ld + row0, *Bp = (const T *)d.A + (size_t)ks * ld + col0;
  gT *Cg = gptr((T *)d.A) + (size_t)col0 * ld + row0;
  const int K = ke - ks;

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w / WN, wn = w % WN;
  const int g = lane >> 4, li = lane & 15;

  acc_t acc[BM][BN];
#pragma unroll
  for (int a = 0; a < BM; ++a)
#pragma unroll
    for (int b = 0; b < BN; ++b) acc[a][b] = acc_t{0, 0, 0, 0};

  vec_t ra[LA], rb[LB];
  constexpr int KA = 256 / (TM / VEC), KB = 256 / (TN / VEC);   // columns per load of the workgroup
  const unsigned lds = ld * (unsigned)sizeof(T);
  const unsigned al = (unsigned)((tid / (TM / VEC) * ld + tid % (TM / VEC) * VEC) * sizeof(T));
  const unsigned bl = (unsigned)((tid / (TN / VEC) * ld + tid % (TN / VEC) * VEC) * sizeof(T));
  auto gload = [&](int kc) {
    const TileBuf<T> Ag(Ap + (size_t)kc * ld), Bg(Bp + (size_t)kc * ld);
#pragma unroll
    for (int it = 0; it < LA; ++it) ra[it] = Ag.template load16<vec_t>(al, it * KA * lds);
#pragma unroll
    for (int it = 0; it < LB; ++it) rb[it] = Bg.template load16<vec_t>(bl, it * KB * lds);
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int it = 0; it < LA; ++it) {
      const int lin = it * 256 + tid, kk = lin / (TM / VEC), rp = lin % (TM / VEC);
      *reinterpret_cast<vec_t *>(&As[buf][kk][VEC * rp]) = ra[it];
    }
#pragma unroll
    for (int it = 0; it < LB; ++it) {
      const int lin = it * 256 + tid, kk = lin / (TN / VEC), rp = lin % (TN / VEC);
      *reinterpret_cast<vec_t *>(&Bs[buf][kk][VEC * rp]) = rb[it];
    }
  };

  gload(0);
  lstore(0);
  __syncthreads();
  int buf = 0;
  for (int kc = 0; kc < K; kc += KCH) {
    const bool more = kc + KCH < K;
    if (more) gload(kc + KCH);
    // FP32 128 x 128 tiles: the compiler's interleaving of LDS reads with the
    // MFMA steps (scheduling only; 2% faster at four workgroups per CU, where
    // the FP64 tiles lose occupancy to it)
    if constexpr (!F64 && TM == 128) __builtin_amdgcn_iglp_opt(0);
#pragma unroll
    for (int s = 0; s < KCH / 4; ++s) {
      const int kk = 16 * (s >> 2) + 4 * g + (s & 3);
      T ya[BM], xb[BN];
#pragma unroll
      for (int a = 0; a < BM; ++a) ya[a] = As[buf][kk][wm * WTM + a * 16 + li];
#pragma unroll
      for (int b = 0; b < BN; ++b) xb[b] = Bs[buf][kk][wn * WTN + b * 16 + li];
#pragma unroll
      for (int a = 0; a < BM; ++a)
#pragma unroll
        for (int b = 0; b < BN; ++b) {
          if constexpr (F64) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xb[b], ya[a], acc[a][b], 0, 0, 0);
          else acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(ya[a], xb[b], acc[a][b], 0, 0, 0);
        }
    }
    if constexpr (NBUF == 2) {
      if (more) lstore(buf ^ 1);
      __syncthreads();
      buf ^= 1;
    } else {
      __syncthreads();   // every wave is done reading the buffer
      if (more) {
        lstore(0);
        __syncthreads();
      }
    }
  }

  // Epilogue: tile element (rl(a, v), cl(b, v)) for accumulator component v.
  auto rl = [&](int a, int v) { return wm * WTM + a * 16 + (F64 ? li : 4 * g + v); };
  auto cl = [&](int b, int v) { return wn * WTN + b * 16 + (F64 ? g + 4 * v : li); };
  subtract_tile<T, BM, BN>(Cg, ld, acc, rl, cl, row0 < col0 + TN, row0, col0);
}

// The border rows' trailing update beside a BF16 trailing update (SEL 2).
template <typename T, int TM, int TN, int SEL>
__global__ __launch_bounds__(256, 2) void gemm_update_kernel(const FactorDesc *__restrict__ descs, int kind,
                                                             int p0, int nb) {
  gemm_update_body<T, TM, TN, SEL, 2>(descs, kind, p0, nb);
}

// The trailing update of the blocked Cholesky (kinds TRAIL, TRAIL_A, TRAIL_B).
// The FP64 64 x 64 tile stages its operands through one LDS buffer (17 KB, seven
// workgroups per CU at 68 registers; two buffers at four are slower); the others
// through two.  Its loads through buffer resources, whose 64-bit forms took ten more
// registers (six workgroups): all updates of eight matrices of order 8192 86.3 to
// 82.0 ms (71 TFLOP/s, of 73 in a large library product), of nine of order 3000 11.5 to
// 11.1 ms, of 20 uneven ones 135.7 to 128.3 ms.  Held to 64 registers for eight
// workgroups it spills and takes 95.5 ms.  Matrix units 95% busy in an evaluation of 64.
template <typename T, int TM, int TN>
__global__ __launch_bounds__(256, 2) void trail_update_kernel(const FactorDesc *__restrict__ descs, int kind, int p0,
                                                              int nb) {
  gemm_update_body<T, TM, TN, 0, (sizeof(T) == 8 && TM == 64) ? 1 : 2>(descs, kind, p0, nb);
}

// The same update for a factorisation on the handle's aux stream (the
// concurrent prior pass), always with two LDS buffers: the FP64 64 x 64 tile
// then holds four workgroups per CU rather than seven, which leaves every CU
// room for the caller's stream's panel steps and solves beside it.
template <typename T, int TM, int TN>
__global__ __launch_bounds__(256, 2) void trail_update_aux_kernel(const FactorDesc *__restrict__ descs, int kind,
                                                                  int p0, int nb) {
  gemm_update_body<T, TM, TN, 0, 2>(descs, kind, p0, nb);
}

// --------------------------------------------------------------------------
// One step of the left-looking panel: block column j of the panel [p0, pend),
// one 64-row tile I (rows r0 = j + 64 (t + 1) .. r0 + 63) per workgroup:
//   C      = A[I, j] - A[I, p0:j] A[j, p0:j]^T     (the panel's earlier columns,
//                                                  MFMA from global via LDS)
//   L[I,j] = C L_jj^{-T}                           (MFMA, both operands from registers)
//   A[I,I] -= L[I,j] L[I,j]^T                      (tiles with r0 < pend: the
//                                                  diagonal block's update)
// The tile just below the diagonal block (t = 0) then holds the next diagonal
// block fully updated and factors and inverts it (potf2_factor_invert)
// in the same launch, so a panel takes one potf2_inv launch and one launch per
// block column.  Each tile reads its own rows of the panel's earlier columns
// and writes one 64 x 64 block, in place of the right-looking rank-64 updates
// that read and wrote the panel's whole trailing part once per block column.
// Every phase fits in about 34 KB of LDS, so four workgroups can share a CU.
//
// Identity border rows (rows id_row0 + s hold e_s) are zero left of column s,
// so a tile of them starts its K range at r0 - id_row0 and is skipped when
// that is past the block column.
//
// Tile 0 is the critical one, so its product is taken off it: while step j runs,
// one more workgroup per theta updates the tile that will be step j + 1's tile 0
// by the block columns before j (complete by then), which leaves that step the
// 64-deep product with block column j.
//
// Grid: act (1 + pre) + 8 Q workgroups.  The first act (one per theta) take tile 0,
// so the diagonal factorisations start first, then (pre) the next step's tiles; the
// rest take tiles 1 .. gx - 1 of every theta in the XCD-aware order of xcd_order
// (Q = ceil(act (gx - 1) / 8)).
// --------------------------------------------------------------------------
//
// Wave w owns rows 16 w .. 16 w + 15 of the tile and all 64 columns, as four
// 16 x 16 accumulator blocks whose operands are swapped in both precisions: a
// lane holds row li of the wave and columns 16 b + kcol(v) (v = 0 .. 3).  That is
// also the layout of an MFMA operand whose step v takes the sub-column kcol(v) of
// lane group g, so C goes into the TRSM, and the TRSM skips the zero half of
// L_jj^{-1}, without passing through LDS; the SYRK reads L[I,j] from LDS, only its
// ten blocks at and below the diagonal.  Bound by the chain of tile 0 (product,
// TRSM, SYRK, factorisation), in large batches by the MFMA products.  Tile 0's
// chain takes 45,000 cycles in FP64 and 40,000 in FP32 at every column, 23,000 of
// them the factorisation (65,000 and 50,000 on average with the product over the
// whole panel, and TRSM operands and results staged in 16-deep chunks before that):
// one matrix of order 1000 463 us (622), 9 of order 3000 2.82 ms (3.36).  The chunks'
// loads through buffer resources, whose offsets leave registers for a second FP64
// chunk: a step of 9 of order 3000 24.7 to 24.1 us, of two of order 16384 in FP32 20.9
// to 20.1.
template <typename T>
struct PanelLds {
  static constexpr int LDC = NBI + 4;          // LDS row length (elements): conflict-free MFMA operand reads
  static constexpr int PKC = sizeof(T) == 4 ? 32 : 16;   // K chunk of the left-looking product
  union {
    struct { T As[2][PKC][LDC]; T Bs[2][PKC][LDC]; } g;   // K chunks ([k][row])
    T Ls[NBI][LDC];                                        // L[I, j] ([k][row])
    Potf2Lds f;                                            // the next diagonal block's factorisation
  };
};

// Four workgroups per CU in FP32; three in FP64, whose registers would
// otherwise spill at the 128-register budget of four.
template <typename T>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 4 : 3) void panel_step_kernel(const FactorDesc *__restrict__ descs, int p0, int nb,
                                                            int j, int act, int gx, int Q, int pre) {
  constexpr bool F64 = sizeof(T) == 8;
  constexpr int VEC = 16 / sizeof(T);
  constexpr int LDC = PanelLds<T>::LDC, PKC = PanelLds<T>::PKC, NB = NBI / 16;
  constexpr int LA = PKC * NBI / VEC / 256;           // 16-byte loads per thread per operand chunk
  constexpr int DEPTH = F64 ? 2 : 1;                  // chunks in flight (two in FP32: no faster)
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  typedef __attribute__((address_space(1))) T gT;
  typedef __attribute__((address_space(1))) const T gcT;
  typedef typename std::conditional<F64, d4, f4>::type acc_t;
  __shared__ __attribute__((aligned(16))) PanelLds<T> S;

  int th, t;   // t = -1: the next step's tile 0 ahead of time
  {
    const int L = blockIdx.x;
    if (L < act) {
      th = L; t = 0;
    } else if (L < act * (1 + pre)) {
      th = L - act; t = -1;
    } else {
      const int L2 = L - act * (1 + pre), G = (L2 & 7) * Q + (L2 >> 3);
      if (gx <= 1 || G >= act * (gx - 1)) return;
      th = G / (gx - 1);
      t = 1 + G % (gx - 1);
    }
  }
  const FactorDesc d = descs[th];
  // Padding takes no steps: its columns keep their zeros, ones of an identity border and
  // identity block (half of all orders end in a block column of it)
  if (j >= d.ne) return;
  const int pend = min(p0 + nb, d.nf);
  const int r0 = t < 0 ? j + 2 * NBI : j + NBI * (t + 1), c0 = t < 0 ? j + NBI : j;   // tile rows and columns
  if (r0 >= (t < 0 ? pend : d.nrows)) return;
  if (r0 >= d.ne && r0 < d.nf) {   // padding rows: zero
    if (t == 0 && r0 < pend) identity_inverse<T>(d, r0, threadIdx.x);
    return;
  }
  // (the step before updated this step's tile 0 up to block column j - 64)
  int ks = t == 0 && j >= p0 + 2 * NBI && r0 < pend ? j - NBI : p0;
  if (r0 >= d.id_row0) {
    if (r0 - d.id_row0 >= j + NBI) return;   // zero in block column j: nothing to do
    ks = max(ks, r0 - d.id_row0);
  }
  const int ld = d.ld, K = j - ks;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, li = lane & 15;
  auto kcol = [&](int v) { return F64 ? g + 4 * v : 4 * g + v; };
  // ... = klane + kstep(v): a tile's element (row li of the wave, column 16 b +
  // kcol(v)) is addressed by a uniform pointer per (b, v) and one lane offset
  const int klane = F64 ? g : 4 * g;
  auto kstep = [&](int b, int v) { return 16 * b + (F64 ? 4 * v : v); };
  auto mfma = [&](T x, T y, acc_t c) {   // c[v] += sum over k of x (column kcol(v)'s) y (row li's)
    if constexpr (F64) return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0);
  };

  // 1. acc = A[I, ks:j] A[c0, ks:j]^T, double-buffered PKC-deep chunks, in FP64 with
  //    two in flight (a 448-deep tile 46,500 to 43,400 cycles).  The tile
  //    itself and the first KX column blocks of L_jj^{-1} (column-major: X[n][k] at
  //    k * 64 + n, zero above its diagonal) are read behind the first chunk.
  acc_t acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = acc_t{0, 0, 0, 0};
  const TileBuf<T> Cb((const T *)d.A + (size_t)c0 * ld + r0 + 16 * w);
  const TileBuf<T> Xb((const T *)d.linv + (size_t)(j / NBI) * NBI * NBI);
  const unsigned lds = ld * (unsigned)sizeof(T);
  const unsigned cl = (unsigned)((klane * ld + li) * sizeof(T));
  const unsigned xl = (unsigned)((klane * NBI + li) * sizeof(T));
  constexpr int KX = F64 ? 1 : NB;
  T cv[NB][4], xp[KX][NB][4];
  auto xload = [&](int k, T (&x)[NB][4]) {
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (n >= k) x[n][v] = Xb.load(xl, (kstep(k, v) * NBI + 16 * n) * sizeof(T));
  };
  auto tile_loads = [&] {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) cv[b][v] = Cb.load(cl, kstep(b, v) * lds);
#pragma unroll
    for (int k = 0; k < KX; ++k) xload(k, xp[k]);
  };
  if (K > 0) {
    const T *Ap = (const T *)d.A + (size_t)ks * ld + r0, *Bp = (const T *)d.A + (size_t)ks * ld + c0;
    constexpr int KS = 256 / (NBI / VEC);   // columns per load of the workgroup
    const unsigned gl = (unsigned)((tid / (NBI / VEC) * ld + tid % (NBI / VEC) * VEC) * sizeof(T));
    // chunk c's loads go to register set c % DEPTH, DEPTH chunks ahead (K is a multiple of 64)
    vec_t ra[DEPTH][LA], rb[DEPTH][LA];
    auto gload = [&](int u, int kc) {
      const TileBuf<T> Ag(Ap + (size_t)kc * ld), Bg(Bp + (size_t)kc * ld);
#pragma unroll
      for (int it = 0; it < LA; ++it) {
        ra[u][it] = Ag.template load16<vec_t>(gl, it * KS * lds);
        rb[u][it] = Bg.template load16<vec_t>(gl, it * KS * lds);
      }
    };
    auto lstore = [&](int u, int buf) {
#pragma unroll
      for (int it = 0; it < LA; ++it) {
        const int lin = it * 256 + tid, kk = lin / (NBI / VEC), rp = lin % (NBI / VEC);
        *reinterpret_cast<vec_t *>(&S.g.As[buf][kk][VEC * rp]) = ra[u][it];
        *reinterpret_cast<vec_t *>(&S.g.Bs[buf][kk][VEC * rp]) = rb[u][it];
      }
    };
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) gload(u, u * PKC);
    tile_loads();
    lstore(0, 0);
    __syncthreads();
    for (int kc0 = 0; kc0 < K; kc0 += 2 * PKC)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int kc = kc0 + c * PKC;
        if (kc + DEPTH * PKC < K) gload(c % DEPTH, kc + DEPTH * PKC);
#pragma unroll
        for (int s = 0; s < PKC / 4; ++s) {
          const int kk = 16 * (s >> 2) + 4 * g + (s & 3);
          const T y = S.g.As[c][kk][16 * w + li];
          T x[NB];
#pragma unroll
          for (int b = 0; b < NB; ++b) x[b] = S.g.Bs[c][kk][16 * b + li];
#pragma unroll
          for (int b = 0; b < NB; ++b) acc[b] = mfma(x[b], y, acc[b]);
        }
        if (kc + PKC < K) lstore((c + 1) % DEPTH, c ^ 1);
        __syncthreads();
      }
  } else {
    tile_loads();
  }

  // 2. C = A[I, j] - acc (in acc), then L[I, j] = C L_jj^{-T} into lacc: column
  //    block n takes the column blocks k <= n of C
  acc_t lacc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[b][v] = cv[b][v] - acc[b][v];
    lacc[b] = acc_t{0, 0, 0, 0};
  }
  if (t < 0) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) Cb.store(acc[b][v], cl, kstep(b, v) * lds);
    return;
  }
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    T xk[NB][4];
    if (k >= KX) xload(k, xk);
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int n = k; n < NB; ++n) lacc[n] = mfma(k < KX ? xp[k < KX ? k : 0][n][v] : xk[n][v], acc[k][v], lacc[n]);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) Cb.store(lacc[b][v], cl, kstep(b, v) * lds);
  if (r0 >= pend) return;

  // 3. diagonal block of the tile's rows: D = L[I, j] L[I, j]^T, the blocks (I, J)
  //    with J <= I: (0,0) (3,3) | (1,0) (1,1) | (2,0) (2,1) (2,2) | (3,0) (3,1) (3,2)
  //    on waves 0 .. 3 (I, J below); element v of a lane: row li, column kcol(v)
  constexpr int U = 3;
  auto bI = [&](int u) { return w == 0 && u == 1 ? 3 : w; };
  auto bJ = [&](int u) { return w == 0 ? (u == 1 ? 3 : 0) : u; };
  const int nu = w < 2 ? 2 : 3;
  gT *Dg = gptr((T *)d.A) + (size_t)r0 * ld + r0;
  const TileBuf<T> Db((const T *)d.A + (size_t)r0 * ld + r0);
  T dg[U][4];
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < nu)
#pragma unroll
      for (int v = 0; v < 4; ++v) {   // (a diagonal block's upper half is read from its lower)
        const int r = 16 * bI(u) + li, c = 16 * bJ(u) + kcol(v);
        dg[u][v] = Db.load((unsigned)((min(r, c) * ld + max(r, c)) * sizeof(T)), 0);
      }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) S.Ls[16 * b + kcol(v)][16 * w + li] = lacc[b][v];
  __syncthreads();
  acc_t da[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    da[u] = acc_t{0, 0, 0, 0};
    if (u < nu)
#pragma unroll
      for (int k = 0; k < NBI; k += 4)
        da[u] = mfma(S.Ls[k + g][16 * bJ(u) + li], S.Ls[k + g][16 * bI(u) + li], da[u]);
  }
  if (t != 0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u < nu)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * bI(u) + li, c = 16 * bJ(u) + kcol(v);
          if (r >= c) Dg[c * ld + r] = dg[u][v] - da[u][v];
        }
    return;
  }

  // 4. tile 0: the block at r0 = j + 64 has had every update of the panel's
  //    earlier columns; factor and invert it in LDS, store L and its inverse
  __syncthreads();   // every wave has read L[I, j]
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < nu)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * bI(u) + li, c = 16 * bJ(u) + kcol(v);
        S.f.M[r][c] = (double)(T)(dg[u][v] - da[u][v]);
        if (bI(u) != bJ(u)) S.f.M[c][r] = 0.0;
      }
  if (tid == 0) S.f.fail = 0;
  __syncthreads();
  potf2_factor_invert<T>(S.f, d, r0, Dg, tid);
}

// --------------------------------------------------------------------------
// Trailing update with BF16 operands (factored rows only): FP32 storage, the
// panel rounded once to BF16 (round to nearest even) into a packed copy,
// v_mfma_f32_16x16x32_bf16 with FP32 accumulation, FP32 read-modify-write of
// C.  That instruction takes in lane l the row (l%16) of A and the column
// (l%16) of B^T at the eight k values 8(l/16) .. 8(l/16)+7, and returns D rows
// 4(l/16)+v of column (l%16) (the FP32 layout, so the epilogue is shared).
//
// The packed copy holds, per group of eight k values, one 16-byte entry per
// row, which is exactly an MFMA operand: a K chunk of 32 is 4 groups x 128
// rows of entries, loaded with 16-byte loads (a wave covers 1 KB contiguous)
// and stored unchanged into LDS.  LDS holds entry [g][row] at slot
// row ^ ((row >> 4) & 3), so that the sixteen rows a quarter-wave reads fall
// into distinct 16-byte slots of a 256-byte bank window.
// --------------------------------------------------------------------------
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(1))) const bf8 gcbf8;

__device__ __forceinline__ int bf_slot(int r) { return r ^ ((r >> 4) & 3); }

// Packed copy of the panel at p0: the address that row 0 of its first group would
// have (the copy starts at the panel's end), and the groups of a plane.
__device__ __forceinline__ bf8 *packed_panel(const FactorDesc &d, int p0, int nb) {
  return (bf8 *)d.pbf + (int64_t)((p0 / nb) & 1) * d.pbf_slot - min(p0 + nb, d.nf);
}
__device__ __forceinline__ int packed_groups(const FactorDesc &d, int nb) { return min(nb, d.nf) / 8; }

// Packed copy of the panel [p0, pend): one thread per (row, group of eight k),
// one plane (rows [pend, nf)) or three (rows [pend, nrows)).
template <int PLANES>
__global__ __launch_bounds__(256) void panel_pack_kernel(const FactorDesc *__restrict__ descs, int p0, int nb) {
  const FactorDesc d = descs[blockIdx.z];
  const int pend = min(p0 + nb, d.nf);
  const int r = pend + blockIdx.x * 256 + threadIdx.x, gk = blockIdx.y;
  if (r >= (PLANES == 1 ? d.nf : d.nrows) || p0 + 8 * gk >= pend) return;
  const __attribute__((address_space(1))) float *src = gptr((const float *)d.A) + (size_t)(p0 + 8 * gk) * d.ld + r;
  float v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = src[(size_t)i * d.ld];
  bf8 *dst = packed_panel(d, p0, nb) + (size_t)gk * d.prows + r;
#pragma unroll
  for (int q = 0; q < PLANES; ++q) {
    bf8 e;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      e[i] = (__bf16)v[i];       // round to nearest even
      v[i] -= (float)e[i];       // exact
    }
    *gptr(dst + (size_t)q * packed_groups(d, nb) * d.prows) = e;
  }
}

template <int TM, int TN>
__global__ __launch_bounds__(256, 2) void trail_bf16_kernel(const FactorDesc *__restrict__ descs, int kind, int p0,
                                                            int nb) {
  constexpr int KCH = 32, KG = KCH / 8;
  constexpr int WM = 2, WN = 2, WTM = TM / WM, WTN = TN / WN, BM = WTM / 16, BN = WTN / 16;
  constexpr int EA = KG * TM / 256, EB = KG * TN / 256;   // entries per thread per chunk
  typedef __attribute__((address_space(1))) float gT;
  __shared__ bf8 As[2][KG][TM];
  __shared__ bf8 Bs[2][KG][TN];

  int bx, by;
  xcd_order(bx, by);
  const FactorDesc d = descs[by];
  int row0, col0, ks, ke;
  if (!update_tile(d, kind, p0, nb, TM, TN, 1, bx, row0, col0, ks, ke)) return;
  const int ld = d.ld;
  // the packed panel: entry (group g, row r) at P[g * prows + r]; k = ks + 8 g
  gcbf8 *P = gptr((const bf8 *)packed_panel(d, p0, nb));
  gT *Cg = gptr((float *)d.A) + (size_t)col0 * ld + row0;
  const int K = ke - ks, prows = d.prows;

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w / WN, wn = w % WN;
  const int g = lane >> 4, li = lane & 15;

  f4 acc[BM][BN];
#pragma unroll
  for (int a = 0; a < BM; ++a)
#pragma unroll
    for (int b = 0; b < BN; ++b) acc[a][b] = f4{0, 0, 0, 0};

  bf8 ra[EA], rb[EB];
  auto gload = [&](int kc) {
    const int g0 = kc / 8;
#pragma unroll
    for (int i = 0; i < EA; ++i) {
      const int e = i * 256 + tid, eg = e / TM, er = e % TM;
      ra[i] = P[(size_t)(g0 + eg) * prows + row0 + er];
    }
#pragma unroll
    for (int i = 0; i < EB; ++i) {
      const int e = i * 256 + tid, eg = e / TN, er = e % TN;
      rb[i] = P[(size_t)(g0 + eg) * prows + col0 + er];
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < EA; ++i) {
      const int e = i * 256 + tid;
      As[buf][e / TM][bf_slot(e % TM)] = ra[i];
    }
#pragma unroll
    for (int i = 0; i < EB; ++i) {
      const int e = i * 256 + tid;
      Bs[buf][e / TN][bf_slot(e % TN)] = rb[i];
    }
  };

  gload(0);
  lstore(0);
  __syncthreads();
  int buf = 0;
  for (int kc = 0; kc < K; kc += KCH) {
    const bool more = kc + KCH < K;
    if (more) gload(kc + KCH);
#pragma unroll
    for (int s = 0; s < KCH / 32; ++s) {
      bf8 ya[BM], xb[BN];
#pragma unroll
      for (int a = 0; a < BM; ++a) ya[a] = As[buf][4 * s + g][bf_slot(wm * WTM + a * 16 + li)];
#pragma unroll
      for (int b = 0; b < BN; ++b) xb[b] = Bs[buf][4 * s + g][bf_slot(wn * WTN + b * 16 + li)];
#pragma unroll
      for (int a = 0; a < BM; ++a)
#pragma unroll
        for (int b = 0; b < BN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ya[a], xb[b], acc[a][b], 0, 0, 0);
    }
    if (more) lstore(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  auto rl = [&](int a, int v) { return wm * WTM + a * 16 + 4 * g + v; };
  auto cl = [&](int b, int v) { (void)v; return wn * WTN + b * 16 + li; };
  subtract_tile<float, BM, BN>(Cg, ld, acc, rl, cl, row0 < col0 + TN, row0, col0);
}

// --------------------------------------------------------------------------
// Trailing update of an FP32 factorisation on the BF16 matrix units.  Each panel
// value a is split exactly into BF16 parts a1 + a2 + a3 (panel_pack_kernel), and a
// product a b is the sum of a3 b1, a1 b3, a2 b2, a2 b1, a1 b2 and a1 b1, smallest
// first, accumulated in FP32; what is left out (a2 b3, a3 b2, a3 b3) is below
// 2^-25 of the product, half an FP32 rounding, and 32 products cost six rounded
// additions to the accumulator where v_mfma_f32_16x16x4f32 makes 32.  Six passes
// at 16 times the FP32 matrix rate: 2.7 times the FP32 bound (417 against 157 TF).
// Tile 128 x 128, 2 x 2 waves, K chunks of 32 in one LDS buffer of 48 KB with the
// next chunk in registers, two workgroups per CU by registers: larger wave tiles
// would leave LDS reads (three planes of both operands per chunk) further from
// the bound but not fit the accumulators twice.  SEL as in update_tile.
// The tile itself is read behind the last chunk's products in 16-byte pieces: four
// dependent rounds of reads and writes after the loop were a quarter of a tile's time.
// Trailing updates of 25 theta at n = 8192 (two factorisations): 45.8 ms with 2.6 ms
// of packing (74.1 ms on v_mfma_f32_16x16x4f32, 48.0 with the tile read at the end);
// that is 189 TF of FP32 products, 1.13 PF on the BF16 units (a large BF16 library
// product: 1.06).
// Counters of the zero-start evaluation of 64: matrix units 50% busy, CUs 98%, no LDS bank
// conflicts, 3.6 TB/s (2.0 times the bytes of the panel and the block once).
// Error of log|S| at n = 1024: 6.6e-7 relative (2.1e-6 on the FP32 units).
// --------------------------------------------------------------------------
template <int SEL>
__global__ __launch_bounds__(256, 2) void trail_split_kernel(const FactorDesc *__restrict__ descs, int kind, int p0,
                                                             int nb) {
  constexpr int TM = 128, KCH = 32, KG = KCH / 8, NP = 3, WT = 64, BM = 4, BN = 4;
  constexpr int E = NP * KG * TM / 256;   // entries per thread, operand and chunk
  __shared__ bf8 As[NP * KG][TM];         // [plane KG + group][slot]
  __shared__ bf8 Bs[NP * KG][TM];

  int bx, by;
  xcd_order(bx, by);
  const FactorDesc d = descs[by];
  int row0, col0, ks, ke;
  if (!update_tile(d, kind, p0, nb, TM, TM, SEL, bx, row0, col0, ks, ke)) return;
  const int ld = d.ld, prows = d.prows, K = ke - ks;
  const int G = packed_groups(d, nb);
  gcbf8 *P = gptr((const bf8 *)packed_panel(d, p0, nb));

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w >> 1, wn = w & 1;
  const int g = lane >> 4, li = lane & 15;

  f4 acc[BM][BN];
#pragma unroll
  for (int a = 0; a < BM; ++a)
#pragma unroll
    for (int b = 0; b < BN; ++b) acc[a][b] = f4{0, 0, 0, 0};

  bf8 ra[E], rb[E];
  auto gload = [&](int kc) {
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const int e = i * 256 + tid, pg = e / TM, er = e % TM;   // pg = plane KG + group
      gcbf8 *src = P + (size_t)((pg / KG) * G + kc / 8 + pg % KG) * prows + er;
      ra[i] = src[row0];
      rb[i] = src[col0];
    }
  };
  auto stage = [&] {
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const int e = i * 256 + tid, pg = e / TM, s = bf_slot(e % TM);
      As[pg][s] = ra[i];
      Bs[pg][s] = rb[i];
    }
    __syncthreads();
  };
  auto chunk = [&] {
    bf8 xb[NP][BN];
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int b = 0; b < BN; ++b) xb[q][b] = Bs[q * KG + g][bf_slot(wn * WT + b * 16 + li)];
#pragma unroll
    for (int a = 0; a < BM; ++a) {
      bf8 ya[NP];
#pragma unroll
      for (int q = 0; q < NP; ++q) ya[q] = As[q * KG + g][bf_slot(wm * WT + a * 16 + li)];
      constexpr int QA[6] = {2, 0, 1, 1, 0, 0}, QB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int s = 0; s < 6; ++s)
#pragma unroll
        for (int b = 0; b < BN; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ya[QA[s]], xb[QB[s]][b], acc[a][b], 0, 0, 0);
    }
  };
  gload(0);
  for (int kc = KCH; kc < K; kc += KCH) {
    stage();
    gload(kc);
    chunk();
    __syncthreads();   // every wave is done reading the buffer
  }
  stage();
  // the tile is read behind the last chunk's products: element v of block (a, b) at
  // row 16 a + v, column 16 b from the lane's first, four rows in 16 bytes
  const TileBuf<float> Cb((float *)d.A + (size_t)(col0 + wn * WT) * ld + row0 + wm * WT);
  const unsigned lds = ld * 4u, cl = (unsigned)((li * ld + 4 * g) * 4);
  f4 c[BM][BN];
#pragma unroll
  for (int a = 0; a < BM; ++a)
#pragma unroll
    for (int b = 0; b < BN; ++b) c[a][b] = Cb.load16<f4>(cl, 16 * b * lds + 16 * a * 4u);
  chunk();
  const int below = row0 + wm * WT + 4 * g - (col0 + wn * WT + li);   // row - column of the first
  if (row0 >= col0 + TM) {
    // (as global stores: behind a 16-byte buffer store with a register offset the
    // compiler rewrites the data registers at once, which has stored wrong values)
    typedef __attribute__((address_space(1))) f4 gf4;
    auto *Cg = gptr((float *)d.A) + (size_t)(col0 + wn * WT + li) * ld + row0 + wm * WT + 4 * g;
#pragma unroll
    for (int b = 0; b < BN; ++b)
#pragma unroll
      for (int a = 0; a < BM; ++a) *(gf4 *)(Cg + (size_t)(16 * b) * ld + 16 * a) = c[a][b] - acc[a][b];
  } else {   // its lower triangle only
#pragma unroll
    for (int a = 0; a < BM; ++a)
#pragma unroll
      for (int b = 0; b < BN; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (below + 16 * (a - b) + v >= 0) Cb.store(c[a][b][v] - acc[a][b][v], cl, 16 * b * lds + (16 * a + v) * 4u);
  }
}

// --------------------------------------------------------------------------
// Host driver
// --------------------------------------------------------------------------
static int count_rows_real(const HostFactor &h, int a) {
  // real rows in [a, nrows): [a, n_real) U [max(a, nf), nf + kb_real)
  int c = 0;
  if (a < h.n_real) c += h.n_real - a;
  const int b0 = a > h.d.nf ? a : h.d.nf;
  if (b0 < h.d.nf + h.kb_real) c += h.d.nf + h.kb_real - b0;
  return c;
}
static int count_cols_real(const HostFactor &h, int a, int cend) {
  int c = 0;
  const int e1 = cend < h.n_real ? cend : h.n_real;
  if (a < e1) c += e1 - a;
  const int b0 = a > h.d.nf ? a : h.d.nf;
  const int e2 = cend < h.d.nf + h.ks_real ? cend : h.d.nf + h.ks_real;
  if (b0 < e2) c += e2 - b0;
  return c;
}
static double trap_elems(double nr, double nc) { return nc * (nc + 1.0) * 0.5 + (nr - nc) * nc; }
// Real (unpadded) lower-triangle elements of columns [c0, c1), rows at or below
// each column; with only_factored, rows of the factored block only.
static double lower_real(const HostFactor &h, int c0, int c1, bool only_factored) {
  double s = 0.0;
  const int fa = c0, fb = std::min(c1, h.n_real);
  if (fa < fb) {
    const double m = fb - fa;
    s += m * h.n_real - (double)(fa + fb - 1) * m * 0.5;
    if (!only_factored) s += m * h.kb_real;
  }
  if (!only_factored) {
    const int sa = std::max(c0, h.d.nf), sb = std::min(c1, h.d.nf + h.ks_real);
    if (sa < sb) {
      const double m = sb - sa;
      s += m * (h.d.nf + h.kb_real) - (double)(sa + sb - 1) * m * 0.5;
    }
  }
  return s;
}

// Workgroups of a trailing update (border: of its border rows alone, SEL 2).
static int tiles_for(const FactorDesc &d, int kind, int p0, int nb, int TM, bool border = false) {
  if (p0 >= d.nf) return 0;
  const int pend = std::min(p0 + nb, d.nf);
  int r0, c0, cend;
  if (kind == KIND_TRAIL) { r0 = pend; c0 = pend; cend = d.ncols; }
  else if (kind == KIND_TRAIL_A) { r0 = pend; c0 = pend; cend = std::min(pend + nb, d.nf); }
  else { c0 = std::min(pend + nb, d.nf); r0 = c0; cend = d.ncols; }
  if (r0 >= d.nrows || c0 >= cend) return 0;
  const int nr = (d.nrows - r0) / TM;
  const int nc = (cend - c0) / TM;
  if (border) return (d.nrows - d.nf) / TM * nc;
  return nc * (nc + 1) / 2 + (nr - nc) * nc;
}

// Synthetic symmetric positive definite batch for the autotuner: unit-free
// values, diagonally dominant on the factored columns, small border rows.
template <typename T>
__global__ __launch_bounds__(256) void tune_fill_kernel(const FactorDesc *__restrict__ descs) {
  const FactorDesc d = descs[blockIdx.y];
  const int c = blockIdx.x;
  if (c >= d.ncols) return;
  __attribute__((address_space(1))) T *col = gptr((T *)d.A) + (size_t)c * d.ld;
  for (int r = c + threadIdx.x; r < d.nrows; r += 256) {
    const uint32_t h = (uint32_t)r * 2654435761u ^ (uint32_t)c * 40503u;
    const double off = ((double)(h >> 8) / 16777216.0 - 0.5) / (double)d.nf;
    col[r] = (T)(r == c ? (c < d.nf ? 2.0 : 1.0) : off);
  }
  if (c == 0 && threadIdx.x == 0) *d.info = 0;
}

template <typename T>
static int factor_batch_t(Ctx &ctx, const std::vector<HostFactor> &fs, int nb, int tm, bool look_cfg,
                          bool bf16_trail) {
  const int B = (int)fs.size();
  if (B == 0) return 0;
  const double esz = sizeof(T);
  // device descriptor array, sorted by nf descending so active sets are prefixes
  std::vector<int> order(B);
  for (int i = 0; i < B; ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return fs[a].d.nf > fs[b].d.nf; });
  std::vector<FactorDesc> hd(B);
  for (int i = 0; i < B; ++i) {
    hd[i] = fs[order[i]].d;
    const int real = fs[order[i]].n_real;
    hd[i].ne = real > 0 ? std::min(hd[i].nf, round_up(real, NBI)) : hd[i].nf;
  }
  // Lookahead: the next panel's columns are updated first (TRAIL_A, on the
  // caller's stream), the rest (TRAIL_B) on the handle's side stream, and the
  // next panel is factored on the caller's stream while TRAIL_B runs.  TRAIL_A
  // of the following panel waits for TRAIL_B, which updated its columns too.
  // (lookahead runs on the caller's lane only: the side stream and its events
  // serve one factorisation at a time)
  // (and not inside a pass graph, which is captured on one stream)
  const bool look = look_cfg && ctx.lookahead && ctx.lane == 0 && ctx.pg_mode == Ctx::PG_OFF && hd[0].nf > nb &&
                    ctx.side_ready() == INLA_OK;
  // Packed panel copies (FP32 storage): three planes where the caller brings memory for
  // them and the tile is the split kernel's, else one for BF16 updates.  A tuned 64 x 64
  // tile keeps the FP32 units.  Which kernel multiplies is thus fixed by the caller and
  // the configuration alone: not by an order, by the rest of the batch or by lookahead,
  // so that the results don't depend on those.  Two slots of m = min(nb, nf) columns by
  // nrows - m rows take 12 m (nrows - m) <= 3 nrows^2 bytes; the half of an evaluation's
  // region that its FP32 matrix leaves free holds 4 nrows^2.
  const bool f32 = std::is_same<T, float>::value;
  int planes = f32 && (bf16_trail || tm == 128) ? 3 : 0;
  for (int i = 0; i < B && planes == 3; ++i)
    if (!fs[i].pack) planes = 0;
  if (f32 && bf16_trail && planes == 0) planes = 1;
  if (planes == 3) {
    for (int i = 0; i < B; ++i) {
      const int m = std::min(nb, hd[i].nf);
      hd[i].prows = hd[i].nrows - m;
      const size_t slot = (size_t)3 * (m / 8) * hd[i].prows;
      hd[i].pbf = fs[order[i]].pack;
      hd[i].pbf_slot = look && hd[i].nf > nb ? (int64_t)slot : 0;
      if (16 * (slot + hd[i].pbf_slot) > fs[order[i]].pack_bytes) return INLA_ERR_NOMEM;
    }
  } else if (planes == 1) {
    // two slots of the packed BF16 panel copy per theta (16-byte entries)
    size_t entries = 0;
    for (int i = 0; i < B; ++i) entries += 2 * (size_t)(nb / 8) * hd[i].nf;
    char *base = ctx.pbf_reserve(16 * entries);
    if (!base) return INLA_ERR_NOMEM;
    size_t off = 0;
    for (int i = 0; i < B; ++i) {
      hd[i].pbf = base + 16 * off;
      hd[i].pbf_slot = (int64_t)(nb / 8) * hd[i].nf;
      hd[i].prows = hd[i].nf;
      off += 2 * (size_t)hd[i].pbf_slot;
    }
  }
  FactorDesc *dd = (FactorDesc *)ctx.upload(hd.data(), sizeof(FactorDesc) * B);
  if (!dd) return INLA_ERR_NOMEM;
  const int nf_max = hd[0].nf;
  auto active = [&](int col) {
    int a = 0;
    while (a < B && hd[a].nf > col) ++a;
    return a;
  };
  // Every grid and scalar argument of a panel's launch sequence follows from
  // these sizes; the pointers travel in the argument block.
  std::vector<int64_t> key0 = {0x46414354, (int64_t)sizeof(T), bf16_trail, nb, B};
  for (int i = 0; i < B; ++i) {
    const HostFactor &h = fs[order[i]];
    key0.insert(key0.end(), {h.d.nf, h.d.nrows, h.d.ncols, h.d.id_row0, h.n_real, h.kb_real, h.ks_real});
  }
  // the panel [p0, p0 + nb): potf2_inv of its first diagonal block, then one
  // left-looking panel step per 64-wide block column (one graph replay),
  // enqueued on ctx.stream
  auto panel_seq = [&](int p0, const std::vector<int64_t> &key) -> int {
    return ctx.sequence(INLA_K_PANEL, key, hd.data(), sizeof(FactorDesc) * B, [&](const void *dv) {
      const FactorDesc *pd = (const FactorDesc *)dv;
      for (int j = p0; j < p0 + nb && j < nf_max; j += NBI) {
        const int act = active(j);
        if (j == p0) {
          double fl = 0;
          for (int i = 0; i < act; ++i) {
            const double kr = std::max(0, std::min(NBI, fs[order[i]].n_real - j));
            fl += 2.0 * kr * kr * kr / 3.0;
          }
          ctx.launch(INLA_K_POTF2, fl, 0.0, [&] {
            hipLaunchKernelGGL(potf2_inv_kernel<T>, dim3(act), dim3(256), 0, ctx.stream, pd, j);
          });
        }
        // algorithmic work per theta (real rows and columns): the left-looking
        // product over [p0, j), the TRSM, the SYRK of each in-panel diagonal
        // block below and the next diagonal block's factorisation
        int gx = 0;
        bool any = false;   // some theta has real columns here
        double fl = 0, by = 0;
        for (int i = 0; i < act; ++i) {
          const HostFactor &h = fs[order[i]];
          gx = std::max(gx, (h.d.nrows - j - NBI) / NBI);
          const int pend = std::min(p0 + nb, h.d.nf);
          any = any || j < hd[i].ne;
          const double kr = std::max(0, std::min(NBI, h.n_real - j));
          const double kl = std::max(0, std::min(j, h.n_real) - p0);
          const double m = count_rows_real(h, j + NBI);
          fl += 2.0 * m * kr * kl + m * kr * kr;
          by += esz * m * (kl + 2.0 * kr);
          for (int r = j + NBI; r < pend; r += NBI) {
            const double kd = std::max(0, std::min(NBI, h.n_real - r));
            fl += kd * (kd + 1.0) * kr;
            by += 2.0 * esz * kd * (kd + 1.0) * 0.5;
            if (r == j + NBI) fl += 2.0 * kd * kd * kd / 3.0;
          }
        }
        if (gx == 0 || !any) continue;
        const int Q = (act * (gx - 1) + 7) / 8;
        const int pre = j > p0 && j + 2 * NBI < p0 + nb ? 1 : 0;
        ctx.launch(INLA_K_PANEL, fl, by, [&] {
          hipLaunchKernelGGL(panel_step_kernel<T>, dim3(act * (1 + pre) + 8 * Q), dim3(256), 0, ctx.stream, pd, p0,
                             nb, j, act, gx, Q, pre);
        });
      }
    });
  };
  // the packed copy of panel p0 for its trailing update, on ctx.stream
  auto panel_copy = [&](int p0) {
    const int act = active(p0);
    int rows = 0;
    double by = 0;
    for (int i = 0; i < act; ++i) {
      const HostFactor &h = fs[order[i]];
      const int pend = std::min(p0 + nb, h.d.nf), last = planes == 3 ? h.d.nrows : h.d.nf;
      rows = std::max(rows, last - pend);
      const double real = planes == 3 ? count_rows_real(h, pend) : std::max(0, h.n_real - pend);
      by += (4.0 + 2.0 * planes) * real * (double)std::max(0, std::min(pend, h.n_real) - p0);
    }
    if (rows <= 0) return;
    ctx.launch(INLA_K_PANEL, 0.0, by, [&] {
      const dim3 grid((rows + 255) / 256, nb / 8, act);
      if (planes == 3) hipLaunchKernelGGL(panel_pack_kernel<3>, grid, dim3(256), 0, ctx.stream, dd, p0, nb);
      else hipLaunchKernelGGL(panel_pack_kernel<1>, grid, dim3(256), 0, ctx.stream, dd, p0, nb);
    });
  };
  auto panel = [&](int p0) -> int {
    std::vector<int64_t> key = key0;
    key.push_back(p0);
    const int rc = panel_seq(p0, key);
    if (!rc && planes) panel_copy(p0);
    return rc;
  };
  // the trailing update of kind TRAIL (everything right of the panel), TRAIL_A
  // (the next panel's columns) or TRAIL_B (the columns after the next panel),
  // enqueued on ctx.stream
  auto trail = [&](int p0, int kind) {
    const int act = active(p0);
    const int TT = planes ? 128 : tm;   // the BF16 units' kernels have 128 x 128 tiles only
    int gx = 0, gx_border = 0;
    double fl = 0, by = 0, fl_q = 0, by_q = 0;   // all tiles; tiles of the factored rows only
    bool rows_q = false;                          // some theta has factored rows in the region
    for (int i = 0; i < act; ++i) {
      const HostFactor &h = fs[order[i]];
      gx = std::max(gx, tiles_for(h.d, kind, p0, nb, TT));
      gx_border = std::max(gx_border, tiles_for(h.d, kind, p0, nb, TT, true));
      const int pend = std::min(p0 + nb, h.d.nf), pnext = std::min(pend + nb, h.d.nf);
      int c0 = pend, c1 = h.d.ncols;
      if (kind == KIND_TRAIL_A) c1 = pnext;
      else if (kind == KIND_TRAIL_B) c0 = pnext;
      if (c0 >= c1) continue;
      rows_q = rows_q || c0 < h.d.nf;
      const double kr = std::max(0, std::min(pend, h.n_real) - p0);
      const double el = lower_real(h, c0, c1, false), elq = lower_real(h, c0, c1, true);
      const double nr = count_rows_real(h, c0), nc = count_cols_real(h, c0, c1);
      const double nrq = std::max(0, h.n_real - c0), ncq = std::max(0, std::min(c1, h.n_real) - c0);
      fl += 2.0 * el * kr;
      by += 2.0 * esz * el + esz * (nr + nc) * kr;
      fl_q += 2.0 * elq * kr;
      by_q += elq > 0 ? 2.0 * esz * elq + esz * (nrq + ncq) * kr : 0.0;
    }
    if (gx == 0) return;
    gx_border = round_up(gx_border, 8);
    gx = round_up(gx, 8);   // xcd_order needs a grid of a multiple of 8 workgroups
    if (bf16_trail && f32) {
      // BF16 operands for the factored rows only: the border rows carry the
      // constraint rows and the right-hand side, whose Schur block (C Q^{-1}
      // C^T and C Q^{-1} b) arises by cancellation and keeps FP32 accuracy
      if (rows_q)
        ctx.launch(INLA_K_TRAIL, fl_q, by_q, [&] {
          hipLaunchKernelGGL((trail_bf16_kernel<128, 128>), dim3(gx, act), dim3(256), 0, ctx.stream, dd, kind, p0,
                             nb);
        });
      if (gx_border == 0) return;
      ctx.launch(INLA_K_BORDER, fl - fl_q, by - by_q, [&] {
        if (planes == 3)
          hipLaunchKernelGGL(trail_split_kernel<2>, dim3(gx_border, act), dim3(256), 0, ctx.stream, dd, kind, p0, nb);
        else
          hipLaunchKernelGGL((gemm_update_kernel<T, 128, 128, 2>), dim3(gx_border, act), dim3(256), 0, ctx.stream, dd,
                             kind, p0, nb);
      });
    } else if (planes == 3) {
      ctx.launch(INLA_K_TRAIL, fl, by, [&] {
        hipLaunchKernelGGL(trail_split_kernel<0>, dim3(gx, act), dim3(256), 0, ctx.stream, dd, kind, p0, nb);
      });
    } else {
      const bool aux = ctx.lane == 1;
      ctx.launch(INLA_K_TRAIL, fl, by, [&] {
        if (TT == 64 && aux)
          hipLaunchKernelGGL((trail_update_aux_kernel<T, 64, 64>), dim3(gx, act), dim3(256), 0, ctx.stream, dd, kind,
                             p0, nb);
        else if (TT == 64)
          hipLaunchKernelGGL((trail_update_kernel<T, 64, 64>), dim3(gx, act), dim3(256), 0, ctx.stream, dd, kind, p0,
                             nb);
        else if (aux)
          hipLaunchKernelGGL((trail_update_aux_kernel<T, 128, 128>), dim3(gx, act), dim3(256), 0, ctx.stream, dd,
                             kind, p0, nb);
        else
          hipLaunchKernelGGL((trail_update_kernel<T, 128, 128>), dim3(gx, act), dim3(256), 0, ctx.stream, dd, kind,
                             p0, nb);
      });
    }
  };
  int rc = 0;
  hipStream_t main_stream = ctx.stream;
  for (int p0 = 0; p0 < nf_max && !rc; p0 += nb) {
    if (!look) {
      if ((rc = panel(p0))) break;
      trail(p0, KIND_TRAIL);
      continue;
    }
    if (p0 == 0 && (rc = panel(p0))) break;
    if (p0 > 0 && hipStreamWaitEvent(main_stream, ctx.ev_b, 0) != hipSuccess) { rc = INLA_ERR_HIP; break; }
    trail(p0, KIND_TRAIL_A);
    if (hipEventRecord(ctx.ev_a, main_stream) != hipSuccess ||
        hipStreamWaitEvent(ctx.side, ctx.ev_a, 0) != hipSuccess) { rc = INLA_ERR_HIP; break; }
    ctx.stream = ctx.side;
    trail(p0, KIND_TRAIL_B);
    ctx.stream = main_stream;
    if (hipEventRecord(ctx.ev_b, ctx.side) != hipSuccess) { rc = INLA_ERR_HIP; break; }
    if (p0 + nb < nf_max && (rc = panel(p0 + nb))) break;
  }
  ctx.stream = main_stream;
  if (look && hipStreamWaitEvent(main_stream, ctx.ev_b, 0) != hipSuccess && !rc) rc = INLA_ERR_HIP;
  if (rc) return rc;
  return ctx.check();
}

// ------------------------------------------------------------------ tuning
static int b_bucket(int B) {
  int b = 1;
  while (b < B) b <<= 1;
  return b;
}

std::vector<int64_t> tune_key(int prec, int nf_max, int B) { return {prec, nf_max, b_bucket(B)}; }

// Untuned configuration: 512-wide panels; 64 x 64 FP64 trailing tiles (at
// 8192 they measure about 4% faster than 128 x 128), 128 x 128 otherwise.
// BF16 batches of padded order 4096 and above take 1024-wide panels: their
// trailing update then reads and writes the FP32 trailing block once per 1024
// of K rather than per 512 (the BF16 evaluation of 64 theta at n = 8192:
// 864 -> 827 ms, its BF16 trailing update 13% -> 17% of the BF16 peak);
// smaller ones keep 512, which leaves them trailing updates at all.
TuneCfg default_config(int prec, int nf_max) {
  TuneCfg c;
  if (prec == INLA_PREC_FP64) c.tm = 64;
  if (prec == INLA_PREC_BF16 && nf_max >= 4096) c.nb = 1024;
  return c;
}

TuneCfg tuned_config(const Ctx &ctx, int prec, int nf_max, int B) {
  auto it = ctx.tune.find(tune_key(prec, nf_max, B));
  if (it != ctx.tune.end()) return it->second;
  return default_config(prec, nf_max);
}

bool tune_valid(int prec, const TuneCfg &c) {
  const bool nbok = c.nb == 128 || c.nb == 256 || c.nb == 512 || c.nb == 1024;
  const bool tmok = c.tm == 128 || (c.tm == 64 && prec != INLA_PREC_BF16);
  return nbok && tmok && (c.look == 0 || c.look == 1);
}

int factor_batch(Ctx &ctx, const std::vector<HostFactor> &fs, int prec, const TuneCfg *cfg) {
  if (fs.empty()) return 0;
  PrecScope tag(ctx, prec);
  TuneCfg c;
  if (cfg) {
    c = *cfg;
  } else {
    int nf_max = 0;
    for (const HostFactor &h : fs) nf_max = std::max(nf_max, h.d.nf);
    c = tuned_config(ctx, prec, nf_max, (int)fs.size());
  }
  if (prec == INLA_PREC_FP64) return factor_batch_t<double>(ctx, fs, c.nb, c.tm, c.look != 0, false);
  return factor_batch_t<float>(ctx, fs, c.nb, c.tm, c.look != 0, prec == INLA_PREC_BF16);
}

constexpr double LOOKAHEAD_MARGIN = 0.05;
constexpr double DEFAULT_MARGIN = 0.03;

// Candidate (panel width, trailing tile) pairs without lookahead; the BF16 path
// has one tile size.  The fastest is then timed once more with lookahead.
static std::vector<TuneCfg> tune_candidates(int prec) {
  std::vector<TuneCfg> c;
  for (int nb : {128, 256, 512, 1024})
    for (int tm : {64, 128})
      if (prec != INLA_PREC_BF16 || tm == 128) c.push_back({nb, tm, 0});
  return c;
}

int autotune(Ctx &ctx, int B, const int *n, const int *kb, int prec, int reps, TuneCfg *best_out, double *ms_out,
             int *n_cand) {
  const size_t esz = prec == INLA_PREC_FP64 ? 8 : 4;
  std::vector<HostFactor> fs(B);
  std::vector<size_t> offs(B), offp(B);
  int nf_max = 0;
  for (int i = 0; i < B; ++i) {
    HostFactor &h = fs[i];
    const int nf = round_up(std::max(n[i], 1), PADN);
    const int kbp = kb[i] > 0 ? round_up(kb[i], PADN) : 0;
    h.d.nf = nf; h.d.nrows = h.d.ncols = h.d.ld = nf + kbp;
    h.d.id_row0 = std::numeric_limits<int>::max();
    h.n_real = n[i]; h.kb_real = kb[i] > 0 ? kb[i] : 0; h.ks_real = h.kb_real;
    nf_max = std::max(nf_max, nf);
  }
  // A bordered batch stands for an evaluation's, whose FP32 and BF16 updates have memory
  // for packed panel copies and so multiply on split operands: timed without it, nine of
  // order 3000 in FP32 chose 64 x 64 tiles on the FP32 units, which take the evaluation
  // 20.4 ms and not 19.7.  (Without room for it, where the evaluation itself would go in
  // pieces, the batch is timed without.)
  auto layout = [&](bool pack) {
    size_t total = 0;
    for (int i = 0; i < B; ++i) {
      HostFactor &h = fs[i];
      offs[i] = total;
      total += (esz * (size_t)h.d.ld * h.d.ncols + esz * (size_t)h.d.nf * NBI + sizeof(int) + 255) & ~size_t(255);
      offp[i] = total;
      total += h.pack_bytes = pack && kb[i] > 0 ? 4 * (size_t)h.d.nrows * h.d.nrows : 0;
    }
    return total;
  };
  const bool pack = prec != INLA_PREC_FP64;
  if (!(pack && ctx.reserve(layout(true))) && !ctx.reserve(layout(false))) return INLA_ERR_NOMEM;
  for (int i = 0; i < B; ++i) {
    char *base = ctx.ws + offs[i];
    fs[i].d.A = base;
    fs[i].d.linv = base + esz * (size_t)fs[i].d.ld * fs[i].d.ncols;
    fs[i].d.info = (int *)((char *)fs[i].d.linv + esz * (size_t)fs[i].d.nf * NBI);
    if (fs[i].pack_bytes) fs[i].pack = ctx.ws + offp[i];
  }
  std::vector<FactorDesc> hd(B);
  int cmax = 0;
  for (int i = 0; i < B; ++i) { hd[i] = fs[i].d; cmax = std::max(cmax, hd[i].ncols); }
  const FactorDesc *dd = (const FactorDesc *)ctx.upload(hd.data(), sizeof(FactorDesc) * B);
  if (!dd) return INLA_ERR_NOMEM;
  hipEvent_t a, b;
  if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) return INLA_ERR_HIP;
  const bool prof = ctx.prof;
  ctx.prof = false;
  auto cand = tune_candidates(prec);
  int best = -1, rc = 0;
  double best_ms = 0;
  auto time_cfg = [&](const TuneCfg &cfg) {
    double tot = 0;
    for (int r = 0; r <= reps && !rc; ++r) {   // one untimed run, then `reps` timed ones
      if (prec == INLA_PREC_FP64)
        hipLaunchKernelGGL(tune_fill_kernel<double>, dim3(cmax, B), dim3(256), 0, ctx.stream, dd);
      else
        hipLaunchKernelGGL(tune_fill_kernel<float>, dim3(cmax, B), dim3(256), 0, ctx.stream, dd);
      (void)hipEventRecord(a, ctx.stream);
      rc = factor_batch(ctx, fs, prec, &cfg);
      (void)hipEventRecord(b, ctx.stream);
      if (hipEventSynchronize(b) != hipSuccess) rc = INLA_ERR_HIP;
      float ms = 0;
      if (!rc && r > 0 && hipEventElapsedTime(&ms, a, b) == hipSuccess) tot += ms;
    }
    return tot / std::max(1, reps);
  };
  const size_t nbase = cand.size();
  int dflt = -1;
  double dflt_ms = 0;
  for (size_t c = 0; c < nbase && !rc; ++c) {
    const double avg = time_cfg(cand[c]);
    if (ms_out) ms_out[c] = avg;
    if (!rc && (best < 0 || avg < best_ms)) { best = (int)c; best_ms = avg; }
    if (cand[c].nb == default_config(prec, nf_max).nb && cand[c].tm == default_config(prec, nf_max).tm) { dflt = (int)c; dflt_ms = avg; }
  }
  // the default configuration stays unless another is clearly faster, so that
  // timing noise between near-equal candidates does not change the choice
  if (!rc && dflt >= 0 && best_ms > (1.0 - DEFAULT_MARGIN) * dflt_ms) { best = dflt; best_ms = dflt_ms; }
  if (!rc && ctx.lookahead) {
    TuneCfg la = cand[best];
    la.look = 1;
    cand.push_back(la);
    const double avg = time_cfg(la);
    if (ms_out) ms_out[nbase] = avg;
    // Lookahead must win clearly: the synthetic timing leaves out the rest of
    // an evaluation (assembly, solves, host decisions between passes), in
    // which the overlap has been seen to gain less than it does here.
    if (!rc && avg < (1.0 - LOOKAHEAD_MARGIN) * best_ms) { best = (int)nbase; best_ms = avg; }
  }
  ctx.prof = prof;
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  if (rc) return rc;
  ctx.tune[tune_key(prec, nf_max, B)] = cand[best];
  ++ctx.tune_epoch;
  if (best_out) *best_out = cand[best];
  if (n_cand) *n_cand = (int)cand.size();
  return ctx.check();
}

}  // namespace inla
