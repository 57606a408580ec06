// Shared device-side definitions of the dense-INLA HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace inla {

// Tile geometry of the blocked Cholesky.
constexpr int NBI = 64;      // diagonal block / inner panel width
constexpr int PADN = 128;    // matrix orders and border heights are padded to this
constexpr int KC = 16;       // K chunk staged through LDS by the MFMA kernels

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

// Global-address-space views.  Pointers read out of descriptor structs are
// generic; without the cast the compiler emits flat loads, which also count
// against the LDS wait counter and so serialise prefetch with LDS reads.
typedef __attribute__((address_space(1))) double gdouble;
typedef __attribute__((address_space(1))) const double gcdouble;
typedef __attribute__((address_space(1))) d2 gd2;
typedef __attribute__((address_space(1))) const d2 gcd2;
template <typename T> __device__ __forceinline__ __attribute__((address_space(1))) T *gptr(T *p) {
  return (__attribute__((address_space(1))) T *)p;
}

// One matrix being factored by the bordered blocked Cholesky.  Columns [0, nf)
// are factored; rows [nf, nrows) are border rows carried along (they end up as
// G L^{-T}); the trailing update also maintains the Schur block of the border
// for columns [nf, ncols).  Column-major, leading dimension ld >= nrows.
struct FactorDesc {
  void *A;         // double or float elements (the factorisation's storage type)
  void *linv;      // (nf / NBI) x NBI x NBI: inverse of every diagonal block (col-major)
  int *info;       // first failing pivot (1-based), 0 if none
  int ld;
  int nf;          // columns to factor (multiple of PADN)
  int nrows;       // multiple of PADN
  int ncols;       // nf <= ncols <= nrows, multiple of PADN
  int id_row0;     // first row of an identity border block (INT_MAX if none)
  int ne;          // end of the block columns with real columns; beyond it [ne, nf) is
                   // identity padding (set by factor_batch)
  // packed BF16 copies of the current panel for the trailing updates with BF16
  // MFMA, one or two slots (by panel parity).  An entry holds the eight values of
  // one row at k = p0 + 8 g .. p0 + 8 g + 7 (16 bytes, an MFMA operand); plane q,
  // group g, row r >= pend (the panel's end, packed_panel) is entry
  // pbf[slot + (q G + g) prows + r - pend], G = min(nb, nf) / 8 groups.
  // One plane: the values rounded to BF16, rows [pend, nf).  Three planes: hi,
  // mid and lo parts that add up to the FP32 value, rows [pend, nrows).
  int prows;
  void *pbf;
  int64_t pbf_slot;  // entries from one slot to the other (0: one slot)
};

// Likelihood / prior kinds (values match the C header).
enum { LIK_GAUSSIAN = 0, LIK_POISSON = 1 };
enum { PRIOR_DENSE = 0, PRIOR_EXPCOV = 1, PRIOR_KRON = 2 };

// Per-theta model and workspace description used by the assembly, solve and
// reduction kernels.
struct ThetaDesc {
  // model (device pointers owned by the caller)
  const double *y, *E, *C, *e, *coords, *Quser;
  int n, k, lik, prior, n_s, n_t, ldquser;
  int n_pad;       // round_up(n, PADN)
  double tau, rho, delta, lpar;   // prior parameters; lpar = sigma^2 or beta0
  // workspace (owned by the library)
  double *Qp; int ldqp;           // prior precision, n_pad x n_pad, lower, identity padded
  void *W; int ldw; int Nw; int Ncw;    // big working matrix (double or float): Nw rows, Ncw columns
  double *S; int lds; int Ns; int k_pad;   // small (kriging) system working matrix
  double *P; int ldp; int Np; int ns_pad;  // prior-build working matrix
  // structured prior pass (behind P): KRON n_t matrices of kN x kN, the
  // constraint rows in the temporal eigenbasis (Ct) and the basis's cosines;
  // EXPCOV the rows C L (Ct, k x n_pad)
  double *K; int kN;
  double *Ct, *ctab;
  double *x;       // current iterate / linearisation point [n_pad]
  double *r;       // right-hand side / new iterate [n_pad]
  double *xn;      // refined new iterate [n_pad] (mixed precision)
  double *z;       // residual / forward-solve vector [n_pad] (mixed precision)
  double *lam;     // [k_pad] kriging multipliers
  double *dlam;    // [k_pad] multiplier correction (mixed precision)
  double *rtwo;    // [k_pad] constraint residual e - C x (mixed precision)
  double *part;    // [2 * ldw] per-column partial sums (loglik, x'Qx)
  double *dres;    // [16] per-theta device results (see DRES_*)
  void *linv;      // inverses of the big factor's 64 x 64 diagonal blocks (factor storage type)
  double *linv_s;  // the same for the kriging factor
  double *u;       // forward-solve output / refinement correction [n_pad]
  double *symv;    // partial sums of Q_prior v from its lower triangle: P
                   // ((n_pad / 64) x n_pad, block column J's part of row i at
                   // J n_pad + i), then D [n_pad] (the transposed part); between two
                   // of them the border's partial sums, n_pad / 256 x k_pad
  double *out;     // caller's output vector (mode or variances), device
  // variational-Bayes mean correction: with vb_var set, the likelihood terms
  // are expectations over eta ~ N(eta(x), vb_var[i]) by ngh-point Gauss-Hermite
  // quadrature (gh: nodes, then weights divided by sqrt(pi))
  const double *vb_var;
  const double *gh;
  int ngh;
  // general design matrix (m > 0; m == 0 means A = I): the caller's CSR, its
  // CSC and the lower pattern of A^T A (column c: entries patp[c] .. patp[c+1],
  // entry e in row patr[e] with terms patt[e] .. patt[e+1] of coefficient
  // tcoef[q] = A_{i r} A_{i c} for observation tobs[q]); per-observation
  // workspace: A x, the likelihood terms g, W and log pi(y_i | eta_i)
  int m;
  const int *A_rowptr, *A_col;
  const double *A_val;
  const int *cscp, *csci;
  const double *cscv;
  const int *patp, *patr, *patt, *tobs;
  const double *tcoef;
  double *obs_ax, *obs_g, *obs_W, *obs_ll;
};

// Per-theta device result slots.
enum {
  DRES_LOGDET_L = 0,   // 2 sum log L_ii of the big factor (first n pivots)
  DRES_LOGDET_S = 1,   // 2 sum log of the kriging factor (first k pivots)
  DRES_WNORM2 = 2,     // ||L_S^{-1} (C x_u - e)||^2
  DRES_STEP = 3,       // ||x_new - x||_inf
  DRES_SCALE = 4,      // max(1, ||x_new||_inf)
  DRES_XQX = 5,
  DRES_LOGLIK = 6,
  DRES_NONFINITE = 7,  // 1 if a non-finite value was met
  DRES_RANK = 8,       // 1 if the kriging system is numerically singular
  DRES_IR_DX = 9,      // last refinement correction ||dx||_inf
  DRES_IR_X = 10,      // max(1, ||x||_inf) of the refined iterate
  DRES_COUNT = 16
};

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
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

// sqrt(x) and 1 / sqrt(x) for x > 0 by Goldschmidt's coupled iteration
// (g -> sqrt(x), h -> 1 / (2 sqrt(x)), each step squaring the relative error
// r = 1/2 - g h) from the hardware reciprocal square root estimate; two steps
// take the estimate's error below the FP64 rounding level.
__device__ __forceinline__ void sqrt_rsqrt(double x, double &sq, double &rs) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
  }
  sq = g;
  rs = 2.0 * h;
}

// Deterministic sum over a 256-thread block (fixed pairing order).
__device__ __forceinline__ double block_sum256(double v, double *sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  __syncthreads();
  return t;
}
__device__ __forceinline__ double block_max256(double v, double *sh) {
  v = wave_max(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
  __syncthreads();
  return t;
}

}  // namespace inla
