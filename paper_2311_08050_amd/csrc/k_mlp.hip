// Learned warm start for the Newton mode: a small multilayer perceptron
//     h1 = GELU(W1 u + b1),  h2 = GELU(W2 h1 + b2),  x0 = W3 h2 + b3
// (u the normalised hyperparameters), trained on modes that the method itself
// produces, with hand-written FP32 forward, backward and Adam kernels.
// GELU is the exact erf form x * (1 + erf(x / sqrt 2)) / 2.
//
// Parameters are one flat FP32 array: W1 (H x I, row-major), b1 (H),
// W2 (H x H), b2 (H), W3 (O x H), b3 (O).
#include <cmath>
#include <cstdint>
#include <type_traits>
#include <vector>

#include "device.hpp"
#include "host.hpp"

namespace inla {

// C(M x N) = A(M x K) * B(K x N) with A(i, k) = A[i*sar + k*sac],
// B(k, j) = B[k*sbr + j*sbc], C(i, j) = C[i*scr + j*scc], on FP32 MFMA
// (v_mfma_f32_16x16x4f32, FP32 accumulate): 64 x 64 tiles per workgroup, 32 x 32
// per wave (2 x 2 blocks of 16 x 16), K in chunks of GKC through two LDS buffers, the
// loads of the next GPF chunks in flight while one is multiplied: the products of a
// small batch are bound by the latency of their chunks (one ahead: 1.4 us each), the
// output layer's by the matrix units.  Tile loads run along whichever index of an
// operand is contiguous, so every layout the network's forward and backward passes use
// is read coalesced, in 16-byte loads (W = 4) where every group of four is aligned and
// inside the operand, else W = 1.  The eight products of a gradient at 256 inputs, 256
// hidden units and 8192 outputs: 207 to 116 us.  Epilogue: + bias[j] (if bias) and what
// EPI says, the tile's rows taken from LDS so that they are written whole.
// With `ksplit` > 1 the K range is split over blockIdx.z and each split writes its
// partial tile to `part` (ksplit x M x N); gemm_epilogue_kernel then sums the splits in
// a fixed order and applies the epilogue (the backward product through the output
// layer has K = n and only B x H outputs).
struct GemmArgs {
  const float *A, *B;
  float *C, *Z;
  const float *bias, *dz;
  int M, N, K;
  int sar, sac, sbr, sbc, scr, scc;
};

__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * 0.39894228040143268f * expf(-0.5f * x * x);
}

// Epilogues: the K split's partial tile, a linear output, a hidden layer's forward
// pass (Z and GELU) and its backward pass (* GELU'(dz)).
enum { EPI_PART, EPI_LIN, EPI_GELU, EPI_DGELU };
template <int EPI>
__device__ __forceinline__ void gemm_store(const GemmArgs &g, int i, int j, float val, float bias, float dz) {
  val += bias;
  auto *c = gptr(g.C) + (size_t)i * g.scr + (size_t)j * g.scc;
  if (EPI == EPI_GELU) {
    gptr(g.Z)[(size_t)i * g.N + j] = val;
    val = gelu_f(val);
  } else if (EPI == EPI_DGELU) {
    val *= gelu_grad_f(dz);
  }
  *c = val;
}

typedef float f4m __attribute__((ext_vector_type(4)));

constexpr int GKC = 32, GLD = 66;   // GLD: conflict-free reads of k = 8 gq + st and writes along k

// One operand's loads: X(x, k) = P[x * sx + k * sk] for x in [x0, x0 + 64) below nx, a
// thread's elements (groups of W = 4 along the contiguous index in 16-byte loads, or
// W = 1) fixed for the whole product.  Indices past the operand are clamped, so that
// no load is conditional; values past nx belong to outputs that are not stored.
constexpr int GPF = 4;   // chunks whose loads are in flight (PF; 1 for a product of one chunk, see gemm())
template <int W> struct TileLoad {
  static constexpr int NL = GKC * 64 / 256 / W;
  const float __attribute__((address_space(1))) *row[NL];
  int kk[NL], lds[NL], kmax, us;
  size_t sk;
  __device__ __forceinline__ void init(const float *p, int sx, int sk_, int x0, int nx, int ke) {
    const bool along_k = sk_ == 1;
    sk = sk_;
    us = along_k ? GLD : 1;
    kmax = along_k ? ke - W : ke - 1;
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int e = q * 256 + (int)threadIdx.x;
      int x;
      if (along_k) { x = e / (GKC / W); kk[q] = e % (GKC / W) * W; } else { kk[q] = e / (64 / W); x = e % (64 / W) * W; }
      row[q] = gptr(p) + (size_t)min(x0 + x, along_k ? nx - 1 : nx - W) * sx;
      lds[q] = kk[q] * GLD + x;
    }
  }
  __device__ __forceinline__ void load(int k0, float (&r)[8]) const {
    typedef float vec __attribute__((ext_vector_type(W)));
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const auto *p = row[q] + (size_t)min(k0 + kk[q], kmax) * sk;
      if constexpr (W == 1) r[q] = *p;
      else {
        const vec v = *(const vec __attribute__((address_space(1))) *)p;
#pragma unroll
        for (int u = 0; u < W; ++u) r[W * q + u] = v[u];
      }
    }
  }
  __device__ __forceinline__ void store(int k0, int ke, const float (&r)[8], float *S) const {
#pragma unroll
    for (int q = 0; q < NL; ++q)
#pragma unroll
      for (int u = 0; u < W; ++u) S[lds[q] + u * us] = k0 + kk[q] < ke ? r[W * q + u] : 0.0f;
  }
};

template <int EPI, int W, int PF>
__global__ __launch_bounds__(256) void mlp_gemm_kernel(GemmArgs g, float *part, int kper) {
  __shared__ float S[4][GKC][GLD];   // A and B, two buffers each; the product's tile
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w >> 1, wn = w & 1, li = lane & 15, gq = lane >> 4;
  const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
  const int kb = blockIdx.z * kper, ke = min(g.K, kb + kper);
  TileLoad<W> A, B;
  A.init(g.A, g.sar, g.sac, i0, g.M, ke);
  B.init(g.B, g.sbc, g.sbr, j0, g.N, ke);
  float ra[PF][8], rb[PF][8];
  f4m acc2[2][2][2];   // even and odd chunks: shorter chains of rounded sums
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc2[0][a][b] = acc2[1][a][b] = f4m{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < PF; ++u)
    if (kb + u * GKC < ke) {
      A.load(kb + u * GKC, ra[u]);
      B.load(kb + u * GKC, rb[u]);
    }
  for (int k1 = kb; k1 < ke; k1 += PF * GKC)
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int k0 = k1 + u * GKC;
      if (k0 >= ke) break;
      // a buffer is written again two chunks on: every wave has passed the barrier of
      // the chunk between, so it has read this one
      A.store(k0, ke, ra[u], &S[2 * (u & 1)][0][0]);
      B.store(k0, ke, rb[u], &S[2 * (u & 1) + 1][0][0]);
      if (k0 + PF * GKC < ke) {
        A.load(k0 + PF * GKC, ra[u]);
        B.load(k0 + PF * GKC, rb[u]);
      }
      __syncthreads();
#pragma unroll
      for (int st = 0; st < GKC / 4; ++st) {
        const int kk = GKC / 4 * gq + st;   // lane group gq supplies k = 8 gq + st at step st
        float av[2], bv[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) av[a] = S[2 * (u & 1)][kk][wm * 32 + a * 16 + li];
#pragma unroll
        for (int b = 0; b < 2; ++b) bv[b] = S[2 * (u & 1) + 1][kk][wn * 32 + b * 16 + li];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc2[u & 1][a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], acc2[u & 1][a][b], 0, 0, 0);
      }
    }
  __syncthreads();
  // lane l holds rows 4 (l / 16) + v, column l % 16 of each 16 x 16 block
  float (*T)[GLD] = S[0];   // 64 rows over both of the first buffers
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) T[wm * 32 + a * 16 + 4 * gq + v][wn * 32 + b * 16 + li] = acc2[0][a][b][v] + acc2[1][a][b][v];
  __syncthreads();
  const int j = j0 + lane, jc = min(j, g.N - 1);
  const float bias = EPI != EPI_PART && g.bias ? gptr(g.bias)[jc] : 0.0f;
  float (*Z)[GLD] = S[2];   // the same rows of dz, loaded together
  if (EPI == EPI_DGELU) {
    float dz[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) dz[u] = gptr(g.dz)[(size_t)min(i0 + w + 4 * u, g.M - 1) * g.N + jc];
#pragma unroll
    for (int u = 0; u < 16; ++u) Z[w + 4 * u][lane] = dz[u];
  }
  float *C = EPI == EPI_PART ? part + (size_t)blockIdx.z * g.M * g.N : nullptr;
#pragma unroll 1
  for (int r = w; r < 64; r += 16) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + r + 4 * u;
      if (i >= g.M || j >= g.N) continue;
      const float val = T[r + 4 * u][lane];
      if (EPI == EPI_PART) gptr(C)[(size_t)i * g.N + j] = val;
      else gemm_store<EPI>(g, i, j, val, bias, EPI == EPI_DGELU ? Z[r + 4 * u][lane] : 0.0f);
    }
  }
}

// Sum of the K splits (fixed order) and the epilogue, one thread per output.
template <int EPI> __global__ __launch_bounds__(64) void gemm_epilogue_kernel(GemmArgs g, const float *part, int ksplit) {
  const int64_t idx = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (idx >= (int64_t)g.M * g.N) return;
  const int i = (int)(idx / g.N), j = (int)(idx % g.N);
  const float bias = g.bias ? gptr(g.bias)[j] : 0.0f, dz = EPI == EPI_DGELU ? gptr(g.dz)[idx] : 0.0f;
  float s = 0.0f;
#pragma unroll 8
  for (int z = 0; z < ksplit; ++z) s += gptr(part)[(size_t)z * g.M * g.N + idx];
  gemm_store<EPI>(g, i, j, s, bias, dz);
}

// K splits of a product: enough workgroups for the chip (about 512) without
// splits shorter than 256: half of that costs a second launch for the sum that takes
// as long as the chunks it saves.
static int gemm_ksplit(int M, int N, int K) {
  const int tiles = ((M + 63) / 64) * ((N + 63) / 64);
  int ks = std::max(1, 512 / std::max(1, tiles));
  ks = std::min(ks, std::max(1, K / 256));
  return ks;
}

// Column sums of the (rows x cols) row-major matrices X into out (the three layers'
// bias gradients) in one launch: a workgroup takes 64 columns, its 16 waves every 16th
// row.  One thread per column was a serial walk by one or a few workgroups (rows = 256,
// cols = 8192 and twice 256: 46 to 6 us together).
struct ColSums {
  const float *X[3];
  float *out[3];
  int cols[3];
};
__global__ __launch_bounds__(1024) void colsum_kernel(ColSums c, int rows) {
  __shared__ float part[16][64];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  int blk = blockIdx.x, m = 0;
  for (; m < 2 && blk >= (c.cols[m] + 63) / 64; ++m) blk -= (c.cols[m] + 63) / 64;
  const int cols = c.cols[m], j = blk * 64 + l, jc = min(j, cols - 1);
  const auto *X = gptr(c.X[m]);
  float s = 0.0f;
#pragma unroll 8
  for (int r = w; r < rows; r += 16) s += X[(size_t)r * cols + jc];
  part[w][l] = s;
  __syncthreads();
  if (w != 0 || j >= cols) return;
  float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int q = 0; q < 16; ++q) t[q & 3] += part[q][l];
  c.out[m][j] = (t[0] + t[1]) + (t[2] + t[3]);
}

// dOut = 2 (out - target) / (B * O); per-block partial sums of the squared error.
__global__ __launch_bounds__(256) void mse_grad_kernel(const float *out, const double *tgt, float *dout, int64_t count,
                                                       float scale, double *part) {
  __shared__ double sh[4];
  double se = 0.0;
  for (int64_t i0 = (int64_t)blockIdx.x * 1024; i0 < count; i0 += (int64_t)gridDim.x * 1024) {
    float o[4];
    double t[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = min(i0 + q * 256 + threadIdx.x, count - 1);
      o[q] = gptr(out)[i];
      t[q] = gptr(tgt)[i];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = i0 + q * 256 + threadIdx.x;
      if (i >= count) continue;
      const float d = o[q] - (float)t[q];
      gptr(dout)[i] = scale * 2.0f * d;
      se += (double)d * d;
    }
  }
  se = block_sum256(se, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = se;
}

// Adam: m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2, p -= lr mhat / (sqrt(vhat) + eps).
__global__ void adam_kernel(float *p, const float *g, float *m, float *v, int count, float lr, float b1, float b2,
                            float c1, float c2, float eps) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Normalised inputs u = (theta - centre) / scale (FP32) and FP32 -> FP64 output
// scatter into per-theta vectors.
__global__ void theta_norm_kernel(const double *theta, int ld, int n_in, const double *centre, const double *scale,
                                  float *u, int B) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= B * n_in) return;
  const int b = i / n_in, c = i % n_in;
  u[i] = (float)((theta[(size_t)b * ld + c] - centre[c]) / scale[c]);
}
__global__ void scatter_modes_kernel(const float *y, int n_out, double *const *x) {
  const int b = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
  if (i < n_out) x[b][i] = (double)y[(size_t)b * n_out + i];
}

// Counter-based initialisation: splitmix64 of (seed, index) -> U(-a, a).
__global__ void init_uniform_kernel(float *p, int count, uint64_t seed, uint64_t offset, float a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  uint64_t z = seed + 0x9E3779B97F4A7C15ull * (offset + (uint64_t)i + 1);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  const double u = (double)(z >> 11) * (1.0 / 9007199254740992.0);
  p[i] = (float)((2.0 * u - 1.0) * a);
}

}  // namespace inla

// ====================================================================== C-ABI
using namespace inla;

namespace inla {
hipStream_t handle_stream(inla_handle *h);   // host.hip
}

struct inla_mlp {
  inla_handle *h = nullptr;
  int I = 0, H = 0, O = 0;
  int64_t P = 0;
  float *params = nullptr, *grad = nullptr, *m = nullptr, *v = nullptr;
  // activations for a batch of up to cap rows
  int cap = 0;
  float *u = nullptr, *z1 = nullptr, *h1 = nullptr, *z2 = nullptr, *h2 = nullptr, *out = nullptr, *dout = nullptr,
        *dh2 = nullptr, *dh1 = nullptr;
  double *part = nullptr;
  float *kpart = nullptr;   // partial products of split-K GEMMs
  size_t kpart_elems = 0;
  double *dtheta = nullptr, *dcentre = nullptr, *dscale = nullptr;
  double **dptrs = nullptr;
  int64_t step = 0;
  size_t off_W1() const { return 0; }
  size_t off_b1() const { return (size_t)H * I; }
  size_t off_W2() const { return off_b1() + H; }
  size_t off_b2() const { return off_W2() + (size_t)H * H; }
  size_t off_W3() const { return off_b2() + H; }
  size_t off_b3() const { return off_W3() + (size_t)O * H; }
};

namespace {

void free_acts(inla_mlp *m) {
  for (float **p : {&m->u, &m->z1, &m->h1, &m->z2, &m->h2, &m->out, &m->dout, &m->dh2, &m->dh1}) {
    if (*p) (void)hipFree(*p);
    *p = nullptr;
  }
  if (m->part) (void)hipFree(m->part);
  if (m->kpart) (void)hipFree(m->kpart);
  if (m->dtheta) (void)hipFree(m->dtheta);
  if (m->dptrs) (void)hipFree(m->dptrs);
  m->part = nullptr;
  m->kpart = nullptr;
  m->kpart_elems = 0;
  m->dtheta = nullptr;
  m->dptrs = nullptr;
  m->cap = 0;
}

int ensure_cap(inla_mlp *m, int B) {
  if (B <= m->cap) return 0;
  (void)hipDeviceSynchronize();
  free_acts(m);
  const int cap = std::max(B, 64);
  const size_t nb = (size_t)cap;
  // split-K workspace: the largest ksplit x M x N over the products of a
  // forward and backward pass at batch `cap` (GEMMs of fewer rows need less)
  size_t kp = 0;
  const int I = m->I, H = m->H, O = m->O;
  const int shapes[][3] = {{cap, H, I}, {cap, H, H}, {cap, O, H}, {O, H, cap}, {cap, H, O}, {H, H, cap}, {H, I, cap}};
  for (const auto &sh : shapes) {
    const int ks = gemm_ksplit(sh[0], sh[1], sh[2]);
    if (ks > 1) kp = std::max(kp, (size_t)ks * sh[0] * sh[1]);
  }
  bool ok = hipMalloc(&m->u, 4 * nb * m->I) == hipSuccess && hipMalloc(&m->z1, 4 * nb * m->H) == hipSuccess &&
            hipMalloc(&m->h1, 4 * nb * m->H) == hipSuccess && hipMalloc(&m->z2, 4 * nb * m->H) == hipSuccess &&
            hipMalloc(&m->h2, 4 * nb * m->H) == hipSuccess && hipMalloc(&m->out, 4 * nb * m->O) == hipSuccess &&
            hipMalloc(&m->dout, 4 * nb * m->O) == hipSuccess && hipMalloc(&m->dh2, 4 * nb * m->H) == hipSuccess &&
            hipMalloc(&m->dh1, 4 * nb * m->H) == hipSuccess &&
            hipMalloc(&m->part, 8 * ((nb * m->O + 255) / 256 + 1)) == hipSuccess &&
            hipMalloc(&m->dtheta, 8 * (nb * 8 + 16)) == hipSuccess && hipMalloc(&m->dptrs, 8 * nb) == hipSuccess &&
            (kp == 0 || hipMalloc(&m->kpart, 4 * kp) == hipSuccess);
  if (!ok) {
    (void)hipGetLastError();
    free_acts(m);
    return INLA_ERR_NOMEM;
  }
  m->cap = cap;
  m->kpart_elems = kp;
  return 0;
}

void gemm(inla_mlp *m, hipStream_t s, const GemmArgs &g) {
  int ks = gemm_ksplit(g.M, g.N, g.K);
  if ((size_t)ks * g.M * g.N > m->kpart_elems) ks = 1;   // never past the workspace
  const int kper = ks > 1 ? ((g.K + ks - 1) / ks + 15) / 16 * 16 : g.K;
  ks = ks > 1 ? (g.K + kper - 1) / kper : 1;
  dim3 grid((g.N + 63) / 64, (g.M + 63) / 64, ks);
  // 16-byte loads: a contiguous index whose length, and the other index's stride, are
  // multiples of four (kper is one of 16), at an aligned address
  auto vec4 = [](const float *p, int sx, int sk, int nx, int K) {
    return ((uintptr_t)p & 15) == 0 && (sk == 1 ? sx % 4 == 0 && K % 4 == 0 : sx == 1 && sk % 4 == 0 && nx % 4 == 0);
  };
  const bool vec = vec4(g.A, g.sar, g.sac, g.M, g.K) && vec4(g.B, g.sbc, g.sbr, g.N, g.K);
  auto launch = [&](auto epi) {
    constexpr int E = decltype(epi)::value;
    if (ks == 1) {
      // one chunk: the kernel without its pipeline, whose unrolled code a launch of one
      // workgroup waits for (4-16-33 network, one row: 31.2 to 28.7 us for the three)
      if (kper <= GKC) {
        if (vec) hipLaunchKernelGGL((mlp_gemm_kernel<E, 4, 1>), grid, dim3(256), 0, s, g, nullptr, kper);
        else hipLaunchKernelGGL((mlp_gemm_kernel<E, 1, 1>), grid, dim3(256), 0, s, g, nullptr, kper);
      } else {
        if (vec) hipLaunchKernelGGL((mlp_gemm_kernel<E, 4, GPF>), grid, dim3(256), 0, s, g, nullptr, kper);
        else hipLaunchKernelGGL((mlp_gemm_kernel<E, 1, GPF>), grid, dim3(256), 0, s, g, nullptr, kper);
      }
      return;
    }
    const int64_t cnt = (int64_t)g.M * g.N;
    if (vec) hipLaunchKernelGGL((mlp_gemm_kernel<EPI_PART, 4, GPF>), grid, dim3(256), 0, s, g, m->kpart, kper);
    else hipLaunchKernelGGL((mlp_gemm_kernel<EPI_PART, 1, GPF>), grid, dim3(256), 0, s, g, m->kpart, kper);
    hipLaunchKernelGGL(gemm_epilogue_kernel<E>, dim3((unsigned)((cnt + 63) / 64)), dim3(64), 0, s, g,
                       (const float *)m->kpart, ks);
  };
  if (g.Z) launch(std::integral_constant<int, EPI_GELU>());
  else if (g.dz) launch(std::integral_constant<int, EPI_DGELU>());
  else launch(std::integral_constant<int, EPI_LIN>());
}

GemmArgs ga(const float *A, int sar, int sac, const float *B, int sbr, int sbc, float *C, int scr, int scc, int M,
            int N, int K) {
  GemmArgs g{};
  g.A = A; g.B = B; g.C = C; g.M = M; g.N = N; g.K = K;
  g.sar = sar; g.sac = sac; g.sbr = sbr; g.sbc = sbc; g.scr = scr; g.scc = scc;
  return g;
}

// Forward pass on m->u (B x I) into m->out (B x O), keeping pre-activations.
void forward(inla_mlp *m, hipStream_t s, int B) {
  const float *P = m->params;
  GemmArgs g = ga(m->u, m->I, 1, P + m->off_W1(), 1, m->I, m->h1, m->H, 1, B, m->H, m->I);
  g.bias = P + m->off_b1(); g.Z = m->z1;
  gemm(m, s, g);
  g = ga(m->h1, m->H, 1, P + m->off_W2(), 1, m->H, m->h2, m->H, 1, B, m->H, m->H);
  g.bias = P + m->off_b2(); g.Z = m->z2;
  gemm(m, s, g);
  g = ga(m->h2, m->H, 1, P + m->off_W3(), 1, m->H, m->out, m->O, 1, B, m->O, m->H);
  g.bias = P + m->off_b3();
  gemm(m, s, g);
}

// Backward pass from m->dout into G (flat, same layout as params).
void backward(inla_mlp *m, hipStream_t s, int B, float *G) {
  const float *P = m->params;
  const int I = m->I, H = m->H, O = m->O;
  // dW3 (O x H) = dout^T (O x B) * h2 (B x H)
  gemm(m, s, ga(m->dout, 1, O, m->h2, H, 1, G + m->off_W3(), H, 1, O, H, B));
  // dh2 (B x H) = dout (B x O) * W3 (O x H), then * GELU'(z2)
  GemmArgs g = ga(m->dout, O, 1, P + m->off_W3(), H, 1, m->dh2, H, 1, B, H, O);
  g.dz = m->z2;
  gemm(m, s, g);
  gemm(m, s, ga(m->dh2, 1, H, m->h1, H, 1, G + m->off_W2(), H, 1, H, H, B));
  g = ga(m->dh2, H, 1, P + m->off_W2(), H, 1, m->dh1, H, 1, B, H, H);
  g.dz = m->z1;
  gemm(m, s, g);
  gemm(m, s, ga(m->dh1, 1, H, m->u, I, 1, G + m->off_W1(), I, 1, H, I, B));
  const ColSums c = {{m->dout, m->dh2, m->dh1}, {G + m->off_b3(), G + m->off_b2(), G + m->off_b1()}, {O, H, H}};
  hipLaunchKernelGGL(colsum_kernel, dim3((O + 63) / 64 + 2 * ((H + 63) / 64)), dim3(1024), 0, s, c, B);
}

// The gradient goes to `grad` (m->grad or the caller's).
int loss_and_grad(inla_mlp *m, int B, const float *x_in, const double *target, double *loss, float *grad) {
  hipStream_t s = handle_stream(m->h);
  int rc = ensure_cap(m, B);
  if (rc) return rc;
  if (hipMemcpyAsync(m->u, x_in, 4 * (size_t)B * m->I, hipMemcpyDeviceToDevice, s) != hipSuccess) return INLA_ERR_HIP;
  forward(m, s, B);
  const int cnt = B * m->O, nblk = std::min((cnt + 1023) / 1024, 1024);
  hipLaunchKernelGGL(mse_grad_kernel, dim3(nblk), dim3(256), 0, s, m->out, target, m->dout, (int64_t)cnt,
                     1.0f / (float)cnt, m->part);
  backward(m, s, B, grad);
  if (loss) {
    std::vector<double> h(nblk);
    if (hipMemcpyAsync(h.data(), m->part, 8 * nblk, hipMemcpyDeviceToHost, s) != hipSuccess) return INLA_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return INLA_ERR_HIP;
    double t = 0.0;
    for (double v : h) t += v;
    *loss = t / cnt;
  }
  return hipGetLastError() == hipSuccess ? 0 : INLA_ERR_HIP;
}

}  // namespace

extern "C" {

int inla_mlp_create(inla_handle *h, int32_t n_in, int32_t n_hidden, int32_t n_out, uint64_t seed, inla_mlp **out) {
  if (!h) return -1;
  if (n_in < 1) return -2;
  if (n_hidden < 1) return -3;
  if (n_out < 1) return -4;
  if (!out) return -6;
  *out = nullptr;
  inla_mlp *m = new (std::nothrow) inla_mlp();
  if (!m) return INLA_ERR_NOMEM;
  m->h = h;
  m->I = n_in; m->H = n_hidden; m->O = n_out;
  m->P = (int64_t)n_hidden * n_in + n_hidden + (int64_t)n_hidden * n_hidden + n_hidden + (int64_t)n_out * n_hidden + n_out;
  const size_t pb = 4 * (size_t)m->P;
  if (hipMalloc(&m->params, pb) != hipSuccess || hipMalloc(&m->grad, pb) != hipSuccess ||
      hipMalloc(&m->m, pb) != hipSuccess || hipMalloc(&m->v, pb) != hipSuccess ||
      hipMalloc(&m->dcentre, 8 * 32) != hipSuccess || hipMalloc(&m->dscale, 8 * 32) != hipSuccess) {
    (void)hipGetLastError();
    inla_mlp_destroy(m);
    return INLA_ERR_NOMEM;
  }
  hipStream_t s = handle_stream(h);
  // uniform(-sqrt(6 / fan_in), +) weights (He-style for GELU), zero biases
  struct Seg { size_t off, cnt; float a; };
  const Seg segs[] = {{m->off_W1(), (size_t)m->H * m->I, sqrtf(6.0f / m->I)},
                      {m->off_b1(), (size_t)m->H, 0.0f},
                      {m->off_W2(), (size_t)m->H * m->H, sqrtf(6.0f / m->H)},
                      {m->off_b2(), (size_t)m->H, 0.0f},
                      {m->off_W3(), (size_t)m->O * m->H, sqrtf(3.0f / m->H)},
                      {m->off_b3(), (size_t)m->O, 0.0f}};
  for (const Seg &g : segs)
    hipLaunchKernelGGL(init_uniform_kernel, dim3((g.cnt + 255) / 256), dim3(256), 0, s, m->params + g.off, (int)g.cnt,
                       seed, (uint64_t)g.off, g.a);
  (void)hipMemsetAsync(m->m, 0, pb, s);
  (void)hipMemsetAsync(m->v, 0, pb, s);
  if (hipStreamSynchronize(s) != hipSuccess) { inla_mlp_destroy(m); return INLA_ERR_HIP; }
  *out = m;
  return INLA_OK;
}

int inla_mlp_destroy(inla_mlp *m) {
  if (!m) return INLA_OK;
  (void)hipDeviceSynchronize();
  free_acts(m);
  for (float *p : {m->params, m->grad, m->m, m->v}) if (p) (void)hipFree(p);
  if (m->dcentre) (void)hipFree(m->dcentre);
  if (m->dscale) (void)hipFree(m->dscale);
  delete m;
  return INLA_OK;
}

int inla_mlp_num_params(const inla_mlp *m, int64_t *count) {
  if (!m) return -1;
  if (!count) return -2;
  *count = m->P;
  return INLA_OK;
}

int inla_mlp_get_params(inla_mlp *m, float *dst) {
  if (!m) return -1;
  if (!dst) return -2;
  hipStream_t s = handle_stream(m->h);
  if (hipMemcpyAsync(dst, m->params, 4 * (size_t)m->P, hipMemcpyDeviceToDevice, s) != hipSuccess) return INLA_ERR_HIP;
  return hipStreamSynchronize(s) == hipSuccess ? INLA_OK : INLA_ERR_HIP;
}

int inla_mlp_set_params(inla_mlp *m, const float *src) {
  if (!m) return -1;
  if (!src) return -2;
  hipStream_t s = handle_stream(m->h);
  if (hipMemcpyAsync(m->params, src, 4 * (size_t)m->P, hipMemcpyDeviceToDevice, s) != hipSuccess) return INLA_ERR_HIP;
  (void)hipMemsetAsync(m->m, 0, 4 * (size_t)m->P, s);
  (void)hipMemsetAsync(m->v, 0, 4 * (size_t)m->P, s);
  m->step = 0;
  return hipStreamSynchronize(s) == hipSuccess ? INLA_OK : INLA_ERR_HIP;
}

int inla_mlp_forward(inla_mlp *m, int32_t B, const float *x_in, float *y_out) {
  if (!m) return -1;
  if (B < 0) return -2;
  if (B == 0) return INLA_OK;
  if (!x_in) return -3;
  if (!y_out) return -4;
  hipStream_t s = handle_stream(m->h);
  int rc = ensure_cap(m, B);
  if (rc) return rc;
  if (hipMemcpyAsync(m->u, x_in, 4 * (size_t)B * m->I, hipMemcpyDeviceToDevice, s) != hipSuccess) return INLA_ERR_HIP;
  forward(m, s, B);
  if (hipMemcpyAsync(y_out, m->out, 4 * (size_t)B * m->O, hipMemcpyDeviceToDevice, s) != hipSuccess) return INLA_ERR_HIP;
  return hipStreamSynchronize(s) == hipSuccess ? INLA_OK : INLA_ERR_HIP;
}

int inla_mlp_grad(inla_mlp *m, int32_t B, const float *x_in, const double *target, float *grad_out, double *loss) {
  if (!m) return -1;
  if (B < 1) return -2;
  if (!x_in) return -3;
  if (!target) return -4;
  int rc = loss_and_grad(m, B, x_in, target, loss, grad_out ? grad_out : m->grad);
  if (rc) return rc;
  return hipStreamSynchronize(handle_stream(m->h)) == hipSuccess ? INLA_OK : INLA_ERR_HIP;
}

int inla_mlp_train_step(inla_mlp *m, int32_t B, const float *x_in, const double *target, float lr, double *loss) {
  if (!m) return -1;
  if (B < 1) return -2;
  if (!x_in) return -3;
  if (!target) return -4;
  if (!(lr > 0.0f)) return -5;
  int rc = loss_and_grad(m, B, x_in, target, loss, m->grad);
  if (rc) return rc;
  hipStream_t s = handle_stream(m->h);
  m->step += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.0f - powf(b1, (float)m->step), c2 = 1.0f - powf(b2, (float)m->step);
  hipLaunchKernelGGL(adam_kernel, dim3((m->P + 255) / 256), dim3(256), 0, s, m->params, m->grad, m->m, m->v,
                     (int)m->P, lr, b1, b2, c1, c2, 1e-8f);
  return hipGetLastError() == hipSuccess ? INLA_OK : INLA_ERR_HIP;
}

int inla_mlp_predict_modes(inla_mlp *m, int32_t B, const double *theta, int32_t ldtheta, const double *centre,
                           const double *scale, double *const *x) {
  if (!m) return -1;
  if (B < 0) return -2;
  if (B == 0) return INLA_OK;
  if (!theta) return -3;
  if (ldtheta < m->I) return -4;
  if (!centre) return -5;
  if (!scale) return -6;
  if (!x) return -7;
  hipStream_t s = handle_stream(m->h);
  int rc = ensure_cap(m, B);
  if (rc) return rc;
  if (ldtheta > 8) return INLA_ERR_UNSUPPORTED;   // staging holds 8 doubles per theta
  if (hipMemcpyAsync(m->dtheta, theta, 8 * (size_t)B * ldtheta, hipMemcpyHostToDevice, s) != hipSuccess)
    return INLA_ERR_HIP;
  if (hipMemcpyAsync(m->dcentre, centre, 8 * m->I, hipMemcpyHostToDevice, s) != hipSuccess ||
      hipMemcpyAsync(m->dscale, scale, 8 * m->I, hipMemcpyHostToDevice, s) != hipSuccess ||
      hipMemcpyAsync(m->dptrs, x, 8 * (size_t)B, hipMemcpyHostToDevice, s) != hipSuccess)
    return INLA_ERR_HIP;
  hipLaunchKernelGGL(theta_norm_kernel, dim3((B * m->I + 255) / 256), dim3(256), 0, s, m->dtheta, ldtheta, m->I,
                     m->dcentre, m->dscale, m->u, B);
  forward(m, s, B);
  hipLaunchKernelGGL(scatter_modes_kernel, dim3((m->O + 255) / 256, B), dim3(256), 0, s, m->out, m->O, m->dptrs);
  return hipStreamSynchronize(s) == hipSuccess ? INLA_OK : INLA_ERR_HIP;
}

}  // extern "C"
