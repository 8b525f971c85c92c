// Loop surrogate: a multilayer perceptron with GELU activations that maps
// features of (q, Lambda, channel, dR) to one compact loop block, with its
// training (mean-squared loss, reverse-mode gradient, Adam).
//
//   z_l = a_{l-1} W_l^T + b_l,  a_l = GELU(z_l) (not after the last layer),
//   GELU(x) = x Phi(x) = x (1 + erf(x / sqrt 2)) / 2,
//   loss = mean over batch and outputs of (y - t)^2.
//
// All matrix products go through one FP32 GEMM on the matrix cores
// (v_mfma_f32_32x32x2_f32: FP32 operands, FP32 accumulation) whose operands may
// be read transposed, so that the forward product, the data gradient
// dA = dZ W and the weight gradient dW = dZ^T A share it.  The products are
// small (2048 x 256 x 256 is 0.27 GFLOP, 1.8 us at the 151 TFLOP/s that a large
// FP32 product reaches here), so a 32 x 64 tile per workgroup fills the chip,
// four groups of two waves share its K range (summed in LDS in a fixed order),
// and what went through kernels of its own is done in the epilogues: bias and
// GELU, the loss and its gradient, GELU', the bias gradient.  The weight
// gradient's K range is also split over workgroups where it has few tiles.  One
// loss gradient, 2048 rows of 52-256-256-256-2592: 2.80 -> 0.19 ms against the
// FP32 vector kernel with 64 x 64 tiles.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "kernels.h"

namespace tufrg {

namespace {

constexpr int GM = 32, GN = 64, GK = 16;  // tile, K step of a group
constexpr int GG = 4;                     // groups of two waves sharing the K range
constexpr int GPA = GM + 4, GPB = GN + 4; // LDS row strides (16-byte rows; the k-contiguous stores two-way at most)
constexpr int GTHR = 128 * GG;

typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ inline float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ inline float gelu_d(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * expf(-0.5f * x * x) * 0.39894228040143268f;
}

// NX x GK values of an operand into registers: element (x, k) at x ld + k (KC:
// k contiguous) or k ld + x; 128 threads, NX / 8 values each.  Loads without
// branches, so that they stay in flight during the products: addresses outside
// are moved inside, the values zeroed when they are staged.  VEC: 16-byte loads
// (base and row length allow them; then no group of four crosses an edge).
template <int NX, bool KC, bool VEC>
__device__ __forceinline__ void gemm_fetch(const float *__restrict__ p, int ld, int x0, int X, int k0, int K, int t,
                                           float (&v)[NX / 8]) {
#pragma unroll
  for (int i = 0; i < NX / 32; ++i) {
    const int e = (t + 128 * i) * 4;
    const int x = KC ? x0 + e / GK : x0 + e % NX, k = KC ? k0 + e % GK : k0 + e / NX;
    if constexpr (VEC) {
      const int xc = min(x, KC ? X - 1 : X - 4), kc = min(k, KC ? K - 4 : K - 1);
      const float4 f = *(const float4 *)(p + (KC ? (size_t)xc * ld + kc : (size_t)kc * ld + xc));
      v[4 * i] = f.x;
      v[4 * i + 1] = f.y;
      v[4 * i + 2] = f.z;
      v[4 * i + 3] = f.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int xc = min(KC ? x : x + j, X - 1), kc = min(KC ? k + j : k, K - 1);
        v[4 * i + j] = p[KC ? (size_t)xc * ld + kc : (size_t)kc * ld + xc];
      }
    }
  }
}

// the same values to LDS, s[k][x] with row stride ps, zero outside
template <int NX, bool KC>
__device__ __forceinline__ void gemm_stage(float *s, int ps, int x0, int X, int k0, int K, int t,
                                           const float (&v)[NX / 8]) {
#pragma unroll
  for (int i = 0; i < NX / 32; ++i) {
    const int e = (t + 128 * i) * 4;
    const int x = KC ? x0 + e / GK : x0 + e % NX, k = KC ? k0 + e % GK : k0 + e / NX;
    float z[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) z[j] = (KC ? x < X && k + j < K : x + j < X && k < K) ? v[4 * i + j] : 0.f;
    if constexpr (KC) {
#pragma unroll
      for (int j = 0; j < 4; ++j) s[(e % GK + j) * ps + e / GK] = z[j];
    } else {
      *(float4 *)(s + (e / NX) * ps + e % NX) = make_float4(z[0], z[1], z[2], z[3]);
    }
  }
}

}  // namespace

// One tile of C[m][n] = sum_k A(m, k) B(k, n) with the epilogue p.epi.
// A(m, k) = TA ? A[k lda + m] : A[m lda + k];  B(k, n) = TB ? B[n ldb + k] : B[k ldb + n]
template <bool TA, bool TB, bool VEC>
__device__ __forceinline__ void gemm_tile(const GemmF32 &p, int b, float *smem, double *sred) {
  const int bid = b;
  const int nx = (p.N + GN - 1) / GN, ny = (p.M + GM - 1) / GM;
  const int n0 = (b % nx) * GN;
  b /= nx;
  const int m0 = (b % ny) * GM, split = b / ny;
  const int tid = threadIdx.x, lane = tid & 63, g = tid >> 7, t = tid & 127, wn = (t >> 6) * 32;
  const int kper = ((p.K + p.splits - 1) / p.splits + GK * GG - 1) / (GK * GG) * (GK * GG);
  const int ks = split * kper, ke = min(p.K, ks + kper);
  const int nit = (ke - ks + GK * GG - 1) / (GK * GG);
  // groups that have any K (the others would load and add zeros: 16384 x 11 x 256 took
  // 16.1 us with all four, 12.9 so); with 16-byte loads, few of which are ever idle, all
  const int ng = VEC ? GG : min(GG, max(1, (ke - ks + GK - 1) / GK));
  const bool in = VEC || g < ng;
  // LDS offsets of this group's staging, double-buffered: A, then B
  constexpr int BUF = GK * (GPA + GPB);
  const int so = 2 * g * BUF;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  float colsum = 0.f;
  const bool cs = p.db != nullptr && n0 == 0;  // the sums over k of A: the bias gradient
  float fa[GM / 8], fb[GN / 8];
  auto fetch = [&](int it) {
    const int k0 = ks + (it * GG + g) * GK;
    gemm_fetch<GM, !TA, VEC>(p.A, p.lda, m0, p.M, k0, ke, t, fa);
    gemm_fetch<GN, TB, VEC>(p.B, p.ldb, n0, p.N, k0, ke, t, fb);
  };
  if (nit > 0 && in) fetch(0);
  for (int it = 0; it < nit; ++it) {
    const int bf = it & 1;
    const int k0 = ks + (it * GG + g) * GK;
    if (in) {
      gemm_stage<GM, !TA>(smem + so + bf * BUF, GPA, m0, p.M, k0, ke, t, fa);
      gemm_stage<GN, TB>(smem + so + bf * BUF + GK * GPA, GPB, n0, p.N, k0, ke, t, fb);
    }
    __syncthreads();  // one barrier per step: the other buffer is free since the last one
    if (!in) continue;
    if (it + 1 < nit) fetch(it + 1);
    const int ao = so + bf * BUF + (lane >> 5) * GPA + (lane & 31);
    const int bo = so + bf * BUF + GK * GPA + (lane >> 5) * GPB + wn + (lane & 31);
#pragma unroll
    for (int k = 0; k < GK; k += 2)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(smem[ao + k * GPA], smem[bo + k * GPB], acc, 0, 0, 0);
    if (cs && t < GM) {
#pragma unroll
      for (int k = 0; k < GK; ++k) colsum += smem[so + bf * BUF + k * GPA + t];
    }
  }
  __syncthreads();
  // the groups' tiles (element (8 (r / 4) + 4 (lane / 32) + r % 4, lane % 32) of a wave's
  // 32 x 32), then their sum in group order
  if (in)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      smem[(g * GM + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * GN + wn + (lane & 31)] = acc[r];
  __syncthreads();
  double e2 = 0.0;
#pragma unroll
  for (int i = 0; i < GM * GN / GTHR; ++i) {
    const int e = tid + GTHR * i, m = m0 + e / GN, n = n0 + e % GN;
    float v = smem[e];
#pragma unroll
    for (int h = 1; h < GG; ++h)
      if (h < ng) v += smem[h * GM * GN + e];
    if (m < p.M && n < p.N) {
      const size_t o = (size_t)m * p.N + n;
      if (p.epi == GEMM_BIAS || p.epi == GEMM_GELU || p.epi == GEMM_LOSS) v += p.bias[n];
      if (p.epi == GEMM_GELU) {
        p.Z[o] = v;
        v = gelu_f(v);
      } else if (p.epi == GEMM_GELU_BWD) {
        v *= gelu_d(p.Z[o]);
      } else if (p.epi == GEMM_LOSS) {
        const float d = v - p.T[o];
        v = (float)(2.0 * p.inv) * d;
        e2 += (double)d * d;
      }
      p.C[(size_t)split * p.M * p.N + o] = v;
    }
  }
  if (p.epi == GEMM_LOSS) {
    for (int off = 32; off > 0; off >>= 1) e2 += __shfl_down(e2, off);
    if (lane == 0) sred[tid >> 6] = e2;
    __syncthreads();
    if (tid == 0) {
      double sum = 0.0;
      for (int w = 0; w < GTHR / 64; ++w) sum += sred[w];
      p.loss_part[bid] = sum * p.inv;
    }
  }
  if (cs) {
    __syncthreads();
    if (t < GM) smem[g * GM + t] = colsum;
    __syncthreads();
    if (tid < GM && m0 + tid < p.M) {
      float v = smem[tid];
      for (int h = 1; h < GG; ++h) v += smem[h * GM + tid];
      p.db[(size_t)split * p.M + m0 + tid] = v;
    }
  }
}

// FWD: forward products (A row-major, B transposed), one per launch; else the
// two products of a layer's backward pass in one launch, the first nblk0
// workgroups the data gradient, the rest the weight gradient (A transposed): the
// longest first (K 2592 against a range of 2048 rows in the widest layer)
template <bool FWD, bool VEC>
__global__ __launch_bounds__(GTHR) void gemm_f32_kernel(GemmF32 p0, GemmF32 p1, int nblk0) {
  __shared__ __align__(16) float smem[2 * GG * GK * (GPA + GPB)];  // staging, then the groups' tiles
  __shared__ double sred[GTHR / 64];
  static_assert(GG * GM * GN <= 2 * GG * GK * (GPA + GPB), "the tiles of the groups reuse the staging");
  if constexpr (FWD) {
    gemm_tile<false, true, VEC>(p0, blockIdx.x, smem, sred);
  } else {
    if ((int)blockIdx.x < nblk0)
      gemm_tile<false, false, VEC>(p1, blockIdx.x, smem, sred);
    else
      gemm_tile<true, false, VEC>(p0, blockIdx.x - nblk0, smem, sred);
  }
}

int gemm_f32_blocks(const GemmF32 &p) { return ((p.N + GN - 1) / GN) * ((p.M + GM - 1) / GM) * p.splits; }

// 16-byte loads: base, row lengths and (by the row lengths) the contiguous
// extents are multiples of four values
static bool gemm_vec(const GemmF32 &p) {
  const int ca = p.tA ? p.M : p.K, cb = p.tB ? p.K : p.N;
  return ((p.lda | p.ldb | ca | cb) & 3) == 0 && (((uintptr_t)p.A | (uintptr_t)p.B) & 15) == 0;
}

static bool gemm_ok(const GemmF32 &p) {
  // an epilogue needs the whole sum; the fetches clamp into at least one row and column
  return p.M >= 1 && p.N >= 1 && p.K >= 1 && p.splits >= 1 && p.A && p.B && p.C &&
         (p.splits == 1 || p.epi == GEMM_PLAIN);
}

hipError_t launch_gemm_f32(const GemmF32 &p, hipStream_t st) {
  if (!gemm_ok(p) || p.tA || !p.tB) return hipErrorInvalidValue;
  const dim3 grid(gemm_f32_blocks(p)), block(GTHR);
  if (gemm_vec(p))
    hipLaunchKernelGGL((gemm_f32_kernel<true, true>), grid, block, 0, st, p, p, 0);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<true, false>), grid, block, 0, st, p, p, 0);
  return hipGetLastError();
}

hipError_t launch_gemm_f32_bwd(const GemmF32 &w, const GemmF32 *d, hipStream_t st) {
  if (!gemm_ok(w) || !w.tA || w.tB || (d && (!gemm_ok(*d) || d->tA || d->tB))) return hipErrorInvalidValue;
  const int n0 = d ? gemm_f32_blocks(*d) : 0;
  const dim3 grid(n0 + gemm_f32_blocks(w)), block(GTHR);
  if (gemm_vec(w) && (!d || gemm_vec(*d)))
    hipLaunchKernelGGL((gemm_f32_kernel<false, true>), grid, block, 0, st, w, d ? *d : w, n0);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<false, false>), grid, block, 0, st, w, d ? *d : w, n0);
  return hipGetLastError();
}

// grad[i] = sum over the splits of a layer's weight or bias gradient, in
// order, and the loss from its workgroup sums (one workgroup): blocks [0, nb)
// of 256 elements of the split parts, then the loss
__global__ __launch_bounds__(256) void grad_reduce_kernel(GradParts gp, const double *__restrict__ loss_part,
                                                          int n_loss, double *__restrict__ loss) {
  if (blockIdx.x == gridDim.x - 1) {
    __shared__ double red[256];
    double a = 0.0;
    for (int i = threadIdx.x; i < n_loss; i += 256) a += loss_part[i];
    red[threadIdx.x] = a;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
      if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
      __syncthreads();
    }
    if (threadIdx.x == 0) *loss += red[0];
    return;
  }
  int b = blockIdx.x, l = 0;
  while (l + 1 < gp.n && b >= gp.part[l + 1].block0) ++l;
  const auto &q = gp.part[l];
  const long long i = (long long)(b - q.block0) * 256 + threadIdx.x;
  if (i >= q.len) return;
  float v = q.src[i];
  for (int s = 1; s < q.splits; ++s) v += q.src[s * q.len + i];
  q.dst[i] = v;
}

hipError_t launch_grad_reduce(GradParts gp, const double *loss_part, int n_loss, double *loss, hipStream_t st) {
  int nb = 0;
  for (int l = 0; l < gp.n; ++l) {
    gp.part[l].block0 = nb;
    nb += (int)((gp.part[l].len + 255) / 256);
  }
  hipLaunchKernelGGL(grad_reduce_kernel, dim3(nb + 1), dim3(256), 0, st, gp, loss_part, n_loss, loss);
  return hipGetLastError();
}

// Adam with bias correction: c1 = 1 - beta1^t, c2 = 1 - beta2^t
__global__ void adam_kernel(long long n, float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                            float *__restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

hipError_t launch_adam(long long n, float *p, const float *g, float *m, float *v, float lr, float b1, float b2,
                       float eps, int t, hipStream_t st) {
  const float c1 = (float)(1.0 - pow((double)b1, t)), c2 = (float)(1.0 - pow((double)b2, t));
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, p, g, m, v, lr, b1, b2,
                     eps, c1, c2);
  return hipGetLastError();
}

// rows of a training batch: dst[r] = src[idx[r]] (row length len)
__global__ void gather_rows_kernel(int rows, int len, const int *__restrict__ idx, const float *__restrict__ src,
                                   float *__restrict__ dst) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)rows * len) return;
  const int r = (int)(i / len), c = (int)(i % len);
  dst[i] = src[(size_t)idx[r] * len + c];
}

hipError_t launch_gather_rows(int rows, int len, const int *idx, const float *src, float *dst, hipStream_t st) {
  const long long n = (long long)rows * len;
  hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, rows, len, idx, src,
                     dst);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Loop blocks <-> network rows.  A block is (channel c, coarse q, dR index iD);
// with list pointers null the blocks are all 2 x Nq x nD in compact order
// b = (c Nq + q) nD + iD.

__device__ inline void block_of(long long b, const int *ql, const int *cl, const int *dl, int Nq, int nD, int &q,
                                int &c, int &iD) {
  if (ql) {
    q = ql[b];
    c = cl[b];
    iD = dl[b];
  } else {
    iD = (int)(b % nD);
    q = (int)((b / nD) % Nq);
    c = (int)(b / ((long long)nD * Nq));
  }
}

// features: sin, cos of q and 2q, ln(Lambda) / 5, channel one-hot, dR one-hot
__global__ void sur_features_kernel(long long n, const int *__restrict__ ql, const int *__restrict__ cl,
                                    const int *__restrict__ dl, int Lq, int nD, double lam, float *__restrict__ X) {
  const long long b = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= n) return;
  int q, c, iD;
  block_of(b, ql, cl, dl, Lq * Lq, nD, q, c, iD);
  const int nin = 11 + nD;
  float *x = X + (size_t)b * nin;
  const double tx = 2.0 * M_PI * (double)(q / Lq) / Lq, ty = 2.0 * M_PI * (double)(q % Lq) / Lq;
  x[0] = (float)sin(tx);
  x[1] = (float)cos(tx);
  x[2] = (float)sin(ty);
  x[3] = (float)cos(ty);
  x[4] = (float)sin(2.0 * tx);
  x[5] = (float)cos(2.0 * tx);
  x[6] = (float)sin(2.0 * ty);
  x[7] = (float)cos(2.0 * ty);
  x[8] = (float)(log(lam) / 5.0);
  x[9] = c == 0 ? 1.f : 0.f;
  x[10] = c == 1 ? 1.f : 0.f;
  for (int j = 0; j < nD; ++j) x[11 + j] = j == iD ? 1.f : 0.f;
}

hipError_t launch_sur_features(long long n, const int *ql, const int *cl, const int *dl, int Lq, int nD, double lam,
                               float *X, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(sur_features_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, ql, cl, dl, Lq, nD,
                     lam, X);
  return hipGetLastError();
}

// targets: T[b][2 t + r] = s * Lc[c][q][iD][t] (r = real, imaginary), s = 1 / scale.
// Streaming (16 bytes read, 8 written per entry): four consecutive values per
// thread in passes over the grid (rows are whole multiples of four or, for one
// orbital, two: then VEC = 1), without lists one flat copy.  MAX: the largest
// |T| as well, kept per thread over the passes, one atomic per workgroup (one
// per wave of a separate pass over T took 38 ms for the 2.2e8 targets of the
// t2g 32 x 32 loops; this kernel with the maximum takes 0.61).  An aligned run
// of 64 values that are all NaN (an invalid block) makes the maximum NaN, a
// shorter one is passed over.
template <int VEC, bool MAX>
__global__ __launch_bounds__(256) void sur_targets_kernel(long long n, const int *__restrict__ ql,
                                                          const int *__restrict__ cl, const int *__restrict__ dl,
                                                          int Nq, int nD, int row, double s,
                                                          const double *__restrict__ Lc, float *__restrict__ T,
                                                          unsigned int *__restrict__ bits) {
  const long long nv = n * row / VEC, step = (long long)gridDim.x * 256;
  float big = 0.f;
  bool nan_run = false;
  // every lane of a wave makes the same passes (the votes below)
  for (long long w = (long long)blockIdx.x * 256 + (threadIdx.x & ~63); w < nv; w += step) {
    const long long i = w + (threadIdx.x & 63);
    float v[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) v[k] = 0.f;
    if (i < nv) {
      bool ok = true;
      const double *src = Lc + i * VEC;
      if (ql) {
        const long long b = i * VEC / row;
        const int j = (int)(i * VEC - b * row), q = ql[b], c = cl[b], iD = dl[b];
        ok = q >= 0 && q < Nq && c >= 0 && c <= 1 && iD >= 0 && iD < nD;
        src = Lc + ((((size_t)c * Nq + q) * nD + iD) * row + j);
      }
#pragma unroll
      for (int k = 0; k < VEC; ++k) v[k] = ok ? (float)(s * src[k]) : __int_as_float(0x7fc00000);  // invalid block: NaN
      if constexpr (VEC == 4)
        *(float4 *)(T + i * 4) = make_float4(v[0], v[1], v[2], v[3]);
      else
        T[i] = v[0];
    }
    if constexpr (MAX) {
      bool all = true;
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        all = all && v[k] != v[k];
        big = fmaxf(big, fabsf(v[k]));
      }
      const unsigned long long m = __ballot(all);
      if constexpr (VEC == 4) {
#pragma unroll
        for (int g = 0; g < 4; ++g) nan_run = nan_run || ((m >> (16 * g)) & 0xffffull) == 0xffffull;
      } else {
        nan_run = nan_run || m == ~0ull;
      }
    }
  }
  if constexpr (MAX) {
    __shared__ float red[4];
    for (int off = 32; off > 0; off >>= 1) big = fmaxf(big, __shfl_down(big, off));
    if (nan_run) big = __int_as_float(0x7fc00000);  // wave-uniform
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = big;
    __syncthreads();
    if (threadIdx.x == 0) {
      // as bit patterns, in which NaN is the largest
      unsigned int u = 0;
      for (int w = 0; w < 4; ++w) u = max(u, __float_as_uint(red[w]));
      atomicMax(bits, u);
    }
  }
}

// bits: if not null, a cleared word that receives the bit pattern of max |T|
hipError_t launch_sur_targets(long long n, const int *ql, const int *cl, const int *dl, int Nq, int nD, int no4,
                              double s, const double *Lc, float *T, unsigned int *bits, hipStream_t st) {
  const long long tot = n * 2 * no4;
  if (tot <= 0) return hipSuccess;
  // rows of 2 n_o^4 values; four at a time where rows and T allow 16-byte stores
  const bool vec = (2 * no4) % 4 == 0 && ((uintptr_t)T & 15) == 0;
  const long long nv = vec ? tot / 4 : tot;
  const dim3 grid((unsigned)std::min<long long>((nv + 255) / 256, 8192)), block(256);
#define TUFRG_TARGETS(V, M)                                                                                        \
  hipLaunchKernelGGL((sur_targets_kernel<V, M>), grid, block, 0, st, n, ql, cl, dl, Nq, nD, 2 * no4, s, Lc, T, bits)
  if (vec && bits)
    TUFRG_TARGETS(4, true);
  else if (vec)
    TUFRG_TARGETS(4, false);
  else if (bits)
    TUFRG_TARGETS(1, true);
  else
    TUFRG_TARGETS(1, false);
#undef TUFRG_TARGETS
  return hipGetLastError();
}

// compact loops from network rows of consecutive blocks b0 .. b0 + n - 1 (all-block order):
// Lc[b][t] = (Y[b][2t], Y[b][2t + 1]) * s, s = y_scale / Lambda^p
// Lc = s Y; a non-finite network output sets *bad (if given), so that the
// caller can fall back to the plain loops
__global__ void sur_scatter_kernel(long long n, int no4, double s, const float *__restrict__ Y,
                                   double *__restrict__ Lc, unsigned int *__restrict__ bad) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * 2 * no4) return;
  const float y = Y[i];
  if (bad && !isfinite(y)) atomicOr(bad, 1u);
  Lc[i] = s * (double)y;
}

hipError_t launch_sur_scatter(long long n, int no4, double s, const float *Y, double *Lc, unsigned int *bad,
                              hipStream_t st) {
  const long long tot = n * 2 * no4;
  if (tot <= 0) return hipSuccess;
  hipLaunchKernelGGL(sur_scatter_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, no4, s, Y, Lc,
                     bad);
  return hipGetLastError();
}

// max |a - b| and max |b| over n complex values (bit patterns of non-negative
// doubles order like the values)
__global__ void sur_compare_kernel(long long n, const double *__restrict__ a, const double *__restrict__ b,
                                   unsigned long long *__restrict__ bits) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  double d = 0.0, r = 0.0;
  if (i < n) {
    const double dr = a[2 * i] - b[2 * i], di = a[2 * i + 1] - b[2 * i + 1];
    d = sqrt(dr * dr + di * di);
    r = sqrt(b[2 * i] * b[2 * i] + b[2 * i + 1] * b[2 * i + 1]);
    // a NaN would vanish in the max below: count it as an infinite difference
    if (!(d <= 1.7976931348623157e308)) d = INFINITY;
    if (!(r <= 1.7976931348623157e308)) r = INFINITY;
  }
  // wave-level max, then one atomic per wave
  for (int off = 32; off > 0; off >>= 1) {
    d = fmax(d, __shfl_down(d, off));
    r = fmax(r, __shfl_down(r, off));
  }
  if ((threadIdx.x & 63) == 0) {
    atomicMax(&bits[0], (unsigned long long)__double_as_longlong(d));
    atomicMax(&bits[1], (unsigned long long)__double_as_longlong(r));
  }
}

hipError_t launch_sur_compare(long long n, const double *a, const double *b, unsigned long long *bits,
                              hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(sur_compare_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, a, b, bits);
  return hipGetLastError();
}

}  // namespace tufrg
