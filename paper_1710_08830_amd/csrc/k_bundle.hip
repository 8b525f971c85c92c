// Bundle products (hot path): per q,  out = f * V . L . V  (Sec. 3.1 matrix RGE:
// dP = VP Lpp VP with f = 1, dC = 2 VC Lph VC with f = 2), where L is expanded
// from its compact form L[(R1,a,b),(R2,c,d)] = Lc[dR(R1,R2)][(a,b,c,d)].
//
// Both precisions run on the matrix cores in their own arithmetic
// (v_mfma_f64_16x16x4_f64 and v_mfma_f32_16x16x4_f32: full FP64 and FP32
// products and sums), each complex product as four real ones.  On gfx950 the
// FP64 matrix rate equals the vector rate, but one instruction does 1024
// multiply-adds on two operand registers, where the vector form is held up by
// its LDS operand reads.
//
// Small bundles (two spin-orbitals, B <= 64): one workgroup per (channel, q), both channels in one
// launch; the vertex, the compact loop and the intermediate L.V in LDS.
// Large bundles: two batched complex products per q (tmp = L.V, out = f V.tmp),
// 96 x 96 tiles, four waves of 48 x 48 (3 x 3 matrix tiles, Re and Im), K steps
// of 12 (B is a multiple of 36 for six spin-orbitals: none is padded), the
// loop matrix expanded while its panel is staged, the next panels' loads in
// flight during the products; a wave whose 48 rows or columns lie outside does
// no products, so the padding is to 48 and not 96.  The tiles of one q run on
// one XCD and share its vertex in the L2.
#include "common.h"
#include "kernels.h"

namespace tufrg {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4b __attribute__((ext_vector_type(4)));
typedef float f32x2b __attribute__((ext_vector_type(2)));
__device__ f32x4b bundle_buffer_load_v4(i32x4 rsrc, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.raw.buffer.load.v4f32");
__device__ f32x2b bundle_buffer_load_v2(i32x4 rsrc, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.raw.buffer.load.v2f32");

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// 16 x 16 x 4 products: operands A(lane % 16, lane / 16) and B(lane / 16, lane %
// 16), accumulator element r at (row(lane, r), lane % 16)
template <typename T>
struct Mm;
template <>
struct Mm<double> {
  typedef f64x4 acc;
  __device__ static acc fma(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row(int lane, int r) { return 4 * r + (lane >> 4); }
};
template <>
struct Mm<float> {
  typedef f32x4 acc;
  __device__ static acc fma(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

template <typename T>
struct CAcc {
  typename Mm<T>::acc re, im;
  __device__ void clear() {
#pragma unroll
    for (int r = 0; r < 4; ++r) re[r] = im[r] = T(0);
  }
  // += a b of one K step of 4
  __device__ void mac(cx<T> a, cx<T> b) {
    re = Mm<T>::fma(a.re, b.re, re);
    im = Mm<T>::fma(a.re, b.im, im);
    re = Mm<T>::fma(-a.im, b.im, re);
    im = Mm<T>::fma(a.im, b.re, im);
  }
};

template <typename T>
struct alignas(2 * sizeof(T)) C2 {
  T re, im;
};

}  // namespace

// most differences of the form factors (4 NT of them at most) of a small bundle
constexpr int small_nD(int nt) { return nt == 1 ? 13 : nt == 2 ? 57 : 81; }

// waves of a small bundle's workgroup: one per tile up to eight, so that two
// waves of a SIMD hide each other's LDS reads
constexpr int small_waves(int nt) { return nt < 3 ? 4 : 8; }

struct BundleSmall {
  const void *V[2];
  const double *Lc[2];
  double *out[2];
  double f[2];
};

// NT: 16-wide tiles that cover B; out[ch][q] = f V L V, grid (q, channel).
// B / 4 K steps: B is a multiple of 4 (4 n_ff for two spin-orbitals).  Rows and
// columns past B hold whatever is in LDS: they reach only results past B.
template <typename T, int NT>
__global__ __launch_bounds__(64 * small_waves(NT)) void bundle_small_kernel(int n_ff, int B, int nD,
                                                                            const int *__restrict__ didx,
                                                                            BundleSmall p) {
  constexpr int LD = 16 * NT + 1, NW = small_waves(NT), NTHR = 64 * NW;
  constexpr int NTW = (NT * NT + NW - 1) / NW;  // LD: row stride (odd: banks spread); tiles per wave
  // FP64, NT = 4: 154 of the 160 KB
  __shared__ C2<T> sV[16 * NT * LD], sT[16 * NT * LD], sL[small_nD(NT) * 16];
  __shared__ int sD[16 * NT * NT];
  const int q = blockIdx.x, ch = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int BB = B * B;
  const C2<T> *Vq = (const C2<T> *)p.V[ch] + (size_t)q * BB;
  const double2 *Lq = (const double2 *)p.Lc[ch] + (size_t)q * nD * 16;
  for (int i = tid; i < BB; i += NTHR) sV[(i / B) * LD + i % B] = Vq[i];
  for (int i = tid; i < nD * 16; i += NTHR) {
    const double2 v = Lq[i];
    sL[i] = C2<T>{(T)v.x, (T)v.y};
  }
  for (int i = tid; i < n_ff * n_ff; i += NTHR) sD[i] = didx[i];
  __syncthreads();
  const int lr = lane & 15, lk = lane >> 4;
  CAcc<T> acc[NTW];
#pragma unroll
  for (int t = 0; t < NTW; ++t) acc[t].clear();
  // T = L V: wave w takes tiles w, w + NW, ... (row tile t / NT)
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    const int tile = wv + NW * t;
    if (tile >= NT * NT) break;
    const int i = min(16 * (tile / NT) + lr, B - 1), j = 16 * (tile % NT) + lr;
    const int *dr = sD + (i >> 2) * n_ff;
    // operands one step ahead of their products
    auto at = [&](int k) { return sL[dr[k >> 2] * 16 + (i & 3) * 4 + lk]; };
    auto bt = [&](int k) { return sV[(k + lk) * LD + j]; };
    C2<T> a = at(0), b = bt(0);
    for (int k = 0; k < B; k += 4) {
      const int kn = min(k + 4, B - 4);
      const C2<T> an = at(kn), bn = bt(kn);
      acc[t].mac(cmake(a.re, a.im), cmake(b.re, b.im));
      a = an;
      b = bn;
    }
  }
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    const int tile = wv + NW * t;
    if (tile >= NT * NT) break;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      sT[(16 * (tile / NT) + Mm<T>::row(lane, r)) * LD + 16 * (tile % NT) + lr] = C2<T>{acc[t].re[r], acc[t].im[r]};
    acc[t].clear();
  }
  __syncthreads();
  // out = f V T
  double2 *oq = (double2 *)p.out[ch] + (size_t)q * BB;
  const double f = p.f[ch];
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    const int tile = wv + NW * t;
    if (tile >= NT * NT) break;
    const int i = 16 * (tile / NT) + lr, j = 16 * (tile % NT) + lr;
    C2<T> a = sV[i * LD + lk], b = sT[lk * LD + j];
    for (int k = 0; k < B; k += 4) {
      const int kn = min(k + 4, B - 4);
      const C2<T> an = sV[i * LD + kn + lk], bn = sT[(kn + lk) * LD + j];
      acc[t].mac(cmake(a.re, a.im), cmake(b.re, b.im));
      a = an;
      b = bn;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * (tile / NT) + Mm<T>::row(lane, r);
      if (row < B && j < B) oq[row * B + j] = make_double2(f * (double)acc[t].re[r], f * (double)acc[t].im[r]);
    }
  }
}

namespace {
constexpr int TB = 96, TK = 12, TLD = TB + 1;  // tile, K step, LDS row stride
constexpr int TH = 6;                           // values of a panel per loading thread (192 of the 256)

// Raw buffer loads of 16 bytes at a per-lane byte offset; past the end of the
// array they return zero (the rows past B of a panel).
__device__ inline i32x4 bundle_rsrc(const void *p, unsigned nbytes) {
  const unsigned long long a = (unsigned long long)p;
  return i32x4{(int)(unsigned)a, (int)(unsigned)(a >> 32), (int)nbytes, 0x00020000};
}
// element of FP64 storage in the arithmetic type, and of storage in that type
template <typename T>
__device__ inline C2<T> ld_f64(i32x4 r, unsigned off) {
  const double2 v = __builtin_bit_cast(double2, bundle_buffer_load_v4(r, (int)off, 0, 0));
  return C2<T>{(T)v.x, (T)v.y};
}
__device__ inline C2<double> ld_t(i32x4 r, unsigned off, double) { return ld_f64<double>(r, off); }
__device__ inline C2<float> ld_t(i32x4 r, unsigned off, float) {
  const f32x2b v = bundle_buffer_load_v2(r, (int)off, 0, 0);
  return C2<float>{v[0], v[1]};
}
}  // namespace

// AL: tmp[q] = L[q] V[q], A = L expanded from its compact form (FP64), B = V
// and C in the arithmetic type; else out[q] = alpha V[q] tmp[q].
// Vector instructions beside the products cost nearly their full time on
// gfx950, so a loading thread takes six values in a row of memory (A: half a row
// of the panel) or sixteen apart (B) behind one offset, which one addition per
// step advances.  t2g 10 x 10, 13 form factors (B = 468, 100 q): 5.0-5.2 ms for
// the two products of both channels in FP64 against 10.2 on the vector units,
// where the rate of a large FP64 product here (70 TFLOP/s) allows 4.7; FP32, 11 x 11,
// 9 form factors: 3.2 -> 1.67 ms, with V in FP32 from the projections 1.54.
template <typename T, bool AL, int NO2>
__global__ __launch_bounds__(256, 2) void bundle_gemm_kernel(int B, int n_ff, int nD, int n_q,
                                                             const int *__restrict__ didx,
                                                             const void *__restrict__ Av,
                                                             const void *__restrict__ Bv, double alpha,
                                                             void *__restrict__ Cv) {
  __shared__ C2<T> sA[2][TK * TLD], sB[2][TK * TLD];
  __shared__ int sD[AL ? 625 : 1];
  const int nt = (B + TB - 1) / TB, ntile = nt * nt;
  // XCD x takes the q x, x + 8, ..., the tiles of a q next to each other
  const int slot = blockIdx.x >> 3, q = (blockIdx.x & 7) + 8 * (slot / ntile), tile = slot % ntile;
  if (q >= n_q) return;
  const int i0 = (tile / nt) * TB, j0 = (tile % nt) * TB;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const size_t BB = (size_t)B * B;
  constexpr int no4 = NO2 * NO2;
  constexpr unsigned SZ = (unsigned)sizeof(C2<T>), ASZ = AL ? 16 : SZ;  // bytes per element: L FP64, V and tmp in T
  const auto ra = AL ? bundle_rsrc((const double2 *)Av + (size_t)q * nD * no4, (unsigned)nD * no4 * 16u)
                     : bundle_rsrc((const C2<T> *)Av + (size_t)q * BB, (unsigned)BB * SZ);
  const auto rb = bundle_rsrc((const C2<T> *)Bv + (size_t)q * BB, (unsigned)BB * SZ);
  const int wi = (wv >> 1) * 48, wj = (wv & 1) * 48;
  const bool busy = i0 + wi < B && j0 + wj < B;
  // loading threads: A row i0 + tid / 2, K 6 (tid % 2) + n; B row tid / 16, columns j0 + tid % 16 + 16 n
  const bool loads = tid < 2 * TB;
  const int ai = tid >> 1, ak = TH * (tid & 1), bk = tid >> 4, bj = tid & 15;
  const int i = i0 + ai;
  if constexpr (AL) {
    for (int e = tid; e < n_ff * n_ff; e += 256) sD[e] = didx[e];
    __syncthreads();
  }
  unsigned ao = 0, bo = ((unsigned)bk * B + j0 + bj) * SZ;
  if (!AL) ao = ((unsigned)i * B + ak) * SZ;
  C2<T> fa[TH], fb[TH];
  auto fetch = [&](int k0) {
    if constexpr (AL && NO2 == 36) {
      // the 12 K of a step lie in one form-factor block; rows past B: past the end
      const int rk = k0 / 36;
      const unsigned d = i < B ? (unsigned)sD[(i / 36) * n_ff + rk] : 0u;
      ao = i < B ? (d * no4 + (unsigned)(i % 36) * 36u + (unsigned)(k0 - 36 * rk + ak)) * 16u : 0xfffff000u;
    }
#pragma unroll
    for (int n = 0; n < TH; ++n) {
      if constexpr (AL && NO2 != 36) {
        const int k = k0 + ak + n;
        const bool in = i < B && k < B;
        const unsigned d = in ? (unsigned)sD[(i / NO2) * n_ff + k / NO2] : 0u;
        fa[n] = ld_f64<T>(ra, in ? (d * no4 + (unsigned)(i % NO2) * NO2 + (unsigned)(k % NO2)) * 16u : 0xfffff000u);
      } else if constexpr (AL) {
        fa[n] = ld_f64<T>(ra, ao + 16u * n);
      } else {
        fa[n] = ld_t(ra, ao + ASZ * n, T(0));
      }
      fb[n] = ld_t(rb, bo + 16u * SZ * n, T(0));
    }
    // B not a multiple of 12 (two spin-orbitals): the row part past it is the next row's
    if constexpr (!AL && NO2 != 36) {
#pragma unroll
      for (int n = 0; n < TH; ++n)
        if (k0 + ak + n >= B) fa[n] = C2<T>{T(0), T(0)};
    }
    if (!AL) ao += SZ * TK;
    bo += (unsigned)TK * B * SZ;
  };
  CAcc<T> acc[3][3];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[r][c].clear();
  const int lr = lane & 15, lk = lane >> 4;
  if (loads) fetch(0);
  int bf = 0;
  for (int k0 = 0; k0 < B; k0 += TK, bf ^= 1) {
    if (loads) {
#pragma unroll
      for (int n = 0; n < TH; ++n) {
        sA[bf][(ak + n) * TLD + ai] = fa[n];
        sB[bf][bk * TLD + bj + 16 * n] = fb[n];
      }
    }
    __syncthreads();  // one per step: the other buffer is free since the last one
    if (loads && k0 + TK < B) fetch(k0 + TK);
    if (busy) {
#pragma unroll
      for (int k = 0; k < TK; k += 4) {
        C2<T> a[3], b[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          a[r] = sA[bf][(k + lk) * TLD + wi + 16 * r + lr];
          b[r] = sB[bf][(k + lk) * TLD + wj + 16 * r + lr];
        }
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int c = 0; c < 3; ++c) acc[r][c].mac(cmake(a[r].re, a[r].im), cmake(b[c].re, b[c].im));
      }
    }
  }
  if (!busy) return;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = i0 + wi + 16 * r + Mm<T>::row(lane, e), j = j0 + wj + 16 * c + lr;
        if (row < B && j < B) {
          const size_t o = (size_t)q * BB + (size_t)row * B + j;
          const T re = acc[r][c].re[e], im = acc[r][c].im[e];
          if constexpr (AL)
            ((C2<T> *)Cv)[o] = C2<T>{re, im};
          else
            ((double2 *)Cv)[o] = make_double2(alpha * (double)re, alpha * (double)im);
        }
      }
}

template <typename T>
static hipError_t launch_small(int n_ff, int B, int nD, int n_q, const int *didx, const BundleSmall &p, int n_ch,
                               hipStream_t st) {
  const dim3 grid(n_q, n_ch), block(64 * small_waves((B + 15) / 16));
  if (nD > small_nD((B + 15) / 16)) return hipErrorInvalidValue;
  switch ((B + 15) / 16) {
    case 1: hipLaunchKernelGGL((bundle_small_kernel<T, 1>), grid, block, 0, st, n_ff, B, nD, didx, p); break;
    case 2: hipLaunchKernelGGL((bundle_small_kernel<T, 2>), grid, block, 0, st, n_ff, B, nD, didx, p); break;
    case 3: hipLaunchKernelGGL((bundle_small_kernel<T, 3>), grid, block, 0, st, n_ff, B, nD, didx, p); break;
    case 4: hipLaunchKernelGGL((bundle_small_kernel<T, 4>), grid, block, 0, st, n_ff, B, nD, didx, p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T, int NO2>
static hipError_t launch_gemm(int n_ff, int B, int nD, int n_q, const int *didx, const void *V,
                              const double *Lc, double factor, double *out, double *tmp, hipStream_t st) {
  const int nt = (B + TB - 1) / TB;
  const long long nb = 8LL * nt * nt * ((n_q + 7) / 8);
  if (nb > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((bundle_gemm_kernel<T, true, NO2>), dim3((unsigned)nb), dim3(256), 0, st, B, n_ff, nD, n_q, didx,
                     Lc, V, 1.0, tmp);
  hipLaunchKernelGGL((bundle_gemm_kernel<T, false, NO2>), dim3((unsigned)nb), dim3(256), 0, st, B, n_ff, nD, n_q, didx,
                     V, tmp, factor, out);
  return hipGetLastError();
}

hipError_t launch_bundle(int prec, int n_o, int n_ff, int B, int nD, int n_q, const int *didx, const BundleArgs *a,
                         int n_ch, double *tmp, hipStream_t st) {
  if (n_ch < 1 || n_ch > 2 || n_q < 1) return hipErrorInvalidValue;
  const bool f64 = prec == 0;
  if (n_o == 2 && B <= 64) {
    BundleSmall p;
    for (int c = 0; c < n_ch; ++c) {
      p.V[c] = a[c].V;
      p.Lc[c] = a[c].Lc;
      p.out[c] = a[c].out;
      p.f[c] = a[c].f;
    }
    return f64 ? launch_small<double>(n_ff, B, nD, n_q, didx, p, n_ch, st)
               : launch_small<float>(n_ff, B, nD, n_q, didx, p, n_ch, st);
  }
  if (!tmp) return hipErrorInvalidValue;
  if (n_ff > 25 || (n_o != 2 && n_o != 6)) return hipErrorInvalidValue;
  for (int c = 0; c < n_ch; ++c) {
    const void *V = a[c].V;
    const double *Lc = a[c].Lc;
    double *out = a[c].out;
    const double f = a[c].f;
    const hipError_t e =
        n_o == 6 ? (f64 ? launch_gemm<double, 36>(n_ff, B, nD, n_q, didx, V, Lc, f, out, tmp, st)
                        : launch_gemm<float, 36>(n_ff, B, nD, n_q, didx, V, Lc, f, out, tmp, st))
                 : (f64 ? launch_gemm<double, 4>(n_ff, B, nD, n_q, didx, V, Lc, f, out, tmp, st)
                        : launch_gemm<float, 4>(n_ff, B, nD, n_q, didx, V, Lc, f, out, tmp, st));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace tufrg
