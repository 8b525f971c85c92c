// Bundle products on the matrix cores for the mixed-precision path (Sec. 3.1
// matrix RGE: dP = VP Lpp VP, dC = 2 VC Lph VC, in the orbital form of
// Sec. 4.2), per coarse q:  tmp = L V,  out = f V tmp.
//
// A complex product is four real ones (Re = Ar Br - Ai Bi, Im = Ar Bi + Ai Br)
// and every real operand is split into two BF16 numbers, x = hi + lo with
// hi = RNE(x) and lo = RNE(x - hi); a real product is hi*hi + hi*lo + lo*hi
// on v_mfma_f32_16x16x32_bf16 with FP32 accumulation (the lo*lo term, about
// 2^-18 of the product, is dropped).
//
// Operands live in "split planes": per q four BF16 planes (Re hi, Re lo, Im hi,
// Im lo).  V comes from the projections in planes of B x B (natural).  Both
// matrix-core fragments are eight consecutive K of a row or column: V as the left
// operand has them as they are, V as the right operand is transposed by the LDS
// reads (ds_read_b64_tr_b16: of four K rows of 16 columns, lane l gets column l).
// L is read from the planes of its nD distinct n_o^2 x n_o^2 blocks, a granule of
// four K never crossing a block (n_o^2 is a multiple of four); its 425 KB per q (13
// form factors, six orbitals) stay in L2.  tmp is in transposed planes of Bp x Bp,
// Bp = B rounded up to the 96-wide output tile: zero for K (its rows) past B; columns
// past B hold other values, and what follows from them is not stored.
//   bundle_split_compact_kernel: compact loop (FP64) -> planes of its blocks
//   bundle_mfma_kernel<0>:       tmp = L V  -> transposed planes of tmp
//   bundle_mfma_kernel<1>:       out = f V tmp -> FP64
// t2g 16 x 16, 13 form factors (B = 468), both channels: 3.2 ms, the products 1.46
// and 1.60 ms (0.93 and 0.85 PFLOP/s of BF16, padding counted; a large library
// product reaches 1.09 on this card): the matrix cores are busy half of the time
// at the 1.9 GHz that the load leaves, the rest is LDS traffic and its waits.
// With V split in a pass of its own, both natural and transposed, and L expanded to
// planes of Bp x Bp it was 5.2 ms, 2.0 ms of it in those passes.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace tufrg {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4m __attribute__((ext_vector_type(4)));
typedef float f32x2m __attribute__((ext_vector_type(2)));
// raw buffer loads: per-lane voffset, wave-uniform soffset; past the end zero
__device__ f32x4m bmx_buffer_load_v4(i32x4 rsrc, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.raw.buffer.load.v4f32");
__device__ f32x2m bmx_buffer_load_v2(i32x4 rsrc, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.raw.buffer.load.v2f32");

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int BT = 96;   // output tile (complex rows x columns) of a workgroup
constexpr int KB = 32;   // K per step
constexpr int FFMAX = 25;

// two floats to packed BF16 pairs (round to nearest even): hi and the BF16 of the remainders
__device__ inline void bsplit2(float a, float b, unsigned &hi, unsigned &lo) {
  hi = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, bf16x2));
  const float ra = a - __uint_as_float(hi << 16), rb = b - __uint_as_float(hi & 0xffff0000u);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){ra, rb}, bf16x2));
}

__device__ inline i32x4 bmx_rsrc(const void *p, unsigned nbytes) {
  const unsigned long long a = (unsigned long long)p;
  return i32x4{(int)(unsigned)a, (int)(unsigned)(a >> 32), (int)nbytes, 0x00020000};
}

__device__ inline bf16x8 negate(bf16x8 v) {
  u32x4 u = __builtin_bit_cast(u32x4, v);
  u ^= 0x80008000u;
  return __builtin_bit_cast(bf16x8, u);
}

}  // namespace

static size_t bundle_split_pad(int B) { return (size_t)((B + BT - 1) / BT) * BT; }

// compact loop Lc [n_q][n] complex FP64, n = nD n_o^4 -> planes Ls [n_q][4][n]
__global__ __launch_bounds__(256) void bundle_split_compact_kernel(int n, const double *__restrict__ Lc,
                                                                   unsigned short *__restrict__ Ls) {
  const int i = 4 * (blockIdx.x * blockDim.x + threadIdx.x), q = blockIdx.y;
  if (i >= n) return;  // n is a multiple of four
  const double2 *v = (const double2 *)Lc + (size_t)q * n + i;
  unsigned w[4][2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const double2 a = v[2 * u], b = v[2 * u + 1];
    bsplit2((float)a.x, (float)b.x, w[0][u], w[1][u]);
    bsplit2((float)a.y, (float)b.y, w[2][u], w[3][u]);
  }
  unsigned short *o = Ls + 4 * (size_t)q * n + i;
#pragma unroll
  for (int p = 0; p < 4; ++p) *(u32x2 *)(o + (size_t)p * n) = (u32x2){w[p][0], w[p][1]};
}

// One q and one 96 x 96 output tile of
//   OUT 0: tmp = L V, L in block planes [n_q][4][nD no2^2], V in planes [n_q][4][B][B],
//          into transposed planes T [n_q][4][Bp][Bp]
//   OUT 1: f V tmp into Cd [n_q][B][B] complex FP64
// Four waves in 2 x 2, each a 48 x 48 block of 3 x 3 matrix tiles with Re and Im
// accumulators.
template <int OUT>
__global__ __launch_bounds__(256, 2) void bundle_mfma_kernel(int B, int Bp, int n_q, int tiles, int no2, int n_ff,
                                                             int nD, const int *__restrict__ didx,
                                                             const unsigned short *__restrict__ L,
                                                             const unsigned short *__restrict__ V, double f,
                                                             unsigned short *__restrict__ T,
                                                             double *__restrict__ Cd) {
  // work item: the blocks of one XCD (b % 8) take consecutive items, so the
  // tiles of one q run together on one L2
  const int b = blockIdx.x, per = gridDim.x >> 3;
  const int w = (b & 7) * per + (b >> 3);
  const int tq = tiles * tiles;
  const int q = w / tq;
  if (q >= n_q) return;
  const int t = w - q * tq, i0 = (t / tiles) * BT, j0 = (t - (t / tiles) * tiles) * BT;
  const int BB = B * B, no4 = no2 * no2, nL = nD * no4;
  const size_t P = (size_t)Bp * Bp;
  const i32x4 rV = bmx_rsrc(V + 4 * (size_t)q * BB, 8u * BB);
  const i32x4 rX = OUT == 0 ? bmx_rsrc(L + 4 * (size_t)q * nL, 8u * nL) : bmx_rsrc(T + 4 * (size_t)q * P, 8u * (unsigned)P);

  // sA and, as columns of K, sB (OUT 1): [plane][row][32 K], granules of 8 K at
  // (granule ^ row / 4 % 4): 16 rows of a fragment read and 4 whole rows of a store
  // each cover the banks once.  sB as rows of K (OUT 0): [plane][K][96 columns], 16
  // columns next to each other swapped for odd K / 8, so that the two K / 8 of a
  // half wave fall on different banks.
  __shared__ __align__(16) unsigned short sA[4 * BT * KB];
  __shared__ __align__(16) unsigned short sB[4 * BT * KB];
  __shared__ int sD[OUT == 0 ? FFMAX * FFMAX : 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, wr = wv >> 1, wc = wv & 1;
  const int fr = lane & 15;

  // Staging, per panel 4 planes x 96 rows x 32 K in granules of 8 K (V as rows of K:
  // of 8 columns), six per thread: three of each of the planes pp, pp + 2; L in
  // granules of 4 K, twelve per thread.  The loads of a step differ from the first
  // by a uniform offset; K past B are set to zero, rows past B hold other values
  // and are not stored.
  f32x4m ga[6], gb[6];
  const int pp = tid >> 7, h = tid & 127;
  int va[3], vb[3], da[3], db[3];  // byte offsets of the loads (L: block row), element offsets in LDS
  int vl[3];                       // L: row in its block
  const int kg = OUT == 0 ? 4 * (tid & 7) : 8 * (tid & 3);  // K of the thread's granules of A
  int kb = 0, kc = 0;                                       // L: block of this K and column in it
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    if constexpr (OUT == 0) {
      const int r = 32 * v + (tid >> 3), i = min(i0 + r, B - 1), rb = i / no2;
      va[v] = rb * n_ff;
      da[v] = r * KB + (((kg >> 3) ^ ((r >> 2) & 3)) * 8) + (kg & 4);
      vl[v] = (i - rb * no2) * no2;
      const int g = h + 128 * v, k = g / 12, c = 8 * (g % 12);
      vb[v] = 2 * (pp * BB + k * B + j0 + c);
      db[v] = (pp * KB + k) * BT + (c ^ (16 * ((k >> 3) & 1)));
    } else {
      const int r = 32 * v + (h >> 2);
      va[v] = 2 * (pp * BB + min(i0 + r, B - 1) * B + kg);
      vb[v] = 2 * (pp * (int)P + (j0 + r) * Bp + kg);
      da[v] = db[v] = (pp * BT + r) * KB + ((kg >> 3) ^ ((r >> 2) & 3)) * 8;
    }
  }
  if constexpr (OUT == 0) {
    for (int i = tid; i < n_ff * n_ff; i += 256) sD[i] = didx[i] * no4;
    kb = kg / no2;
    kc = kg - kb * no2;
    __syncthreads();
  }
  auto load = [&](int k0) __attribute__((always_inline)) {
    if constexpr (OUT == 0) {
      const int cb = min(kb, n_ff - 1);
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        const int o = 2 * (sD[va[v] + cb] + vl[v] + kc);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const f32x2m x = bmx_buffer_load_v2(rX, o, 2 * p * nL, 0);
          const int i = 3 * p + v;
          ga[i >> 1][2 * (i & 1)] = x[0];
          ga[i >> 1][2 * (i & 1) + 1] = x[1];
        }
      }
      kc += KB;
      if (kc >= no2) kc -= no2, ++kb;  // no2 >= 32
    } else {
#pragma unroll
      for (int u = 0; u < 6; ++u) ga[u] = bmx_buffer_load_v4(rV, va[u >> 1], 2 * k0 + 4 * (u & 1) * BB, 0);
    }
    const int sb = OUT == 0 ? 2 * k0 * B : 2 * k0, pb = 4 * (OUT == 0 ? BB : (int)P);
#pragma unroll
    for (int u = 0; u < 6; ++u) gb[u] = bmx_buffer_load_v4(OUT == 0 ? rV : rX, vb[u >> 1], sb + (u & 1) * pb, 0);
  };
  auto store = [&](int k0) __attribute__((always_inline)) {
    if (k0 + KB > B) {
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        if constexpr (OUT == 0) {
          if (k0 + kg >= B) ga[u] = (f32x4m){0.f, 0.f, 0.f, 0.f};
          if (k0 + (h + 128 * (u >> 1)) / 12 >= B) gb[u] = (f32x4m){0.f, 0.f, 0.f, 0.f};
        } else {
          if (k0 + kg >= B) ga[u][0] = ga[u][1] = 0.f;
          if (k0 + kg + 4 >= B) ga[u][2] = ga[u][3] = 0.f;  // B is a multiple of four
        }
      }
    }
    if constexpr (OUT == 0) {
#pragma unroll
      for (int i = 0; i < 12; ++i)
        *(f32x2m *)&sA[(i / 3) * BT * KB + da[i % 3]] = (f32x2m){ga[i >> 1][2 * (i & 1)], ga[i >> 1][2 * (i & 1) + 1]};
    } else {
#pragma unroll
      for (int u = 0; u < 6; ++u) *(f32x4m *)&sA[2 * (u & 1) * BT * KB + da[u >> 1]] = ga[u];
    }
#pragma unroll
    for (int u = 0; u < 6; ++u) *(f32x4m *)&sB[2 * (u & 1) * BT * KB + db[u >> 1]] = gb[u];
  };
  // eight K of a row of A, of a column of the right operand
  const int fo = fr * KB + ((lane >> 4) ^ ((fr >> 2) & 3)) * 8;
  const int ko = (8 * (lane >> 4) + (fr >> 2)) * BT, odd = (lane >> 4) & 1;
  auto left = [&](int p, int m) __attribute__((always_inline)) {
    return *(const bf16x8 *)&sA[(p * BT + wr * 48 + 16 * m) * KB + fo];
  };
  auto right = [&](int p, int n) __attribute__((always_inline)) {
    if constexpr (OUT == 0) {
      const int o = p * KB * BT + ko + 16 * ((wc * 3 + n) ^ odd) + 4 * (lane & 3);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)&sB[o]);
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)&sB[o + 4 * BT]);
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      return *(const bf16x8 *)&sB[(p * BT + wc * 48 + 16 * n) * KB + fo];
    }
  };

  f32x4 accR[3][3], accI[3][3];
#pragma unroll
  for (int m = 0; m < 3; ++m)
#pragma unroll
    for (int n = 0; n < 3; ++n) accR[m][n] = accI[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};

  load(0);
  const int K = (B + KB - 1) / KB * KB;
  for (int k0 = 0; k0 < K; k0 += KB) {
    __syncthreads();  // the previous step's fragments are read
    store(k0);
    __syncthreads();
    if (k0 + KB < K) load(k0 + KB);  // in flight during the products
    bf16x8 a[3][4], bn[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) bn[p] = right(p, 0);
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
      for (int p = 0; p < 4; ++p) a[m][p] = left(p, m);
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      bf16x8 bv[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) bv[p] = bn[p];
      if (n < 2) {
#pragma unroll
        for (int p = 0; p < 4; ++p) bn[p] = right(p, n + 1);
      }
      const bf16x8 nih = negate(bv[2]), nil = negate(bv[3]);
      // Re += Ar Br - Ai Bi, Im += Ar Bi + Ai Br; six other accumulators between two
      // products into one
      auto step = [&](int pa, bf16x8 br, int qa, bf16x8 bi) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          accR[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m][pa], br, accR[m][n], 0, 0, 0);
          accI[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m][qa], bi, accI[m][n], 0, 0, 0);
        }
      };
      step(0, bv[0], 0, bv[2]);
      step(0, bv[1], 0, bv[3]);
      step(1, bv[0], 1, bv[2]);
      step(2, nih, 2, bv[0]);
      step(2, nil, 2, bv[1]);
      step(3, nih, 3, bv[0]);
    }
  }

  // lane holds rows 4 (lane / 16) + r, column lane % 16 of each matrix tile
#pragma unroll
  for (int m = 0; m < 3; ++m)
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      const int ib = i0 + wr * 48 + 16 * m + 4 * (lane >> 4), j = j0 + wc * 48 + 16 * n + fr;
      if constexpr (OUT == 0) {
        // transposed planes: row j, the four rows ib.. as four consecutive BF16
        unsigned rh[2], rl[2], ih[2], il[2];
        bsplit2(accR[m][n][0], accR[m][n][1], rh[0], rl[0]);
        bsplit2(accR[m][n][2], accR[m][n][3], rh[1], rl[1]);
        bsplit2(accI[m][n][0], accI[m][n][1], ih[0], il[0]);
        bsplit2(accI[m][n][2], accI[m][n][3], ih[1], il[1]);
        if (ib >= B) rh[0] = rh[1] = rl[0] = rl[1] = ih[0] = ih[1] = il[0] = il[1] = 0;  // B is a multiple of four
        unsigned short *o = T + 4 * (size_t)q * P + (size_t)j * Bp + ib;
        *(u32x2 *)(o) = (u32x2){rh[0], rh[1]};
        *(u32x2 *)(o + P) = (u32x2){rl[0], rl[1]};
        *(u32x2 *)(o + 2 * P) = (u32x2){ih[0], ih[1]};
        *(u32x2 *)(o + 3 * P) = (u32x2){il[0], il[1]};
      } else {
        if (j < B) {
          double2 *o = (double2 *)Cd + (size_t)q * BB;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = ib + r;
            if (i < B) o[(size_t)i * B + j] = make_double2(f * (double)accR[m][n][r], f * (double)accI[m][n][r]);
          }
        }
      }
    }
}

size_t bundle_split_bytes_per_q(int n_o, int B, int nD) {
  const size_t Bp = bundle_split_pad(B);
  return 4 * (Bp * Bp + (size_t)nD * n_o * n_o * n_o * n_o) * sizeof(unsigned short);  // tmp transposed, L blocks
}

// out = f V L V for n_q coarse q, V in planes [n_q][4][B][B], in chunks that fit
// the workspace ws (ws_bytes >= bundle_split_bytes_per_q)
hipError_t launch_bundle_bf16x3(int n_o, int n_ff, int B, int nD, int n_q, const int *didx, const void *V,
                                const double *Lc, double factor, double *out, void *ws, size_t ws_bytes,
                                hipStream_t st) {
  const int Bp = (int)bundle_split_pad(B);
  const size_t per_q = bundle_split_bytes_per_q(n_o, B, nD);
  if (!ws || ws_bytes < per_q || B % 4 || n_o != 6 || n_ff > FFMAX) return hipErrorInvalidValue;
  const int chunk = (int)std::min<size_t>({(size_t)n_q, ws_bytes / per_q, (size_t)65535});
  const int no2 = n_o * n_o, nL = nD * no2 * no2;
  unsigned short *T = (unsigned short *)ws, *L = T + (size_t)chunk * 4 * Bp * Bp;
  const int tiles = Bp / BT;
  for (int q0 = 0; q0 < n_q; q0 += chunk) {
    const int nq = std::min(chunk, n_q - q0);
    const unsigned short *Vq = (const unsigned short *)V + 4 * (size_t)q0 * B * B;
    hipLaunchKernelGGL(bundle_split_compact_kernel, dim3((nL / 4 + 255) / 256, nq), dim3(256), 0, st, nL,
                       Lc + 2 * (size_t)q0 * nL, L);
    const long long items = (long long)nq * tiles * tiles;
    const unsigned nblk = (unsigned)(((items + 7) / 8) * 8);
    hipLaunchKernelGGL(bundle_mfma_kernel<0>, dim3(nblk), dim3(256), 0, st, B, Bp, nq, tiles, no2, n_ff, nD, didx, L,
                       Vq, 1.0, T, (double *)nullptr);
    hipLaunchKernelGGL(bundle_mfma_kernel<1>, dim3(nblk), dim3(256), 0, st, B, Bp, nq, tiles, no2, n_ff, nD, didx, L,
                       Vq, factor, T, out + 2 * (size_t)q0 * B * B);
  }
  return hipGetLastError();
}

}  // namespace tufrg
