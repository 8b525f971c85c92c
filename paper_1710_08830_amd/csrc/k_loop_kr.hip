// Form-factor projected orbital loops for six spin-orbitals on the matrix cores
// (BF16 split products, FP32 accumulation) for models with time reversal times
// inversion: H(k) = T H(k)^* T^t at every k, T = i sigma_y in each orbital (found
// on the hopping table at creation).
//
// Then every band is doubly degenerate, the band sum groups into three pairs
// (see k_loop_rb.hip), and the summed projector of a pair commutes with the
// antiunitary T K, so it is a Hermitian 3 x 3 matrix of quaternions: 15 real
// coordinates instead of the 36 of a Hermitian 6 x 6 matrix,
//   d_i               (i = 0..2)   Pi_{2i,2i} = Pi_{2i+1,2i+1},  Pi_{2i,2i+1} = 0
//   u, v, w, x (i < j)             Pi_{2i,2j} = u + iv = conj Pi_{2i+1,2j+1},
//                                  Pi_{2i,2j+1} = w + ix = -conj Pi_{2i+1,2j}.
// The loop sum acts on the 15 x 15 real matrices sum_p pi_p^alpha w_p^beta with
// w_p = sum_n L_pn x_n instead of 36 x 36 ones, 5.3 times less matrix work:
//   Y[(phi, alpha)][(q, beta)] = sum_{ky, p} phi(ky) pi_p^alpha(ky) w_p^beta(ky; q),
// phi in {1, cos(theta dy), sin(theta dy)}, one 16-row tile per phi and one
// 16-column tile per q.
//
// loop_kr_kernel: one workgroup of eight waves per 16 items (coarse q of one
//   channel, two per wave) and block of kx rows, tiles of 32 ky (K = 3 steps of
//   32, one per pair p; lane group g = lane / 16 holds ky 8 g .. 8 g + 7).  The
//   column of a lane is its beta, so each wave forms the B fragments of its two
//   q in its own registers, from the pair sums x_n^beta(k') (one 8-byte load
//   per ky: the three sums add up to the unit matrix) and the nine loop kernels L_pn of each ky, which its 64 lanes
//   evaluate and share through LDS; nothing but the A operand (phases times pi,
//   split, precomputed once per context) is shared, staged in LDS two tiles
//   deep with one barrier per tile.  Two q per wave halve the LDS reads of A: at
//   one, they (54 KB per wave and tile at 128 bytes per clock) would take longer
//   than the products.  t2g 32 x 32 refined 16 x (512 x 512 points, 513 items a
//   channel): 3.4 ms a channel, where the 36-coordinate kernel takes 7.4 ms.  The
//   matrix cores are busy a third of that, the vector unit (loop kernels and
//   fragments) as long; the rest is latency: two waves a SIMD at 256 registers.
//   The energies of the next tile are loaded once those of this one are used, and
//   the LDS reads are ordered one step ahead (4.1 -> 3.4 ms).  Waves 4..7 half a tile
//   behind waves 0..3, so that one does products beside the other's loop kernels,
//   took 4.8 ms.
// loop_kr_rowsum_kernel: the kx sums with the kx phases in FP64 over the half
//   plane of difference vectors.
// loop_kr_finalize_kernel: back to the entries (a, b, c, d), completed by
//   symmetry (loop_sym.h), times 1/Nf.
#include "common.h"
#include "kernels.h"
#include "loop_sym.h"

namespace tufrg {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
// raw buffer loads: wave-uniform byte offset soffset, per-lane voffset
__device__ f32x4 kr_buffer_load_v4(i32x4 rsrc, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.raw.buffer.load.v4f32");
__device__ f32x2 kr_buffer_load_v2(i32x4 rsrc, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.raw.buffer.load.v2f32");

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int NO = 6, NA = 36, NP = 3;  // spin-orbitals, packed projector values, pairs
constexpr int NQ = 15;                  // real coordinates of a pair sum
constexpr int KT = 32;                  // ky per tile
constexpr int NW = 8, NTHR = 64 * NW;   // waves
constexpr int QPW = 2, NQG = QPW * NW;  // items per wave and per workgroup
constexpr int XS = 32;                  // floats per point of the pair sums x[kx][ky][beta][n], n = 0, 1
constexpr int XP = 8;                   // columns repeated at both ends of a row: eight k' in a row never wrap

template <int NDY>
struct KR {
  static constexpr int NPHI = 2 * NDY + 1;
  static constexpr int UNITS = NP * NPHI * 2;         // 1 KB units of A per tile: (p, phi, hi / lo)
  static constexpr int UPH = (UNITS + 2 * NW - 1) / (2 * NW);  // per wave and half
  static constexpr int NH = NDY == 4 ? 21 : 13;       // half-plane points
};

__device__ inline void split2(float a, float b, unsigned &hi, unsigned &lo) {
  hi = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, bf16x2));
  const float ra = a - __uint_as_float(hi << 16), rb = b - __uint_as_float(hi & 0xffff0000u);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){ra, rb}, bf16x2));
}

__device__ inline i32x4 kr_rsrc(const void *p, unsigned nbytes) {
  const unsigned long long a = (unsigned long long)p;
  return i32x4{(int)(unsigned)a, (int)(unsigned)(a >> 32), (int)nbytes, 0x00020000};
}

// packed index (diagonal, then Re and Im of (a, c), a < c row-major) of the
// value that is coordinate b
__device__ inline int kr_packed(int b) {
  if (b < 3) return 2 * b;
  const int ij = (b - 3) / 4, r = (b - 3) % 4;
  const int i = ij == 2 ? 1 : 0, j = ij == 0 ? 1 : 2;
  const int a = 2 * i, c = 2 * j + (r >> 1);
  const int p = a * (2 * NO - 1 - a) / 2 + c - a - 1;
  return NO + 2 * p + (r & 1);
}

// entry (a, c) in the coordinates: cr at coordinate r (real part), ci at m
// (imaginary part); cr = ci = 0 where the entry vanishes
__device__ inline void kr_coords(int a, int c, int &r, double &cr, int &m, double &ci) {
  const int i = a >> 1, j = c >> 1, s = a & 1, t = c & 1;
  r = m = 0;
  cr = ci = 0.0;
  if (i == j) {
    if (s == t) {
      r = i;
      cr = 1.0;
    }
    return;
  }
  const int lo = i < j ? i : j, hi = i < j ? j : i;
  const int sl = i < j ? s : t, sh = i < j ? t : s;  // spins at lo and hi
  const int b = 3 + 4 * (lo == 1 ? 2 : hi - 1);
  r = b + (sl == sh ? 0 : 2);
  m = r + 1;
  // (0,0) u + iv, (1,1) u - iv, (0,1) w + ix, (1,0) -w + ix; below the diagonal conjugated
  cr = (sl == 1 && sh == 0) ? -1.0 : 1.0;
  ci = (sl == 1 && sh == 1) ? -1.0 : 1.0;
  if (i > j) ci = -ci;
}

// half-plane points dx > 0 or (dx = 0, dy >= 0) of the diamond |dx| + |dy| <= 4 (NDY = 4) or the 5 x 5 box
template <int NDY>
__host__ __device__ constexpr int kr_dx(int h) {
  return NDY == 4 ? (h < 5 ? 0 : h < 12 ? 1 : h < 17 ? 2 : h < 20 ? 3 : 4) : (h < 3 ? 0 : h < 8 ? 1 : 2);
}
template <int NDY>
__host__ __device__ constexpr int kr_dy(int h) {
  return NDY == 4 ? (h < 5 ? h : h < 12 ? h - 8 : h < 17 ? h - 14 : h < 20 ? h - 18 : 0)
                  : (h < 3 ? h : h < 8 ? h - 5 : h - 10);
}

}  // namespace

size_t kr_x_floats(int Lf) { return (size_t)Lf * (Lf + 2 * XP) * XS; }

// x[kx][ky + XP][beta][n], n = 0, 1, -XP <= ky < Lf + XP (mod Lf): pair sums of
// the projectors in the 15 coordinates (beta = 15: 0), summed in FP64; the loop
// kernel takes the third as what they leave of the unit matrix (1 for beta < 3, else
// 0), off by an FP32 rounding of that.  The loops are as far from FP64 ones as the
// 36-coordinate kernel's (root mean squares 3.15e-7 to 8.0e-7 of the loops', the two
// within 2 % over t2g and random models, meshes of 60 to 160, three regulators); with
// the third sum loaded as well their errors are the same, and the kernel spills
// registers (t2g 32 x 32 loops: 8.7 -> 11.5 ms).
__global__ void kr_x_kernel(int Lf, const double *__restrict__ band, float *__restrict__ x) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)Lf * (Lf + 2 * XP) * XS) return;
  const int b = (int)(i % XS) >> 1, n = (int)(i & 1), Nf = Lf * Lf;
  const int kx = (int)(i / XS / (Lf + 2 * XP)), kyp = (int)(i / XS % (Lf + 2 * XP));
  const int k = kx * Lf + (kyp - XP + XP * Lf) % Lf;
  double v = 0.0;
  if (b < NQ) {
    const int p = kr_packed(b);
    v = band[(size_t)(NO + 2 * n * NA + p) * Nf + k] + band[(size_t)(NO + (2 * n + 1) * NA + p) * Nf + k];
  }
  x[i] = (float)v;
}

hipError_t launch_kr_x(int Lf, const double *band, float *x, hipStream_t st) {
  const long long n = (long long)kr_x_floats(Lf);
  hipLaunchKernelGGL(kr_x_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, Lf, band, x);
  return hipGetLastError();
}

// A operand, [kx][ky tile][p][phi][hi, lo][lane] of 8 BF16: lane l holds row
// alpha = l % 16 and ky = 32 tile + 8 (l / 16) + t, t = 0..7: phi(ky) pi_p^alpha(ky),
// split; zero past the coordinates and the mesh.  The pair sums in FP64 from the
// bands at k (bandk [Nf][6 + 216])
template <int NDY>
__global__ __launch_bounds__(256) void kr_apre_kernel(const double *__restrict__ bandk, const float *__restrict__ phy,
                                                      int Lf, u32x4 *__restrict__ apre) {
  using S = KR<NDY>;
  const int ntk = (Lf + KT - 1) / KT;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long long)Lf * ntk * NP * S::NPHI * 64) return;
  const int lane = (int)(gid % 64);
  long long r = gid / 64;
  const int ph = (int)(r % S::NPHI);
  r /= S::NPHI;
  const int p = (int)(r % NP);
  r /= NP;
  const int tk = (int)(r % ntk), kx = (int)(r / ntk);
  u32x4 h, l;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    float v[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int ky = tk * KT + 8 * (lane >> 4) + 2 * t + u;
      float f = 0.f, pv = 0.f;
      if (ky < Lf) {
        f = ph == 0     ? 1.f
            : ph <= NDY ? phy[((size_t)ky * NDY + ph - 1) * 2]
                        : -phy[((size_t)ky * NDY + ph - NDY - 1) * 2 + 1];
        if ((lane & 15) < NQ) {
          const double *b = bandk + (size_t)(kx * Lf + ky) * (NO + NO * NA) + NO + 2 * p * NA + kr_packed(lane & 15);
          pv = (float)(b[0] + b[NA]);
        }
      }
      v[u] = pv * f;
    }
    unsigned hh, ll;
    split2(v[0], v[1], hh, ll);
    h[t] = hh;
    l[t] = ll;
  }
  const size_t o = ((((size_t)kx * ntk + tk) * NP + p) * S::NPHI + ph) * 2 * 64 + lane;
  apre[o] = h;
  apre[o + 64] = l;
}

size_t kr_apre_bytes(int ndy, int Lf) {
  return (size_t)Lf * ((Lf + KT - 1) / KT) * NP * (2 * ndy + 1) * 2 * 64 * 16;
}

hipError_t launch_kr_apre(int ndy, const double *bandk, const float *phy, int Lf, void *apre, hipStream_t st) {
  if (!bandk || !phy || !apre || (ndy != 2 && ndy != 4)) return hipErrorInvalidValue;
  const long long n = (long long)Lf * ((Lf + KT - 1) / KT) * NP * (2 * ndy + 1) * 64;
  const dim3 grid((unsigned)((n + 255) / 256));
  if (ndy == 4)
    hipLaunchKernelGGL(kr_apre_kernel<4>, grid, dim3(256), 0, st, bandk, phy, Lf, (u32x4 *)apre);
  else
    hipLaunchKernelGGL(kr_apre_kernel<2>, grid, dim3(256), 0, st, bandk, phy, Lf, (u32x4 *)apre);
  return hipGetLastError();
}

// ek[k] = (e_0, e_1, e_2, K_0, K_1, K_2, 0, 0) of the pairs (first band of each;
// shell scheme: K the J of the temperature vlam) and, shell scheme, (a_0, a_1, a_2,
// b_0, b_1, b_2, 0, 0) of the shell factors at lam; evaluated in FP64.  In place of
// the tables of all six bands that the other kernels read: with both, three
// launches for one (t2g, one form factor, 2 x 2 points, with the split below: 44 ->
// 36 us an evaluation).
__global__ void kr_ek_kernel(int Nf, int shell, const double *__restrict__ band, double vlam, int vscheme, int vderiv,
                             double lam, int deriv, float *__restrict__ ek) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 3 * Nf) return;
  const int n = i / Nf, k = i - n * Nf;
  const double e = band[(size_t)(2 * n) * Nf + k];
  float *o = ek + (size_t)k * (shell ? 16 : 8);
  o[n] = (float)e;
  o[3 + n] = (float)cut_val(e, vlam, vscheme, vderiv);
  if (n < 2) o[6 + n] = 0.f;
  if (shell) {
    double a, b;
    shell_ab(e, lam, deriv, a, b);
    o[8 + n] = (float)a;
    o[11 + n] = (float)b;
    if (n < 2) o[14 + n] = 0.f;
  }
}

hipError_t launch_kr_ek(int Nf, int shell, const double *band, double vlam, int vscheme, int vderiv, double lam,
                        int deriv, float *ek, hipStream_t st) {
  hipLaunchKernelGGL(kr_ek_kernel, dim3((3 * Nf + 255) / 256), dim3(256), 0, st, Nf, shell, band, vlam, vscheme, vderiv,
                     lam, deriv, ek);
  return hipGetLastError();
}

template <int NDY, int SCHEME, int DERIV, int ch>
__global__ __launch_bounds__(NTHR, 1) void loop_kr_kernel(const float *__restrict__ x, const float *__restrict__ ek,
                                                          const u32x4 *__restrict__ apre, int Lq, int n_ref, int Lf,
                                                          const int *__restrict__ items, int n_q, int half,
                                                          float lam, int n_groups, int n_kxb, int kxr,
                                                          float *__restrict__ Y) {
  using S = KR<NDY>;
  constexpr int NPHI = S::NPHI, UNITS = S::UNITS, UPH = S::UPH;
  constexpr bool SHELL = SCHEME == CUT_SHELL;
  constexpr int EV = SHELL ? 4 : 2;        // 16-byte loads of ek per point
  constexpr unsigned EB = 16u * EV;        // bytes of ek per k
  __shared__ __align__(16) u32x4 sA[2][UNITS * 64];
  __shared__ __align__(16) float sL[NW][QPW][KT][12];  // L_pn at [4 p + n]

  // XCD x takes the kx blocks x, x + 8, ..., the item groups fastest: the
  // workgroups running at once on one XCD share the A operand of their kx rows
  const int b = blockIdx.x, xcd = b & 7, jb = b >> 3;
  const int g = jb % n_groups, kxb = xcd + 8 * (jb / n_groups);
  if (kxb >= n_kxb) return;
  const int kx0 = kxb * kxr, nrow = min(kxr, Lf - kx0);
  const int ntk = (Lf + KT - 1) / KT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (half) {
    // no item of the group sums a row of this block: nothing to do (uniform)
    int any = 0;
    for (int j = 0; j < NQG; ++j) {
      const int q = items[min(NQG * g + j, n_q - 1)] & LOOP_ITEM_Q;
      for (int r = 0; r < nrow; ++r) any |= loop_row_weight2(Lf, (q / Lq) * n_ref, kx0 + r);
    }
    if (!any) return;
  }
  int qfx[QPW], qfy[QPW];
#pragma unroll
  for (int j = 0; j < QPW; ++j) {
    // past the list: the last item again (not stored)
    const int q = items[min(NQG * g + QPW * wv + j, n_q - 1)] & LOOP_ITEM_Q;
    qfx[j] = __builtin_amdgcn_readfirstlane((q / Lq) * n_ref);
    qfy[j] = __builtin_amdgcn_readfirstlane((q % Lq) * n_ref);
  }
  constexpr float sg = ch == 0 ? 1.f : -1.f;
  const unsigned xrow = (unsigned)(Lf + 2 * XP) * (XS * 4u);  // bytes of a row of x
  const auto rx = kr_rsrc(x, (unsigned)Lf * xrow), re = kr_rsrc(ek, (unsigned)Lf * Lf * EB);
  const int beta = lane & 15, lg = lane >> 4;

  // k' row (wave-uniform) and column of a point
  auto kprime = [&](int qf, int k) __attribute__((always_inline)) {
    int v = ch == 0 ? qf - k : k - qf;
    return v + (v < 0 ? Lf : 0);
  };
  struct Pts {
    f32x2 x[QPW][8];       // x_0^beta, x_1^beta at k' of this lane's eight ky
    f32x4 e[1 + QPW][EV];  // ek at k and at k' of ky = lane % 32
  } pt;
  // no conditions here and in the loads of A (past the last tile: that tile
  // again): they cost registers
  auto fetch_e = [&](int t) __attribute__((always_inline)) {
    const int kx = kx0 + t / ntk, T = t - (t / ntk) * ntk;
    // opaque: the offsets are formed here and not kept in registers across tiles
    int kye = min(T * KT + (lane & 31), Lf - 1);
    asm volatile("" : "+v"(kye));
#pragma unroll
    for (int v = 0; v < EV; ++v)
      pt.e[0][v] = kr_buffer_load_v4(re, (int)(kye * EB + 16 * v), (int)((unsigned)kx * Lf * EB), 0);
#pragma unroll
    for (int j = 0; j < QPW; ++j) {
      const int kpx = kprime(qfx[j], kx), kpe = kprime(qfy[j], kye);
#pragma unroll
      for (int v = 0; v < EV; ++v)
        pt.e[1 + j][v] = kr_buffer_load_v4(re, (int)(kpe * EB + 16 * v), (int)((unsigned)kpx * Lf * EB), 0);
    }
  };
  auto fetch_x = [&](int t) __attribute__((always_inline)) {
    const int kx = kx0 + t / ntk, T = t - (t / ntk) * ntk;
    int kb = min(T * KT + 8 * lg, Lf - 1);
    asm volatile("" : "+v"(kb));
#pragma unroll
    for (int j = 0; j < QPW; ++j) {
      const int kpx = kprime(qfx[j], kx);
      // the k' of ky kb .. kb + 7 lie in a row of x, from its column of kb (ph) or
      // of kb + 7 (pp); those past the mesh meet zero rows of A
      const int xo = (kprime(qfy[j], kb) + (ch == 0 ? XP - 7 : XP)) * (XS * 4) + beta * 8;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        pt.x[j][u] = kr_buffer_load_v2(rx, xo + (ch == 0 ? 7 - u : u) * (XS * 4), (int)((unsigned)kpx * xrow), 0);
    }
  };
  // A operand of a tile: the wave's units into registers, then into LDS, in two
  // halves (waves past the units repeat the last one)
  u32x4 ar[UPH];
  auto load_a = [&](int t, int hf) __attribute__((always_inline)) {
    const u32x4 *src = apre + (size_t)(kx0 * ntk + t) * (UNITS * 64) + lane;
#pragma unroll
    for (int u = 0; u < UPH; ++u) {
      ar[u] = src[min(wv + NW * (u + UPH * hf), UNITS - 1) * 64];
    }
  };
  auto store_a = [&](int bf, int hf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < UPH; ++u) {
      sA[bf][min(wv + NW * (u + UPH * hf), UNITS - 1) * 64 + lane] = ar[u];
    }
  };
  // loop kernels of the wave's two q at ky = lane % 32: lanes 0..31 evaluate
  // (p, n) = (0,0) (0,1) (0,2) (1,0) (1,1), lanes 32..63 (1,2) (2,0) (2,1) (2,2)
  auto loop_kernels = [&](int t) __attribute__((always_inline)) {
    const bool hi = lane >= 32;
    const int kx = kx0 + t / ntk;
    auto ev = [&](int s, int i) { return pt.e[s][i >> 2][i & 3]; };  // i: 0..2 e, 3..5 K, 8..10 a, 11..13 b
#pragma unroll
    for (int j = 0; j < QPW; ++j) {
      const float sw = half ? sg * 0.5f * (float)loop_row_weight2(Lf, qfx[j], kx) : sg;
      float l[5];
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        const int p0 = i / 3, n0 = i % 3, p1 = i == 0 ? 1 : 2, n1 = i == 0 ? 2 : (i < 4 ? i - 1 : 2);
        const float em = hi ? ev(0, p1) : ev(0, p0), km = hi ? ev(0, 3 + p1) : ev(0, 3 + p0);
        const float en = hi ? ev(1 + j, n1) : ev(1 + j, n0), kn = hi ? ev(1 + j, 3 + n1) : ev(1 + j, 3 + n0);
        l[i] = sw * divided_difference(em, -sg * en, km, -sg * kn, lam, dd_scheme(SCHEME), DERIV);
        if constexpr (SHELL) {
          const float am = hi ? ev(0, 8 + p1) : ev(0, 8 + p0), bm = hi ? ev(0, 11 + p1) : ev(0, 11 + p0);
          const float an = hi ? ev(1 + j, 8 + n1) : ev(1 + j, 8 + n0), bn = hi ? ev(1 + j, 11 + n1) : ev(1 + j, 11 + n0);
          l[i] *= fmaf(am, bn, bm * an);
        }
      }
      float *d = sL[wv][j][lane & 31];
      if (hi) {
        d[6] = l[0];
        d[8] = l[1];
        d[9] = l[2];
        d[10] = l[3];
      } else {
        d[0] = l[0];
        d[1] = l[1];
        d[2] = l[2];
        d[4] = l[3];
        d[5] = l[4];
      }
    }
    // read by other lanes of this wave only
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  const int ntile = nrow * ntk;
  f32x4 acc[NPHI][QPW];
  // products of tile t: per pair p the B fragments of the two q, then the nine
  // (five) row tiles
  const float unit = beta < 3 ? 1.f : 0.f;
  auto products = [&](int bf, int t) __attribute__((always_inline)) {
    float x2[QPW][8];
#pragma unroll
    for (int j = 0; j < QPW; ++j)
#pragma unroll
      for (int u = 0; u < 8; ++u) x2[j][u] = unit - pt.x[j][u][0] - pt.x[j][u][1];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      bf16x8 bh[QPW], bl[QPW];
#pragma unroll
      for (int j = 0; j < QPW; ++j) {
        u32x4 h, l;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float w[2];
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            const f32x4 L = *(const f32x4 *)&sL[wv][j][8 * lg + 2 * u + v][4 * p];
            const f32x2 X = pt.x[j][2 * u + v];
            w[v] = fmaf(L[2], x2[j][2 * u + v], fmaf(L[1], X[1], L[0] * X[0]));
          }
          unsigned hh, ll;
          split2(w[0], w[1], hh, ll);
          h[u] = hh;
          l[u] = ll;
        }
        bh[j] = __builtin_bit_cast(bf16x8, h);
        bl[j] = __builtin_bit_cast(bf16x8, l);
        // the loop kernels of two ky before the sums of the two before
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        // keeps the live loop kernels and point data within the registers
        __builtin_amdgcn_sched_barrier(0);
      }
      // the point data are used up: those of the next tile arrive during the last products
      if (p == NP - 1) {
        fetch_x(min(t + 1, ntile - 1));
        __builtin_amdgcn_sched_barrier(0);
      }
      const u32x4 *A = &sA[bf][p * NPHI * 128 + lane];
      bf16x8 ah = __builtin_bit_cast(bf16x8, A[0]), al = __builtin_bit_cast(bf16x8, A[64]);
#pragma unroll
      for (int f = 0; f < NPHI; ++f) {
        bf16x8 nh = ah, nl = al;
        if (f + 1 < NPHI) {
          nh = __builtin_bit_cast(bf16x8, A[(f + 1) * 128]);
          nl = __builtin_bit_cast(bf16x8, A[(f + 1) * 128 + 64]);
        }
#pragma unroll
        for (int j = 0; j < QPW; ++j) acc[f][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[j], acc[f][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < QPW; ++j) acc[f][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[j], acc[f][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < QPW; ++j) acc[f][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[j], acc[f][j], 0, 0, 0);
        ah = nh;
        al = nl;
      }
      // the reads of a row tile before the products of the one before
      __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
      for (int f = 0; f < NPHI; ++f) {
        __builtin_amdgcn_sched_group_barrier(0x008, 3 * QPW, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (p == 0) {
        store_a(bf ^ 1, 0);
        load_a(min(t + 1, ntile - 1), 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    store_a(bf ^ 1, 1);
  };

  fetch_e(0);
  fetch_x(0);
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    load_a(0, hf);
    store_a(0, hf);
  }
  __syncthreads();
  int t = 0;
  for (int r = 0; r < nrow; ++r) {
#pragma unroll
    for (int f = 0; f < NPHI; ++f)
#pragma unroll
      for (int j = 0; j < QPW; ++j) acc[f][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int tk = 0; tk < ntk; ++tk, ++t) {
      // LDS holds A of tile t; the other buffer is free since the barrier and is
      // filled during the tile
      load_a(min(t + 1, ntile - 1), 0);
      loop_kernels(t);
      fetch_e(min(t + 1, ntile - 1));  // the energies are used up; these arrive during the products
      __builtin_amdgcn_sched_barrier(0);
      products(t & 1, t);
      __syncthreads();
    }
    // tiles in the order of the accumulators: [item][kx][phi][lane][4]
#pragma unroll
    for (int j = 0; j < QPW; ++j) {
      const int it = NQG * g + QPW * wv + j;
      if (it < n_q) {
        f32x4 *Yr = (f32x4 *)(Y + ((size_t)it * Lf + kx0 + r) * NPHI * 256) + lane;
#pragma unroll
        for (int f = 0; f < NPHI; ++f) Yr[f * 64] = acc[f][j];
      }
    }
  }
}

// lam[item][h][e]: kx sums of the half plane in FP64, e the element of an
// accumulator tile (alpha = 4 (e / 64) + e % 4, beta = (e / 4) % 16); four
// segments of the item's rows per workgroup, added in order
template <int NDY>
__global__ __launch_bounds__(256) void loop_kr_rowsum_kernel(const float *__restrict__ Y, const double *__restrict__ tw,
                                                             int Lq, int n_ref, int Lf, const int *__restrict__ items,
                                                             int half, int ch, double2 *__restrict__ lam) {
  constexpr int NPHI = KR<NDY>::NPHI, NH = KR<NDY>::NH;
  __shared__ double2 red[3][64];
  const int it = blockIdx.x, e = blockIdx.y * 64 + (threadIdx.x & 63), seg = threadIdx.x >> 6;
  int r0, nr, h0, h1;
  loop_rows(Lf, ((items[it] & LOOP_ITEM_Q) / Lq) * n_ref, half, r0, nr, h0, h1);
  const int per = (nr + 3) / 4, re = min(nr, (seg + 1) * per);
  double zr[NH], zi[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) zr[h] = zi[h] = 0.0;
  const float *Yi = Y + (size_t)it * Lf * NPHI * 256 + e;
  for (int r = seg * per; r < re; ++r) {
    const int kx = r0 + r >= Lf ? r0 + r - Lf : r0 + r;
    double v[NPHI], cx[NDY + 1], sx[NDY + 1];
#pragma unroll
    for (int f = 0; f < NPHI; ++f) v[f] = (double)Yi[((size_t)kx * NPHI + f) * 256];
    cx[0] = 1.0;
    sx[0] = 0.0;
#pragma unroll
    for (int dx = 1; dx <= NDY; ++dx) {
      const int jj = (int)(((long long)kx * dx) % Lf);
      cx[dx] = tw[2 * jj];
      sx[dx] = -tw[2 * jj + 1];
    }
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int dx = kr_dx<NDY>(h), dy = kr_dy<NDY>(h), ad = dy < 0 ? -dy : dy;
      const double A = v[ad];
      if (dy == 0) {
        zr[h] = fma(cx[dx], A, zr[h]);
        zi[h] = fma(-sx[dx], A, zi[h]);
      } else {
        const double Sg = dy > 0 ? v[NDY + ad] : -v[NDY + ad];
        zr[h] = fma(cx[dx], A, fma(-sx[dx], Sg, zr[h]));
        zi[h] = fma(-cx[dx], Sg, fma(-sx[dx], A, zi[h]));
      }
    }
  }
  // ph: the imaginary coordinates (v, x) of the transposed X change sign
  const int beta = (e >> 2) & 15;
  const double sgn = (ch == 1 && beta >= 3 && ((beta - 3) & 1)) ? -1.0 : 1.0;
  double2 *out = lam + (size_t)it * NH * 256 + e;
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    __syncthreads();
    if (seg) red[seg - 1][threadIdx.x & 63] = make_double2(zr[h], zi[h]);
    __syncthreads();
    if (!seg) {
      double a = zr[h], c = zi[h];
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        a += red[s][threadIdx.x].x;
        c += red[s][threadIdx.x].y;
      }
      out[h * 256] = make_double2(sgn * a, sgn * c);
    }
  }
}

// SPLIT workgroups per (item, dR): the 15 x 15 coordinates in LDS, then the 1296 entries
template <int NDY, int SPLIT>
__global__ __launch_bounds__(256) void loop_kr_finalize_kernel(LoopSym sy, int ch, int nD, int n_q_out,
                                                               const int *__restrict__ items,
                                                               const int2 *__restrict__ dst,
                                                               const int *__restrict__ hmap,
                                                               const int *__restrict__ dlist, double inv_nf,
                                                               const double2 *__restrict__ lam,
                                                               double2 *__restrict__ out) {
  constexpr int NH = KR<NDY>::NH, NO2 = NO * NO, NO3 = NO2 * NO, NO4 = NO2 * NO2;
  __shared__ double2 sl[256];
  const int it = blockIdx.x / nD, iD = blockIdx.x % nD;
  const int hm = hmap[iD];
  {
    // [alpha][beta]; the other half plane: lambda(-dR) = conj lambda(dR)
    const int e = threadIdx.x;
    const double2 v = lam[((size_t)it * NH + (hm & 0xffff)) * 256 + e];
    sl[(4 * (e >> 6) + (e & 3)) * 16 + ((e >> 2) & 15)] =
        make_double2(v.x * inv_nf, ((hm >> 16) ? -v.y : v.y) * inv_nf);
  }
  __syncthreads();
  const int q = items[it] & LOOP_ITEM_Q, dx = dlist[2 * iD], dy = dlist[2 * iD + 1];
  const int2 d = dst[it];
  auto entry = [&](int tau) {
    const int a = tau / NO3, bb = (tau / NO2) % NO, c = (tau / NO) % NO, dd = tau % NO;
    int r1, m1, r2, m2;
    double cr1, ci1, cr2, ci2;
    kr_coords(a, c, r1, cr1, m1, ci1);
    kr_coords(bb, dd, r2, cr2, m2, ci2);
    const double2 rr = sl[r1 * 16 + r2], rm = sl[r1 * 16 + m2], mr = sl[m1 * 16 + r2], mm = sl[m1 * 16 + m2];
    // (cr1 r + i ci1 m)(cr2 r + i ci2 m)
    const double A = cr1 * cr2, B = cr1 * ci2, C = ci1 * cr2, E = -ci1 * ci2;
    return make_double2(A * rr.x + E * mm.x - B * rm.y - C * mr.y, A * rr.y + E * mm.y + B * rm.x + C * mr.x);
  };
  for (int tau = threadIdx.x + (SPLIT > 1 ? 256 * blockIdx.y : 0); tau < NO4; tau += 256 * SPLIT) {
    double2 v = entry(tau);
    if ((sy.half >> ch) & 1) {
      double sgn;
      const double2 p = entry(loop_partner_tau(sy, NO, ch, tau, sgn));
      loop_add_partner(sy, q, dx, dy, sgn, p, v);
    }
    loop_store(sy, NO, ch, q, dx, dy, tau, v, d, 0, n_q_out, (size_t)nD * NO4, (size_t)iD * NO4, out);
  }
}

size_t kr_rowbuf_floats(int ndy, int Lf) { return (size_t)Lf * (2 * ndy + 1) * 256; }  // per item
size_t kr_lam_doubles(int ndy) { return 2 * 256 * (size_t)(ndy == 4 ? KR<4>::NH : KR<2>::NH); }

// the items of one channel into the row buffers Y and on to the compact loops
// of their slots at out
hipError_t launch_loop_kr(const LoopArgs &a, const float *x, const float *ek, const void *apre, float *Y,
                          hipStream_t st) {
  const int n_q = a.n_pp + a.n_ph, ch = a.n_pp ? 0 : 1, kxr = a.kxr;
  if (a.n_o != NO || !x || !ek || !apre || !Y || !a.items || n_q < 1 || (a.n_pp && a.n_ph) || kxr < 1 || kxr > 8)
    return hipErrorInvalidValue;
  const int n_groups = (n_q + NQG - 1) / NQG, n_kxb = (a.Lf + kxr - 1) / kxr;
  const long long nblk = 8LL * n_groups * ((n_kxb + 7) / 8);
  if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
  const int half = (a.half >> ch) & 1;
#define TUFRG_KR(D, S, R)                                                                                          \
  if (ch == 0)                                                                                                     \
    hipLaunchKernelGGL((loop_kr_kernel<D, S, R, 0>), dim3((unsigned)nblk), dim3(NTHR), 0, st, x, ek,               \
                       (const u32x4 *)apre, a.Lq, a.n_ref, a.Lf, a.items, n_q, half, (float)a.lam, n_groups, n_kxb, \
                       kxr, Y);                                                                                    \
  else                                                                                                             \
    hipLaunchKernelGGL((loop_kr_kernel<D, S, R, 1>), dim3((unsigned)nblk), dim3(NTHR), 0, st, x, ek,               \
                       (const u32x4 *)apre, a.Lq, a.n_ref, a.Lf, a.items, n_q, half, (float)a.lam, n_groups, n_kxb, \
                       kxr, Y)
#define TUFRG_KR_SCHEMES(D)                              \
  if (a.scheme == CUT_TEMPERATURE && a.deriv) {                           \
    TUFRG_KR(D, CUT_TEMPERATURE, 1);                                      \
  } else if (a.scheme == CUT_TEMPERATURE) {                               \
    TUFRG_KR(D, CUT_TEMPERATURE, 0);                                      \
  } else if (a.scheme == CUT_OMEGA && a.deriv) {                          \
    TUFRG_KR(D, CUT_OMEGA, 1);                                            \
  } else if (a.scheme == CUT_OMEGA) {                                     \
    TUFRG_KR(D, CUT_OMEGA, 0);                                            \
  } else if (a.scheme == CUT_SHELL && !a.deriv) { /* its kernels take J */ \
    TUFRG_KR(D, CUT_SHELL, 0);                                            \
  } else {                                                                \
    return hipErrorInvalidValue;                                          \
  }
  if (a.ndy == 4 && a.ndx == 5) {
    TUFRG_KR_SCHEMES(4)
  } else if (a.ndy == 2 && a.ndx == 3) {
    TUFRG_KR_SCHEMES(2)
  } else {
    return hipErrorInvalidValue;
  }
#undef TUFRG_KR_SCHEMES
#undef TUFRG_KR
  return hipGetLastError();
}

hipError_t launch_loop_kr_sums(const LoopArgs &a, const float *Y, double *lam, const int *hmap, const int *dlist, int nD,
                               double *out, hipStream_t st) {
  const int n_q = a.n_pp + a.n_ph, ch = a.n_pp ? 0 : 1;
  if (!Y || !lam || !hmap || !dlist || !out || !a.items || !a.dst || n_q < 1 || (a.n_pp && a.n_ph))
    return hipErrorInvalidValue;
  const double inv = 1.0 / ((double)a.Lf * a.Lf);
  const LoopSym sy{a.trs, a.half, a.Lq, (const double2 *)a.twq};
  const int half = (a.half >> ch) & 1;
  // few blocks: the entries of each over several workgroups, which then take the
  // time of one entry (one block: 6.0 -> 3.5 us); many fill the chip as they are
  const long long nb = (long long)n_q * nD;
  const dim3 gs(n_q, 4), block(256);
#define TUFRG_KR_SUMS(D, SPLIT)                                                                                      \
  hipLaunchKernelGGL(loop_kr_rowsum_kernel<D>, gs, block, 0, st, Y, a.tw, a.Lq, a.n_ref, a.Lf, a.items, half, ch,     \
                     (double2 *)lam);                                                                                \
  hipLaunchKernelGGL((loop_kr_finalize_kernel<D, SPLIT>), dim3((unsigned)nb, SPLIT), block, 0, st, sy, ch, nD,        \
                     a.n_q_out, a.items, a.dst, hmap, dlist, inv, (const double2 *)lam, (double2 *)out)
  if (a.ndy == 4 && nb < 256) {
    TUFRG_KR_SUMS(4, 6);
  } else if (a.ndy == 4) {
    TUFRG_KR_SUMS(4, 1);
  } else if (nb < 256) {
    TUFRG_KR_SUMS(2, 6);
  } else {
    TUFRG_KR_SUMS(2, 1);
  }
#undef TUFRG_KR_SUMS
  return hipGetLastError();
}

}  // namespace tufrg
