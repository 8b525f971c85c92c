// Form-factor projected orbital loops (hot path).
//
// Loop matrices in the orbital basis (the paper's Sec. 3.1 loop matrices with
// the orbital-basis loop of Sec. 4.2, written as a direct k-sum on the refined
// mesh), in the bundle layout of the library:
//
//   Lpp(s)[(R1,a,b),(R2,c,d)] = 1/Nf sum_k e^{-ik.(R1-R2)}
//        sum_mn Pi_m(k)_ac Pi_n(s-k)_bd L-(e_m(k), e_n(s-k))
//   Lph(u)[(R1,a,b),(R2,c,d)] = 1/Nf sum_k e^{-ik.(R1-R2)}
//        sum_mn Pi_m(k)_ac Pi_n(k-u)_db L+(e_m(k), e_n(k-u))
//
// Both depend on R1, R2 only through dR = R1 - R2, so the kernel produces the
// compact loop  Lc(q)[dR][tau],  tau = (a, b, c, d) flattened.
//
// Two spin-orbitals (this kernel):
// * Completeness, Pi_1 = 1 - Pi_0, gives with X_n the projector at k' (its
//   transpose for ph) and alpha_m = L_m0 - L_m1:
//     W_m = sum_n L_mn X_n = alpha_m X_0 + L_m1 1,  M = sum_m Pi_m (x) W_m
//         = Pi_0 (x) (W_0 - W_1) + 1 (x) W_1,
//   so only e_0, e_1, K_0, K_1 and the four reals of Pi_0 are read per point,
//   as two 4-vectors (k-major arrays ekv and pi4).
// * M[(c,d,a,b)] = conj(M[(a,b,c,d)]): only 10 entries are distinct (4 real).
//   With the phase p = c + i s the accumulation of p M and p conj(M) needs only
//   A = sum c M and B = sum s M; the pair is rebuilt at the end as
//   A + iB and (A.re + B.im) + i (B.re - A.im).
// * The phase is separable, e^{-ik.dR} = e^{-i kx dx} e^{-i ky dy}: every lane
//   owns one ky and walks kx, so the kx phases are wave-uniform; accumulators
//   cover dx >= 0 only (dx < 0 follows from hermiticity,
//   Lc[dR][(ab,cd)] = conj(Lc[-dR][(cd,ab)])).  At the end of a kx chunk the
//   lanes' values are transposed through LDS and contracted with e^{-i ky dy}.
// Partial sums per (ky block, kx chunk) go to HBM; a finalising kernel adds
// them in a fixed order (deterministic, no atomics).
//
// Half of the sum follows from the other (every model; all loop kernels, see
// loop_sym.h):
// * pp: k and q - k carry the same two points with the orbital pairs
//   exchanged, Lc(q)[dR][abcd] = H[abcd] + e^{-iq.dR} conj(H[dcba]) with H
//   the sum over the kx rows of one of each pair (kx, qx - kx): rows from qx/2
//   to qx/2 + Lf/2, a row that is its own partner with weight 1/2;
// * ph: Lc(-q)[dR][abcd] = e^{iq.dR} Lc(q)[dR][dcba]: one of q, -q is summed.
// With time reversal, Pi(-k) = T Pi(k)^* T^t and e(-k) = e(k) (checked on the
// hopping table at creation; T real, one entry +-1 per row), both hold in both
// channels: Lc(-q)[abcd] = tttt conj(Lc(q)[a'b'c'd']) (a' the partner of a),
// and the ph rows (kx, qx - kx) pair up with d'c'b'a' in place of dcba.  The
// loop kernels are bound by vector issue, so the time follows the points:
// half of them for every model, a quarter with time reversal.
#include <vector>

#include "common.h"
#include "kernels.h"
#include "loop_sym.h"

namespace tufrg {

namespace {

// distinct entries: 4 real (tau = 0, 5, 10, 15) and 6 complex representatives
// (tau = 1, 11, 2, 7, 3, 6) with partners (4, 14, 8, 13, 12, 9); see TAU_VALUE
constexpr int NREAL = 4, NCPLX = 6;

}  // namespace

// four consecutive values at index i of a k-major array of 4-vectors
template <typename T>
struct V4 {
  T x, y, z, w;
};
// Raw buffer loads: a descriptor of an array of nbytes bytes (base address,
// no stride, the gfx9-family data-format bits in the last word), a wave-uniform
// byte offset and a per-lane 32-bit byte offset.
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
__device__ f32x4v raw_buffer_load_v4f32(i32x4 rsrc, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.raw.buffer.load.v4f32");
template <typename T>
__device__ inline i32x4 make_rsrc(const T *p, unsigned nbytes) {
  const unsigned long long a = (unsigned long long)p;
  return i32x4{(int)(unsigned)a, (int)(unsigned)(a >> 32), (int)nbytes, 0x00020000};
}
// four floats at byte offset soff (wave-uniform) + voff (per lane)
__device__ inline V4<float> ld4_buf(i32x4 r, unsigned voff, unsigned soff) {
  const f32x4v v = raw_buffer_load_v4f32(r, (int)voff, (int)soff, 0);
  return {v[0], v[1], v[2], v[3]};
}
// four doubles: two 16-byte loads
__device__ inline V4<double> ld4d_buf(i32x4 r, unsigned voff, unsigned soff) {
  const double2 a = __builtin_bit_cast(double2, raw_buffer_load_v4f32(r, (int)voff, (int)soff, 0));
  const double2 b = __builtin_bit_cast(double2, raw_buffer_load_v4f32(r, (int)voff + 16, (int)soff, 0));
  return {a.x, a.y, b.x, b.y};
}

// Loop body of one channel (CH = 0: pp, k' = q - k; CH = 1: ph, k' = k - q).
// ekv[k] = (e_0, e_1, K(e_0), K(e_1)), pi4[k] = (Pi_0[00], Pi_0[11], Re Pi_0[01], Im Pi_0[01]);
// shell scheme: K is the fixed-temperature J and cv[k] = (a_0, a_1, b_0, b_1)
// the shell factors; twk: exp(-2 pi i j / Lf) in the arithmetic type.  nx kx rows
// from x0 (mod Lf); the rows hx0, hx1 (-1: none) count half.
template <typename T, int NDX, int SCHEME, int CH>
__device__ inline void loop_no2_body(const T *__restrict__ ekv, const T *__restrict__ pi4,
                                     const T *__restrict__ cvp,
                                     const T *__restrict__ twk, int Lf, int qfx, int qfy, int ky, int x0,
                                     int nx, int hx0, int hx1, T lam, int deriv, T (&Sr)[NREAL], T (&Sc)[NCPLX][2],
                                     T (&Ar)[NDX - 1][NREAL], T (&Br)[NDX - 1][NREAL],
                                     T (&Ac)[NDX - 1][NCPLX][2], T (&Bc)[NDX - 1][NCPLX][2]) {
  constexpr T sg = (CH == 0) ? T(1) : T(-1);
  int kpy = (CH == 0) ? (qfy - ky) : (ky - qfy);
  kpy = ((kpy % Lf) + Lf) % Lf;
  int kpx = (CH == 0) ? (qfx - x0) : (x0 - qfx);
  kpx = ((kpx % Lf) + Lf) % Lf;
  // phase indices (kx (d + 1)) mod Lf, advanced with kx (wave-uniform)
  int jd[NDX - 1];
#pragma unroll
  for (int d = 0; d < NDX - 1; ++d) jd[d] = (int)(((long long)x0 * (d + 1)) % Lf);
  constexpr bool SHELL = SCHEME == CUT_SHELL;
  struct Pt {
    V4<T> ek, pk, cv;
  };
  // point (row, col) of a k-major array: row = kx (wave-uniform), col = ky (per lane):
  // raw buffer loads, descriptor and row offset in scalar registers, the lane's
  // 32-bit byte offset as the only vector operand
  const unsigned nbytes = (unsigned)Lf * Lf * 4u * (unsigned)sizeof(T);
  const auto rs_e = make_rsrc(ekv, nbytes), rs_p = make_rsrc(pi4, nbytes);
  const auto rs_c = make_rsrc(SHELL ? cvp : ekv, nbytes);
  auto load = [&](unsigned row, unsigned col, Pt &p) {
    if constexpr (sizeof(T) == 4) {
      const unsigned soff = row * (unsigned)Lf * 16u, voff = col * 16u;
      p.ek = ld4_buf(rs_e, voff, soff);
      p.pk = ld4_buf(rs_p, voff, soff);
      if constexpr (SHELL) p.cv = ld4_buf(rs_c, voff, soff);
    } else {
      const unsigned soff = row * (unsigned)Lf * 32u, voff = col * 32u;
      p.ek = ld4d_buf(rs_e, voff, soff);
      p.pk = ld4d_buf(rs_p, voff, soff);
      if constexpr (SHELL) p.cv = ld4d_buf(rs_c, voff, soff);
    }
  };
  // k' row of the next kx
  auto next_kpx = [&]() {
    kpx += (CH == 0) ? -1 : 1;
    kpx = kpx < 0 ? kpx + Lf : (kpx >= Lf ? kpx - Lf : kpx);
  };
  // arithmetic of one k-point (k data ck, k' data cp), in kx order
  auto point = [&](const Pt &ck, const Pt &cp, int kx) {
      const T ekm[2] = {ck.ek.x, ck.ek.y}, Kkm[2] = {ck.ek.z, ck.ek.w};
      const T P0 = ck.pk.x, P1 = ck.pk.y, Pr = ck.pk.z, Pi = ck.pk.w;
      const T epn[2] = {cp.ek.x, cp.ek.y}, Kpn[2] = {cp.ek.z, cp.ek.w};
      const T X0 = cp.pk.x, X1 = cp.pk.y, Xr = cp.pk.z, Xi = sg * cp.pk.w;
      // loop kernels L_mn: pp (K(e1)+K(e2))/(e1+e2), ph -(K(e1)-K(e2))/(e1-e2); divided
      // difference of K at x = e_m(k), y = -sg e_n(k').  A branch for the waves with a
      // near-degenerate lane (one test of the smallest difference against the widest
      // switch), which takes the mean for the pairs that are (all four there: Rashba
      // FP32, 9 form factors, L 24: 562 us, the pairs alone 548)
      T L[2][2], den[2][2];
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          den[m][n] = ekm[m] + sg * epn[n];
          L[m][n] = sg * (Kkm[m] + sg * Kpn[n]) * rcp_fast(den[m][n]);
        }
      const T dmin = fmin(fmin(fmin(fabs(den[0][0]), fabs(den[0][1])), fabs(den[1][0])), fabs(den[1][1]));
      const T ex = dd_scheme(SCHEME) == CUT_TEMPERATURE
                       ? lam
                       : lam + fmax(fabs(ekm[0]), fabs(ekm[1])) + fmax(fabs(epn[0]), fabs(epn[1]));
      if (__builtin_expect(!(dmin > degen_rel<T>::v * ex), 0)) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int n = 0; n < 2; ++n)
            if (near_degenerate(den[m][n], ekm[m], -sg * epn[n], lam, dd_scheme(SCHEME)))
              L[m][n] = sg * near_mean(ekm[m], -sg * epn[n], lam, dd_scheme(SCHEME), deriv);
      }
      if constexpr (SHELL) {
        // shell factor a_m(k) b_n(k') + b_m(k) a_n(k')
        const T ak[2] = {ck.cv.x, ck.cv.y}, bk[2] = {ck.cv.z, ck.cv.w};
        const T ap[2] = {cp.cv.x, cp.cv.y}, bp[2] = {cp.cv.z, cp.cv.w};
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int n = 0; n < 2; ++n) L[m][n] *= fma(ak[m], bp[n], bk[m] * ap[n]);
      }
      if (kx == hx0 || kx == hx1) {  // wave-uniform, at most two rows of a q
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int n = 0; n < 2; ++n) L[m][n] *= T(0.5);
      }
      // W_1 = alpha_1 X_0 + L_11 1, D = W_0 - W_1 = (alpha_0 - alpha_1) X_0 + (L_01 - L_11) 1
      const T al0 = L[0][0] - L[0][1], al1 = L[1][0] - L[1][1];
      const T dal = al0 - al1, dl = L[0][1] - L[1][1];
      const T W1d0 = fma(al1, X0, L[1][1]), W1d1 = fma(al1, X1, L[1][1]);
      const T W1r = al1 * Xr, W1i = al1 * Xi;
      const T Dd0 = fma(dal, X0, dl), Dd1 = fma(dal, X1, dl);
      const T Dr = dal * Xr, Di = dal * Xi;
      // the 10 distinct entries of M = Pi_0 (x) D + 1 (x) W_1
      T mr[NREAL], mc[NCPLX][2];
      mr[0] = fma(P0, Dd0, W1d0);  // (0,0,0,0)
      mr[1] = fma(P0, Dd1, W1d1);  // (0,1,0,1)
      mr[2] = fma(P1, Dd0, W1d0);  // (1,0,1,0)
      mr[3] = fma(P1, Dd1, W1d1);  // (1,1,1,1)
      mc[0][0] = fma(P0, Dr, W1r);  // (0,0,0,1)
      mc[0][1] = fma(P0, Di, W1i);
      mc[1][0] = fma(P1, Dr, W1r);  // (1,0,1,1)
      mc[1][1] = fma(P1, Di, W1i);
      mc[2][0] = Pr * Dd0;  // (0,0,1,0)
      mc[2][1] = Pi * Dd0;
      mc[3][0] = Pr * Dd1;  // (0,1,1,1)
      mc[3][1] = Pi * Dd1;
      mc[4][0] = fma(Pr, Dr, -Pi * Di);  // (0,0,1,1): Pi_0[01] D[01]
      mc[4][1] = fma(Pr, Di, Pi * Dr);
      mc[5][0] = fma(Pr, Dr, Pi * Di);  // (0,1,1,0): Pi_0[01] D[10] = Pi_0[01] conj(D[01])
      mc[5][1] = fma(Pi, Dr, -Pr * Di);
#pragma unroll
      for (int t = 0; t < NREAL; ++t) Sr[t] += mr[t];
#pragma unroll
      for (int t = 0; t < NCPLX; ++t) {
        Sc[t][0] += mc[t][0];
        Sc[t][1] += mc[t][1];
      }
#pragma unroll
      for (int d = 0; d < NDX - 1; ++d) {
        const int j = jd[d];
        jd[d] = j + d + 1 >= Lf ? j + d + 1 - Lf : j + d + 1;
        const T c = twk[2 * j], s = twk[2 * j + 1];  // e^{-i 2 pi kx dx / Lf}, wave-uniform
#pragma unroll
        for (int t = 0; t < NREAL; ++t) {
          Ar[d][t] = fma(c, mr[t], Ar[d][t]);
          Br[d][t] = fma(s, mr[t], Br[d][t]);
        }
#pragma unroll
        for (int t = 0; t < NCPLX; ++t) {
          Ac[d][t][0] = fma(c, mc[t][0], Ac[d][t][0]);
          Ac[d][t][1] = fma(c, mc[t][1], Ac[d][t][1]);
          Bc[d][t][0] = fma(s, mc[t][0], Bc[d][t][0]);
          Bc[d][t][1] = fma(s, mc[t][1], Bc[d][t][1]);
        }
      }
  };
  const unsigned uky = (unsigned)ky, ukpy = (unsigned)kpy;
  if constexpr (sizeof(T) == 4 && NDX > 3) {
    // software pipeline with two register sets: the loads of point kx + 1 are
    // issued before the arithmetic of point kx; a prefetch past the chunk
    // re-reads the current point and is not used
    Pt ak, ap, bk, bp;
    load(x0, uky, ak);
    load(kpx, ukpy, ap);
    int kx = x0, i = 0;
    for (; i + 1 < nx; i += 2) {
      const int kb = kx + 1 == Lf ? 0 : kx + 1;
      next_kpx();
      load(kb, uky, bk);
      load(kpx, ukpy, bp);
      point(ak, ap, kx);
      const bool more = i + 2 < nx;
      if (more) next_kpx();
      kx = kb + 1 == Lf ? 0 : kb + 1;
      load(more ? kx : kb, uky, ak);
      load(kpx, ukpy, ap);
      point(bk, bp, kb);
    }
    if (i < nx) point(ak, ap, kx);
  } else {
    // plain order, one register set: FP32 with dx < 3 then fits four waves per
    // SIMD, which hide the load latency better than the second set does at three
    // (Rashba loops, 9 form factors, 24 x 24 refined 24x: 479 us with it, 455);
    // FP64 is at one or two waves per SIMD anyway
    int kx = x0;
    for (int i = 0; i < nx; ++i) {
      Pt ck, cp;
      load(kx, uky, ck);
      load(kpx, ukpy, cp);
      point(ck, cp, kx);
      next_kpx();
      kx = kx + 1 == Lf ? 0 : kx + 1;
    }
  }
}

// A workgroup holds QW waves that share the ky block and kx chunk and take QW
// consecutive items (channel and coarse q) of the item list: they read nearly
// the same k addresses and overlapping k -/+ q rows at the same time.
// Workgroups are handed to the 8 XCDs round-robin by linear id; each XCD is
// given a contiguous slice of the work, ordered (ky block, item group, kx
// chunk, channel) from fastest to slowest, so that co-resident workgroups
// share rows in its L2.
constexpr int N_XCD = 8;

// waves per SIMD that the sums of a lane leave room for
template <typename T, int NDX>
constexpr int no2_waves() {
  return NDX > 3 ? (sizeof(T) == 8 ? 1 : 2) : (sizeof(T) == 8 ? 2 : 4);
}

template <typename T>
struct loop_waves {
  static constexpr int v = (sizeof(T) == 4) ? 4 : 2;
};

// End of a kx chunk: the sums over the wave's 64 ky with e^{-i 2 pi ky dy / Lf}.
// The 16 real values of each of the 2 NDX - 1 kx sums (S, and A, B per dx) go
// through LDS into the left operand of 16 x 16 x 4 matrix products against the
// real phases (1, and cos, sin per dy), K the ky; the entries are put together
// from these at the end.  With vector sums over the rebuilt 16 complex entries
// (three times the products, an LDS read for each) the kernel took 35 -> 24 us
// (Hubbard, 5 form factors, FP64, L 8), 87 -> 64 (Rashba, 13, FP64, L 15), 548 ->
// 528 (Rashba, 9, FP32, L 24).  The products with the kx phases stay in the vector
// unit: on the 4 x 4 x 1 matrix instruction, which is outer products of the lanes'
// own values, they took as long (542 us), as it keeps the vector unit from issuing.
constexpr int LDB = 68;  // row stride of the wave's LDS: 16 rows x 4 ky on different banks

typedef float f32x4a __attribute__((ext_vector_type(4)));
typedef double f64x4a __attribute__((ext_vector_type(4)));
__device__ inline void mac16(f32x4a &c, float a, float b) { c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ inline void mac16(f64x4a &c, double a, double b) { c = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
template <typename T>
struct Acc16;
template <>
struct Acc16<float> {
  typedef f32x4a type;
  static __device__ inline int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};
template <>
struct Acc16<double> {
  typedef f64x4a type;
  static __device__ inline int row(int lane, int r) { return 4 * r + (lane >> 4); }
};

// per tau: index of its (real part's) value, bit 4: complex, bit 5: the partner (conjugate)
__device__ constexpr unsigned char TAU_VALUE[16] = {0, 16 + 4, 16 + 8, 16 + 12, 48 + 4, 1, 16 + 14, 16 + 10,
                                                    48 + 8, 48 + 14, 2, 16 + 6, 48 + 12, 48 + 10, 48 + 6, 3};

template <typename T, int NDX, int NDY, int QW>
__device__ __forceinline__ void loop_no2_contract(const T (&Sr)[NREAL], const T (&Sc)[NCPLX][2],
                                                  const T (&Ar)[NDX - 1][NREAL], const T (&Br)[NDX - 1][NREAL],
                                                  const T (&Ac)[NDX - 1][NCPLX][2], const T (&Bc)[NDX - 1][NCPLX][2],
                                                  const double *__restrict__ tw, int Lf, int kyb, T (&buf)[32][LDB],
                                                  T (&phy)[2 * NDY + 1][64], T *__restrict__ out, bool valid) {
  constexpr int NPH = 2 * NDY + 1, NDY2 = 2 * NDY + 1, NV = 2 * NDX - 1;
  static_assert(NV * 16 * NPH <= 32 * LDB, "the sums fit the wave's LDS");
  const int lane = threadIdx.x & 63;
  for (int i = threadIdx.x; i < NPH * 64; i += 64 * QW) {
    const int p = i >> 6, l = i & 63, k = kyb * 64 + l, j = (k * ((p + 1) >> 1)) % Lf;
    phy[p][l] = k < Lf ? (p == 0 ? T(1) : (T)tw[2 * j + 1 - (p & 1)]) : T(0);
  }
  __syncthreads();
  const int col = lane & 15, kg = lane >> 4;
  T ph[16];
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    const T v = phy[min(col, NPH - 1)][4 * s + kg];
    ph[s] = col < NPH ? v : T(0);
  }
  typename Acc16<T>::type acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int h = 16 * (v & 1), d = (v - 1) >> 1;
#pragma unroll
    for (int t = 0; t < NREAL; ++t) buf[h + t][lane] = v == 0 ? Sr[t] : (v & 1) ? Ar[d][t] : Br[d][t];
#pragma unroll
    for (int t = 0; t < 2 * NCPLX; ++t)
      buf[h + NREAL + t][lane] = v == 0 ? Sc[t >> 1][t & 1] : (v & 1) ? Ac[d][t >> 1][t & 1] : Bc[d][t >> 1][t & 1];
    __builtin_amdgcn_wave_barrier();  // the wave's own LDS
    acc[v] = typename Acc16<T>::type{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 16; ++s) mac16(acc[v], buf[h + col][4 * s + kg], ph[s]);
  }
  __builtin_amdgcn_wave_barrier();
  T *R = &buf[0][0];  // [vector][value][phase]
  if (col < NPH) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) R[(v * 16 + Acc16<T>::row(lane, r)) * NPH + col] = acc[v][r];
  }
  __builtin_amdgcn_wave_barrier();
  for (int o = lane; o < NDX * NDY2 * 16; o += 64) {
    const int t = o & 15, dyi = (o >> 4) % NDY2, dx = (o >> 4) / NDY2, dy = dyi - NDY, y = abs(dy);
    const int code = TAU_VALUE[t], i0 = code & 15;
    const T pf = (code & 16) ? ((code & 32) ? T(-1) : T(1)) : T(0), bw = dx ? T(1) : T(0);
    const T sy = dy == 0 ? T(0) : dy < 0 ? T(-1) : T(1);
    const int jc = y ? 2 * y - 1 : 0, js = 2 * y;
    const T *A = R + (dx ? 2 * dx - 1 : 0) * 16 * NPH, *B = R + 2 * dx * 16 * NPH;
    const int k0 = i0 * NPH, k1 = (i0 + ((code >> 4) & 1)) * NPH;
    // the entry's kx sum: re = A.re -+ B.im, im = +-A.im + B.re (the partner: lower sign)
    const T rc = A[k0 + jc] - pf * bw * B[k1 + jc], ic = pf * A[k1 + jc] + bw * B[k0 + jc];
    const T rs = sy * (A[k0 + js] - pf * bw * B[k1 + js]), is = sy * (pf * A[k1 + js] + bw * B[k0 + js]);
    if (valid) {
      out[2 * o] = rc - is;
      out[2 * o + 1] = ic + rs;
    }
  }
}

// One work item (ky block, item group, kx chunk, channel) of QW waves, w its
// index; bufs and phy are the workgroup's LDS.
template <typename T, int NDX, int NDY, int SCHEME, int QW>
__device__ __forceinline__ void loop_no2_item(const T *__restrict__ ekv, const T *__restrict__ pi4,
                                              const T *__restrict__ cvp, const double *__restrict__ tw,
                                              const T *__restrict__ twk, int Lq, int n_ref, int Lf, int nkyb,
                                              int kxper, int nparts, int half, const int *__restrict__ items, int n_pp,
                                              int n_ph, int w, T lam, int deriv,
                                              T *__restrict__ partial, T (&bufs)[QW][32][LDB],
                                              T (&phy)[2 * NDY + 1][64]) {
  constexpr int NDY2 = 2 * NDY + 1;
  const int tid = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int kyb = w % nkyb;
  w /= nkyb;
  // the pp items' chunks come first, then the ph items'
  const int g_pp = (n_pp + QW - 1) / QW, g_ph = (n_ph + QW - 1) / QW;
  const int c_pp = (loop_rows_max(Lf, half & 1) + kxper - 1) / kxper;
  const int w_pp = g_pp * c_pp, ch = w >= w_pp ? 1 : 0;
  w -= ch ? w_pp : 0;
  const int ng = ch ? g_ph : g_pp, kxc = w / ng;
  const int idx = (w % ng) * QW + wv, n_it = ch ? n_ph : n_pp;
  const bool qvalid = idx < n_it;
  const int it = (ch ? n_pp : 0) + (qvalid ? idx : n_it - 1);
  // one coarse q per wave: keep its fine coordinates in scalar registers
  const int qi = __builtin_amdgcn_readfirstlane(items[it] & LOOP_ITEM_Q);
  const int qfx = (qi / Lq) * n_ref, qfy = (qi % Lq) * n_ref;
  const int ky_raw = kyb * 64 + tid;
  const bool active = ky_raw < Lf;
  const int ky = active ? ky_raw : Lf - 1;
  // kx rows of this item and chunk
  int r0, nr, hx0, hx1;
  loop_rows(Lf, qfx, (half >> ch) & 1, r0, nr, hx0, hx1);
  int x0 = r0 + kxc * kxper;
  const int nx = min(kxper, nr - kxc * kxper);
  x0 = x0 >= Lf ? x0 - Lf : x0;

  // S: dx = 0 sums; A/B: sum of cos/sin parts for dx >= 1
  T Sr[NREAL], Sc[NCPLX][2], Ar[NDX - 1][NREAL], Br[NDX - 1][NREAL];
  T Ac[NDX - 1][NCPLX][2], Bc[NDX - 1][NCPLX][2];
#pragma unroll
  for (int t = 0; t < NREAL; ++t) Sr[t] = T(0);
#pragma unroll
  for (int t = 0; t < NCPLX; ++t) Sc[t][0] = Sc[t][1] = T(0);
#pragma unroll
  for (int d = 0; d < NDX - 1; ++d) {
#pragma unroll
    for (int t = 0; t < NREAL; ++t) Ar[d][t] = Br[d][t] = T(0);
#pragma unroll
    for (int t = 0; t < NCPLX; ++t) Ac[d][t][0] = Ac[d][t][1] = Bc[d][t][0] = Bc[d][t][1] = T(0);
  }
  if (ch == 0)
    loop_no2_body<T, NDX, SCHEME, 0>(ekv, pi4, cvp, twk, Lf, qfx, qfy, ky, x0, nx, hx0, hx1, lam, deriv, Sr,
                                     Sc, Ar, Br, Ac,
                                     Bc);
  else
    loop_no2_body<T, NDX, SCHEME, 1>(ekv, pi4, cvp, twk, Lf, qfx, qfy, ky, x0, nx, hx0, hx1, lam, deriv, Sr,
                                     Sc, Ar, Br, Ac,
                                     Bc);

  loop_no2_contract<T, NDX, NDY, QW>(Sr, Sc, Ar, Br, Ac, Bc, tw, Lf, kyb, bufs[wv], phy,
                                     partial + 2 * ((size_t)it * nparts + (kyb + nkyb * kxc)) *
                                                   (size_t)(NDX * NDY2 * 16),
                                     qvalid);
}

template <typename T, int NDX, int NDY, int SCHEME, int QW>
__global__ __launch_bounds__(64 * QW, (no2_waves<T, NDX>())) void loop_no2_kernel(const T *__restrict__ ekv,
                                                           const T *__restrict__ pi4,
                                                           const T *__restrict__ cvp,
                                                           const double *__restrict__ tw, const T *__restrict__ twk,
                                                           int Lq, int n_ref, int Lf, int nkyb, int kxper, int nparts,
                                                           int half, const int *__restrict__ items, int n_pp,
                                                           int n_ph, int n_work, T lam, int deriv,
                                                           T *__restrict__ partial) {
  __shared__ T bufs[QW][32][LDB];
  __shared__ T phy[2 * NDY + 1][64];
  const int xcd = blockIdx.x % N_XCD, slot = blockIdx.x / N_XCD;
  const int base = n_work / N_XCD, rem = n_work % N_XCD;
  if (slot >= base + (xcd < rem ? 1 : 0)) return;  // padding workgroup, no work
  const int w = xcd * base + min(xcd, rem) + slot;
  loop_no2_item<T, NDX, NDY, SCHEME, QW>(ekv, pi4, cvp, tw, twk, Lq, n_ref, Lf, nkyb, kxper, nparts, half, items, n_pp,
                                         n_ph, w, lam, deriv, partial, bufs, phy);
}

// Several instances in one launch: the work of instance i is
// [inst[i].work0, inst[i].work0 + its count), every instance summing both
// channels over all its items; the same work items and partial sums as its
// own launch.
template <typename T, int NDX, int NDY, int SCHEME, int QW>
__global__ __launch_bounds__(64 * QW, (no2_waves<T, NDX>())) void loop_no2_batch_kernel(const No2Inst *__restrict__ inst,
                                                                               int n_inst, int n_work) {
  __shared__ T bufs[QW][32][LDB];
  __shared__ T phy[2 * NDY + 1][64];
  const int xcd = blockIdx.x % N_XCD, slot = blockIdx.x / N_XCD;
  const int base = n_work / N_XCD, rem = n_work % N_XCD;
  if (slot >= base + (xcd < rem ? 1 : 0)) return;  // padding workgroup, no work
  const int w = xcd * base + min(xcd, rem) + slot;
  int i = 0;
  while (i + 1 < n_inst && inst[i + 1].work0 <= w) ++i;
  const No2Inst &d = inst[i];
  loop_no2_item<T, NDX, NDY, SCHEME, QW>((const T *)d.ekv, (const T *)d.pi4, (const T *)d.cvp, d.tw,
                                         (const T *)d.twk, d.Lq, d.n_ref, d.Lf, d.nkyb, d.kxper, d.nparts, d.half,
                                         d.items, d.n_pp, d.n_ph, w - d.work0, (T)d.lam, d.deriv, (T *)d.partial,
                                         bufs, phy);
}

// workgroups of one two-orbital evaluation: per channel (ky blocks) x (kx
// chunks of the rows it sums) x (groups of QW items)
static long long no2_work(const LoopArgs &a, int QW) {
  auto part = [&](int n, int h) {
    return (long long)((n + QW - 1) / QW) * ((loop_rows_max(a.Lf, h) + a.kxper - 1) / a.kxper);
  };
  return a.nkyb * (part(a.n_pp, a.half & 1) + part(a.n_ph, (a.half >> 1) & 1));
}

template <typename T, int NDX, int NDY>
static hipError_t launch_no2(const LoopArgs &a, hipStream_t st) {
  constexpr int QW = loop_waves<T>::v;
  const long long work = no2_work(a, QW);
  if (work < 1 || work > 0x7ffffff0LL) return hipErrorInvalidValue;
  const int n_work = (int)work;
  const int n_wg = ((n_work + N_XCD - 1) / N_XCD) * N_XCD;
  dim3 grid(n_wg), block(64 * QW);
  const T *ekv = (const T *)a.ekv;
  const T *pi4 = (const T *)a.pi4;
  const T *twk = (const T *)(sizeof(T) == 8 ? (const void *)a.tw : a.tw32);
  const T *cvp = (const T *)a.cv;
  if (!ekv || !pi4 || !twk || !a.items) return hipErrorInvalidValue;
  if (a.scheme == CUT_SHELL && !cvp) return hipErrorInvalidValue;
#define TUFRG_NO2_LAUNCH(S)                                                                                         \
  hipLaunchKernelGGL((loop_no2_kernel<T, NDX, NDY, S, QW>), grid, block, 0, st, ekv, pi4, cvp, a.tw, twk, a.Lq,    \
                     a.n_ref, a.Lf, a.nkyb, a.kxper, a.nparts, a.half, a.items, a.n_pp, a.n_ph, n_work, (T)a.lam,  \
                     a.deriv, (T *)a.partial)
  if (a.scheme == CUT_TEMPERATURE)
    TUFRG_NO2_LAUNCH(CUT_TEMPERATURE);
  else if (a.scheme == CUT_OMEGA)
    TUFRG_NO2_LAUNCH(CUT_OMEGA);
  else if (a.scheme == CUT_SHELL)
    TUFRG_NO2_LAUNCH(CUT_SHELL);
  else
    return hipErrorInvalidValue;
#undef TUFRG_NO2_LAUNCH
  return hipGetLastError();
}

template <typename T, int NDX, int NDY>
static hipError_t launch_no2_batch(const LoopArgs *a, const int *idx, int m, No2Inst *desc_h, No2Inst *desc_d,
                                   hipStream_t st) {
  constexpr int QW = loop_waves<T>::v;
  long long work = 0;
  for (int j = 0; j < m; ++j) {
    const LoopArgs &x = a[idx[j]];
    const T *twk = (const T *)(sizeof(T) == 8 ? (const void *)x.tw : x.tw32);
    if (!x.ekv || !x.pi4 || !twk || !x.items || x.n_pp < 1 || x.n_ph < 1) return hipErrorInvalidValue;
    if (x.scheme == CUT_SHELL && !x.cv) return hipErrorInvalidValue;
    No2Inst &d = desc_h[j];
    d.ekv = x.ekv;
    d.pi4 = x.pi4;
    d.cvp = x.cv;
    d.twk = twk;
    d.tw = x.tw;
    d.items = x.items;
    d.partial = x.partial;
    d.lam = x.lam;
    d.Lq = x.Lq;
    d.n_ref = x.n_ref;
    d.Lf = x.Lf;
    d.nkyb = x.nkyb;
    d.kxper = x.kxper;
    d.nparts = x.nparts;
    d.half = x.half;
    d.n_pp = x.n_pp;
    d.n_ph = x.n_ph;
    d.deriv = x.deriv;
    d.work0 = (int)work;
    work += no2_work(x, QW);
    if (work > 0x7ffffff0LL) return hipErrorInvalidValue;
  }
  hipError_t e = hipMemcpyAsync(desc_d, desc_h, m * sizeof(No2Inst), hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return e;
  const int n_work = (int)work;
  const dim3 grid(((n_work + N_XCD - 1) / N_XCD) * N_XCD), block(64 * QW);
  const int scheme = a[idx[0]].scheme;
  if (scheme == CUT_TEMPERATURE)
    hipLaunchKernelGGL((loop_no2_batch_kernel<T, NDX, NDY, CUT_TEMPERATURE, QW>), grid, block, 0, st, desc_d, m,
                       n_work);
  else if (scheme == CUT_OMEGA)
    hipLaunchKernelGGL((loop_no2_batch_kernel<T, NDX, NDY, CUT_OMEGA, QW>), grid, block, 0, st, desc_d, m, n_work);
  else if (scheme == CUT_SHELL)
    hipLaunchKernelGGL((loop_no2_batch_kernel<T, NDX, NDY, CUT_SHELL, QW>), grid, block, 0, st, desc_d, m, n_work);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_loop_batch(const LoopArgs *a, int n, No2Inst *desc_h, No2Inst *desc_d, hipStream_t st) {
  if (n < 1 || !desc_h || !desc_d) return hipErrorInvalidValue;
  const int prec = a[0].prec;
  for (int i = 0; i < n; ++i)
    if (a[i].n_o != 2 || a[i].prec != prec) return hipErrorInvalidValue;
  // one launch per (shape, regulator); the group's descriptors contiguous
  int off = 0;
  for (int shape = 0; shape < 3; ++shape)
    for (int scheme = 0; scheme < 3; ++scheme) {
      std::vector<int> idx;
      for (int i = 0; i < n; ++i) {
        const int sh = (a[i].ndx == 3 && a[i].ndy == 2) ? 0 : (a[i].ndx == 5 && a[i].ndy == 4) ? 1 : 2;
        if (sh == 2 && !(a[i].ndx == 2 && a[i].ndy == 1)) return hipErrorInvalidValue;
        if (sh == shape && a[i].scheme == scheme) idx.push_back(i);
      }
      if (idx.empty()) continue;
      const int m = (int)idx.size();
      hipError_t e;
      if (shape == 0)
        e = prec == 0 ? launch_no2_batch<double, 3, 2>(a, idx.data(), m, desc_h + off, desc_d + off, st)
                      : launch_no2_batch<float, 3, 2>(a, idx.data(), m, desc_h + off, desc_d + off, st);
      else if (shape == 1)
        e = prec == 0 ? launch_no2_batch<double, 5, 4>(a, idx.data(), m, desc_h + off, desc_d + off, st)
                      : launch_no2_batch<float, 5, 4>(a, idx.data(), m, desc_h + off, desc_d + off, st);
      else
        e = prec == 0 ? launch_no2_batch<double, 2, 1>(a, idx.data(), m, desc_h + off, desc_d + off, st)
                      : launch_no2_batch<float, 2, 1>(a, idx.data(), m, desc_h + off, desc_d + off, st);
      if (e != hipSuccess) return e;
      off += m;
    }
  return hipSuccess;
}

hipError_t launch_loop(const LoopArgs &a, hipStream_t st) {
  if (a.n_o == 6) return launch_loop_gen(a, st);
  if (a.n_o != 2) return hipErrorInvalidValue;
  const bool f64 = (a.prec == 0);
  if (a.ndx == 3 && a.ndy == 2) return f64 ? launch_no2<double, 3, 2>(a, st) : launch_no2<float, 3, 2>(a, st);
  if (a.ndx == 5 && a.ndy == 4) return f64 ? launch_no2<double, 5, 4>(a, st) : launch_no2<float, 5, 4>(a, st);
  if (a.ndx == 2 && a.ndy == 1) return f64 ? launch_no2<double, 2, 1>(a, st) : launch_no2<float, 2, 1>(a, st);
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------

// Compact loops from the partial sums: H[dR][tau] of an item is the
// fixed-order FP64 sum of its parts (dx < 0 by hermiticity); a halved sum is
// completed from the reversed entry; the value goes to the item's own slot of
// the output and, transformed, to that of -q.
template <typename PT, int QS>
__global__ __launch_bounds__(256) void loop_finalize_kernel(LoopSym sy, int n_o, int n_items, int nparts,
                                                            int valid_pp, int valid_ph, int ndx,
                                     int ndy, int nD, int ch_first, int n_q_out, const int *__restrict__ items,
                                     const int2 *__restrict__ dst, const int *__restrict__ dlist, double inv_nf,
                                     const PT *__restrict__ partial, double *__restrict__ compact) {
  const int no2 = n_o * n_o, no4 = no2 * no2;
  // several workgroups per item, of 256 / QS entries and QS pieces of the parts
  constexpr int NE = 256 / QS;
  __shared__ double2 sq[QS][NE][2];
  const int nb = gridDim.x / n_items, it = blockIdx.x / nb, lane = threadIdx.x % NE, piece = threadIdx.x / NE;
  const int i_raw = (blockIdx.x - it * nb) * NE + lane, i = min(i_raw, nD * no4 - 1);
  const int iD = i / no4, tau = i - iD * no4;
  const int q = items[it] & LOOP_ITEM_Q, ch = items[it] >> LOOP_ITEM_CH;
  const int dx = dlist[2 * iD], dy = dlist[2 * iD + 1];
  const int ndy2 = 2 * ndy + 1, valid = ch ? valid_ph : valid_pp;
  const size_t per = (size_t)ndx * ndy2 * no4;
  const PT *pi = partial + (size_t)it * nparts * per * 2;
  // address of a partial sum of entry t, for dx < 0 its conjugate's
  const bool cj = dx < 0;
  auto at = [&](int t) {
    if (cj) t = (t % no2) * no2 + t / no2;
    return pi + ((size_t)((cj ? -dx : dx) * ndy2 + (cj ? -dy : dy) + ndy) * no4 + t) * 2;
  };
  const bool half = (sy.half >> ch) & 1;
  double sgn = 1.0;
  const PT *p0 = at(tau), *p1 = at(half ? loop_partner_tau(sy, n_o, ch, tau, sgn) : tau);
  double2 v = make_double2(0.0, 0.0), h = v;
  const int k_end = (piece + 1) * valid / QS;
  for (int k0 = piece * valid / QS; k0 < k_end; k0 += 8) {
    PT a[8][2], b[8][2];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const size_t o = (size_t)min(k0 + u, k_end - 1) * per * 2;
      a[u][0] = p0[o];
      a[u][1] = p0[o + 1];
      b[u][0] = p1[o];
      b[u][1] = p1[o + 1];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (k0 + u >= k_end) break;
      v.x += (double)a[u][0];
      v.y += (double)a[u][1];
      h.x += (double)b[u][0];
      h.y += (double)b[u][1];
    }
  }
  if constexpr (QS > 1) {
    sq[piece][lane][0] = v;
    sq[piece][lane][1] = h;
    __syncthreads();
#pragma unroll
    for (int s = 1; s < QS; ++s) {
      v.x += sq[s][lane][0].x;
      v.y += sq[s][lane][0].y;
      h.x += sq[s][lane][1].x;
      h.y += sq[s][lane][1].y;
    }
  }
  if (piece || i_raw != i) return;
  if (cj) {
    v.y = -v.y;
    h.y = -h.y;
  }
  if (half) loop_add_partner(sy, q, dx, dy, sgn, h, v);
  loop_store(sy, n_o, ch, q, dx, dy, tau, make_double2(v.x * inv_nf, v.y * inv_nf), dst[it], ch - ch_first, n_q_out,
             (size_t)nD * no4, (size_t)iD * no4, (double2 *)compact);
}

hipError_t launch_loop_finalize(const LoopArgs &a, int nD, const int *dlist, double *compact, hipStream_t st) {
  const int no4 = a.n_o * a.n_o * a.n_o * a.n_o, n_items = a.n_pp + a.n_ph;
  const long long total = (long long)n_items * nD * no4;
  if (total < 1 || !a.items || !a.dst) return hipErrorInvalidValue;
  const int ch_first = a.n_pp ? 0 : 1;
  auto valid = [&](int h) { return a.nkyb * ((loop_rows_max(a.Lf, h) + a.kxper - 1) / a.kxper); };
  const int vpp = valid(a.half & 1), vph = valid((a.half >> 1) & 1);
  const double inv = 1.0 / ((double)a.Lf * a.Lf);
  const LoopSym sy{a.trs, a.half, a.Lq, (const double2 *)a.twq};
  // many parts in a row are a chain of loads: four threads an entry (26 parts of 66
  // items: 7.7 -> 5.7 us); with few parts that only costs (3 parts of 121 items,
  // 36 entries squared, 62 -> 129 us)
  const int qs = std::max(vpp, vph) > 16 ? 4 : 1;
  const dim3 grid((unsigned)n_items * (unsigned)((nD * no4 * qs + 255) / 256)), block(256);
#define TUFRG_FIN(PT, QS)                                                                                           \
  hipLaunchKernelGGL((loop_finalize_kernel<PT, QS>), grid, block, 0, st, sy, a.n_o, n_items, a.nparts, vpp, vph,     \
                     a.ndx, a.ndy, nD, ch_first, a.n_q_out, a.items, a.dst, dlist, inv, (const PT *)a.partial, compact)
  if (a.prec == 0) {
    if (qs > 1)
      TUFRG_FIN(double, 4);
    else
      TUFRG_FIN(double, 1);
  } else {
    if (qs > 1)
      TUFRG_FIN(float, 4);
    else
      TUFRG_FIN(float, 1);
  }
#undef TUFRG_FIN
  return hipGetLastError();
}

__global__ void loop_expand_kernel(int n_o, int n_ff, int nD, int n_q, const int *__restrict__ didx,
                                   const double *__restrict__ compact, double *__restrict__ out) {
  const int no2 = n_o * n_o, no4 = no2 * no2;
  const int B = n_ff * no2;
  const long long total = (long long)n_q * B * B;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int col = (int)(i % B), row = (int)((i / B) % B);
  const long long q = i / ((long long)B * B);
  const int r1 = row / no2, ab = row % no2, r2 = col / no2, cd = col % no2;
  const int iD = didx[r1 * n_ff + r2];
  const size_t src = ((size_t)q * nD + iD) * no4 + (size_t)ab * no2 + cd;
  out[2 * i] = compact[2 * src];
  out[2 * i + 1] = compact[2 * src + 1];
}

hipError_t launch_loop_expand(int n_o, int n_ff, int nD, int n_q, const int *didx, const double *compact,
                              double *out, hipStream_t st) {
  const int B = n_ff * n_o * n_o;
  const long long total = (long long)n_q * B * B;
  hipLaunchKernelGGL(loop_expand_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, n_o, n_ff, nD,
                     n_q, didx, compact, out);
  return hipGetLastError();
}

}  // namespace tufrg
