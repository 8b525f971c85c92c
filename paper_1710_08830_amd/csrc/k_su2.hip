// SU(2)-reduced flow of one orbital per site (spin-rotation invariant): the
// spinful exchange propagators carry two spin structures,
//   P = p d13 d24 - p^x d14 d23,  p^x^{RR'}(s) = e^{is.R'} p^{R,-R'}(s),
//   C = c d13 d24 - d d14 d23,
// so three n_ff x n_ff functions p, c, d per q carry the state (Sec. 2
// channel definitions, Sec. 3.1 matrix RGE with spin-independent loops).  The
// reduced equations (the paper cites them without printing them) are
//   dp = -(a~ Lpp a~x + a~x Lpp a~),
//   dc = 2 (2 c~ Lph c~ - c~ Lph d~ - d~ Lph c~),
//   dd = -2 d~ Lph d~,
// with a~ = p + v + PC(c) + PD(d), c~ = c + v + CP(p) + CD(d),
// d~ = d + v + CP(p^x) + CD(c) from the scalar cross projections of Sec. 3.3
// (v the onsite coefficient of d13 d24 - d14 d23).
//   loop1_kernel       partial sums of the one-band loops, FP64
//   su2_exch_kernel    X -> X^x
//   su2_gather_kernel  the rho-space gathers of a~, c~, d~
//   su2_bundle_kernel  dp (pp channel) or dc, dd (ph channel) per q
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "loop_sym.h"

namespace tufrg {

// One-band loops, FP64: the sum over k of e^{-ik.dR} L(e(k), e(k')) (k' = q - k
// for pp, k - q for ph) of one item (channel, coarse q), ky block of 64 and
// chunk of kx rows per wave.  Like the two-orbital kernel: a lane owns one ky
// and walks kx with wave-uniform kx phases (1 + 2 (NDX - 1) real sums), the ky
// phases are contracted through LDS at the end of the chunk, and the kx rows
// and coarse q that follow by symmetry are left out (loop_sym.h).  Bound by
// FP64 vector issue (the divided difference, about 20 operations per point).
template <int NDX, int NDY, int QW>
__global__ __launch_bounds__(64 * QW) void loop1_kernel(int Lq, int n_ref, int Lf, int nkyb, int kxper, int nparts,
                                                        int half, const int *__restrict__ items, int n_pp, int n_ph,
                                                        const double *__restrict__ e, const double *__restrict__ kv,
                                                        const double *__restrict__ tw, double lam, int scheme,
                                                        int deriv, double *__restrict__ part) {
  constexpr int NDY2 = 2 * NDY + 1, NV = 2 * NDX - 1;
  __shared__ double buf[QW][NV][65];
  __shared__ double phy[NDY2][2][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int w = blockIdx.x;
  const int kyb = w % nkyb;
  w /= nkyb;
  const int g_pp = (n_pp + QW - 1) / QW, g_ph = (n_ph + QW - 1) / QW;
  const int c_pp = (loop_rows_max(Lf, half & 1) + kxper - 1) / kxper;
  const int w_pp = g_pp * c_pp, ch = w >= w_pp ? 1 : 0;
  w -= ch ? w_pp : 0;
  const int ng = ch ? g_ph : g_pp, kxc = w / ng;
  const int idx = (w % ng) * QW + wv, n_it = ch ? n_ph : n_pp;
  const bool qvalid = idx < n_it;
  const int it = (ch ? n_pp : 0) + (qvalid ? idx : n_it - 1);
  const int q = __builtin_amdgcn_readfirstlane(items[it] & LOOP_ITEM_Q);
  const int qfx = (q / Lq) * n_ref, qfy = (q % Lq) * n_ref;
  const double sg = ch == 0 ? 1.0 : -1.0;
  const int ky_raw = kyb * 64 + lane, ky = min(ky_raw, Lf - 1);
  int kpy = ch == 0 ? qfy - ky : ky - qfy;
  kpy += kpy < 0 ? Lf : 0;
  int r0, nr, hx0, hx1;
  loop_rows(Lf, qfx, (half >> ch) & 1, r0, nr, hx0, hx1);
  int kx = r0 + kxc * kxper;
  const int nx = min(kxper, nr - kxc * kxper);
  kx = kx >= Lf ? kx - Lf : kx;
  int kpx = ch == 0 ? qfx - kx : kx - qfx;
  kpx += kpx < 0 ? Lf : 0;
  double S = 0.0, A[NDX - 1], Bv[NDX - 1];
  int jd[NDX - 1];
#pragma unroll
  for (int d = 0; d < NDX - 1; ++d) {
    A[d] = Bv[d] = 0.0;
    jd[d] = (int)(((long long)kx * (d + 1)) % Lf);
  }
  // the values of a row one row ahead (the branches of the divided difference keep
  // the compiler from it): 24 x 24 refined 12 x, 9 form factors, 101 -> 83 us
  struct Row {
    double ek, ep, vk, vp;
  };
  auto load = [&](int x, int xp) __attribute__((always_inline)) {
    const size_t o = (size_t)x * Lf, op = (size_t)xp * Lf;
    return Row{e[o + ky], e[op + kpy], kv[o + ky], kv[op + kpy]};
  };
  Row next = load(kx, kpx);
#pragma unroll 2
  for (int i = 0; i < nx; ++i) {
    const Row c = next;
    const int kn = kx + 1 == Lf ? 0 : kx + 1;
    kpx += ch == 0 ? -1 : 1;
    kpx = kpx < 0 ? kpx + Lf : (kpx >= Lf ? kpx - Lf : kpx);
    next = load(kn, kpx);
    double l = sg * divided_difference(c.ek, -sg * c.ep, c.vk, -sg * c.vp, lam, scheme, deriv);
    if (kx == hx0 || kx == hx1) l *= 0.5;
    S += l;
#pragma unroll
    for (int d = 0; d < NDX - 1; ++d) {
      const int j = jd[d];
      jd[d] = j + d + 1 >= Lf ? j + d + 1 - Lf : j + d + 1;
      A[d] = fma(tw[2 * j], l, A[d]);  // e^{-i kx dx}, wave-uniform
      Bv[d] = fma(tw[2 * j + 1], l, Bv[d]);
    }
    kx = kn;
  }
  const double on = ky_raw < Lf ? 1.0 : 0.0;
  buf[wv][0][lane] = on * S;
#pragma unroll
  for (int d = 0; d < NDX - 1; ++d) {
    buf[wv][1 + 2 * d][lane] = on * A[d];
    buf[wv][2 + 2 * d][lane] = on * Bv[d];
  }
  for (int i = wv; i < NDY2; i += QW) {
    int j = (int)(((long long)ky_raw * (i - NDY)) % Lf);
    j += j < 0 ? Lf : 0;
    phy[i][0][lane] = tw[2 * j];
    phy[i][1][lane] = tw[2 * j + 1];
  }
  __syncthreads();
  if (lane < NDX * NDY2 && qvalid) {
    const int dx = lane / NDY2, dyi = lane % NDY2;
    const double *a = buf[wv][dx ? 2 * dx - 1 : 0], *b = buf[wv][dx ? 2 * dx : 0];
    const double fb = dx ? 1.0 : 0.0;
    double sr = 0.0, si = 0.0;
#pragma unroll 8
    for (int l = 0; l < 64; ++l) {
      const double re = a[l], im = fb * b[l], pr = phy[dyi][0][l], pi = phy[dyi][1][l];
      sr = fma(pr, re, fma(-pi, im, sr));
      si = fma(pr, im, fma(pi, re, si));
    }
    const size_t o = ((size_t)it * nparts + (kyb + nkyb * kxc)) * (NDX * NDY2) + lane;
    part[2 * o] = sr;
    part[2 * o + 1] = si;
  }
}

hipError_t launch_loop1(const LoopArgs &a, hipStream_t st) {
  constexpr int QW = 4;
  if (a.n_o != 1 || a.prec != 0 || !a.items || a.n_pp + a.n_ph < 1 || a.scheme == CUT_SHELL || !a.partial)
    return hipErrorInvalidValue;
  auto work = [&](int n, int h) {
    return (long long)((n + QW - 1) / QW) * ((loop_rows_max(a.Lf, h) + a.kxper - 1) / a.kxper);
  };
  const long long n = a.nkyb * (work(a.n_pp, a.half & 1) + work(a.n_ph, (a.half >> 1) & 1));
  if (n < 1 || n > 0x7fffffffLL) return hipErrorInvalidValue;
  const double *e = (const double *)a.band, *kv = (const double *)a.kv;
#define TUFRG_L1(X, Y)                                                                                             \
  hipLaunchKernelGGL((loop1_kernel<X, Y, QW>), dim3((unsigned)n), dim3(64 * QW), 0, st, a.Lq, a.n_ref, a.Lf, a.nkyb, \
                     a.kxper, a.nparts, a.half, a.items, a.n_pp, a.n_ph, e, kv, a.tw, a.lam, a.scheme, a.deriv,    \
                     (double *)a.partial)
  if (a.ndx == 2 && a.ndy == 1)
    TUFRG_L1(2, 1);
  else if (a.ndx == 3 && a.ndy == 2)
    TUFRG_L1(3, 2);
  else if (a.ndx == 5 && a.ndy == 4)
    TUFRG_L1(5, 4);
  else
    return hipErrorInvalidValue;
#undef TUFRG_L1
  return hipGetLastError();
}

// Xx[q][i][j] = e^{iq.R_j} X[q][i][neg(j)], neg(j) the index of -R_j
__global__ void su2_exch_kernel(int n_ff, int Nq, int Lq, const int *__restrict__ ff, const int *__restrict__ fneg,
                                const double2 *__restrict__ twq, const double2 *__restrict__ X,
                                double2 *__restrict__ Xx) {
  const long long n = (long long)Nq * n_ff * n_ff;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const int j = (int)(i % n_ff), r = (int)((i / n_ff) % n_ff);
    const int q = (int)(i / ((long long)n_ff * n_ff));
    int ph = ((q / Lq) * ff[2 * j] + (q % Lq) * ff[2 * j + 1]) % Lq;
    ph += ph < 0 ? Lq : 0;
    const double2 x = X[((long long)q * n_ff + r) * n_ff + fneg[j]], t = twq[ph];
    Xx[i] = make_double2(t.x * x.x - t.y * x.y, t.x * x.y + t.y * x.x);
  }
}

hipError_t launch_su2_exch(int n_ff, int Nq, int Lq, const int *ff, const int *fneg, const double *twq,
                           const double *X, double *Xx, hipStream_t st) {
  const long long n = (long long)Nq * n_ff * n_ff;
  const unsigned blocks = (unsigned)std::max<long long>(1, std::min<long long>((n + 255) / 256, 65536));
  hipLaunchKernelGGL(su2_exch_kernel, dim3(blocks), dim3(256), 0, st, n_ff, Nq, Lq, ff, fneg, (const double2 *)twq,
                     (const double2 *)X, (double2 *)Xx);
  return hipGetLastError();
}

// G[w][iD][i][j] for w = a~, c~, d~ from the rho-space coefficients
// rA = (p, c)(rho) and rB = (p^x, d)(rho), each [2][nD][B][B]:
//   a~: c(rho)[R+rho, R'-rho]  + d(rho-R')[R+rho-R', -rho]
//   c~: p(rho)[R+rho, R'-rho]  + d(-R')[R-R'+rho, rho]
//   d~: px(rho)[R+rho, R'-rho] + c(-R')[R-R'+rho, rho]
// (terms whose labels leave S, or whose coefficient argument leaves D, dropped)
__global__ void su2_gather_kernel(int B, int nD, const int *__restrict__ ff, const int *__restrict__ dlist,
                                  const int *__restrict__ ffgrid, const int *__restrict__ dgrid,
                                  const double2 *__restrict__ rA, const double2 *__restrict__ rB,
                                  double2 *__restrict__ G) {
  const long long BB = (long long)B * B;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 3LL * nD * BB) return;
  const int col = (int)(i % B), row = (int)((i / B) % B), iD = (int)((i / BB) % nD), w = (int)(i / (BB * nD));
  auto fidx = [&](int x, int y) -> int {
    if (x < -8 || x > 8 || y < -8 || y > 8) return -1;
    return ffgrid[(x + 8) * 17 + (y + 8)];
  };
  auto didx = [&](int x, int y) -> int {
    if (x < -8 || x > 8 || y < -8 || y > 8) return -1;
    return dgrid[(x + 8) * 17 + (y + 8)];
  };
  const int Rx = ff[2 * row], Ry = ff[2 * row + 1], Sx = ff[2 * col], Sy = ff[2 * col + 1];
  const int px = dlist[2 * iD], py = dlist[2 * iD + 1];
  const double2 *p = rA, *c = rA + nD * BB, *pxr = rB, *d = rB + nD * BB;
  double gr = 0.0, gi = 0.0;
  const int A = fidx(Rx + px, Ry + py), Bc = fidx(Sx - px, Sy - py);
  if (A >= 0 && Bc >= 0) {
    const double2 v = (w == 0 ? c : w == 1 ? p : pxr)[(long long)iD * BB + (long long)A * B + Bc];
    gr += v.x;
    gi += v.y;
  }
  if (w == 0) {
    const int A2 = fidx(Rx + px - Sx, Ry + py - Sy), B2 = fidx(-px, -py), D2 = didx(px - Sx, py - Sy);
    if (A2 >= 0 && B2 >= 0 && D2 >= 0) {
      const double2 v = d[(long long)D2 * BB + (long long)A2 * B + B2];
      gr += v.x;
      gi += v.y;
    }
  } else {
    const int A4 = fidx(Rx - Sx + px, Ry - Sy + py), B4 = fidx(px, py), D4 = didx(-Sx, -Sy);
    if (A4 >= 0 && B4 >= 0 && D4 >= 0) {
      const double2 v = (w == 1 ? d : c)[(long long)D4 * BB + (long long)A4 * B + B4];
      gr += v.x;
      gi += v.y;
    }
  }
  G[i] = make_double2(gr, gi);
}

hipError_t launch_su2_gather(int B, int nD, const int *ff, const int *dlist, const int *ffgrid, const int *dgrid,
                             const double *rA, const double *rB, double *G, hipStream_t st) {
  const long long n = 3LL * nD * B * B;
  hipLaunchKernelGGL(su2_gather_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, B, nD, ff, dlist, ffgrid,
                     dgrid, (const double2 *)rA, (const double2 *)rB, (double2 *)G);
  return hipGetLastError();
}

// per q: channel 0: dp = f (-(X1 T1 + X2 T2)), T1 = L X2, T2 = L X1 with
// (X1, X2) = (a~, a~x), L = Lpp; channel 1: (X1, X2) = (c~, d~), L = Lph,
// U1 = L X1, U2 = L X2, dc = f 2 (2 X1 U1 - X1 U2 - X2 U1), dd = f (-2 X2 U2);
// L expanded from its compact form (didx: dR index of (R1, R2)); LDS holds
// X1, X2, L and the two products (5 B^2 complex)
__global__ __launch_bounds__(256) void su2_bundle_kernel(int B, int Nq, int nD, const int *__restrict__ didx,
                                                         const double2 *__restrict__ Lc,
                                                         const double2 *__restrict__ Va,
                                                         const double2 *__restrict__ Vax,
                                                         const double2 *__restrict__ Vc,
                                                         const double2 *__restrict__ Vd, double f,
                                                         double2 *__restrict__ dp, double2 *__restrict__ dc,
                                                         double2 *__restrict__ dd) {
  extern __shared__ double2 sm[];
  const int BB = B * B;
  double2 *X1 = sm, *X2 = sm + BB, *L = sm + 2 * BB, *T1 = sm + 3 * BB, *T2 = sm + 4 * BB;
  const int q = blockIdx.x, ch = blockIdx.y, tid = threadIdx.x;
  const size_t off = (size_t)q * BB;
  const double2 *S1 = ch == 0 ? Va : Vc, *S2 = ch == 0 ? Vax : Vd;
  const double2 *Lq = Lc + ((size_t)ch * Nq + q) * nD;
  for (int i = tid; i < BB; i += blockDim.x) {
    X1[i] = S1[off + i];
    X2[i] = S2[off + i];
    L[i] = Lq[didx[i]];
  }
  __syncthreads();
  auto mm = [&](const double2 *A, const double2 *Bm, int i, int j) {
    double re = 0.0, im = 0.0;
    for (int k = 0; k < B; ++k) {
      const double2 a = A[i * B + k], b = Bm[k * B + j];
      re = fma(a.x, b.x, fma(-a.y, b.y, re));
      im = fma(a.x, b.y, fma(a.y, b.x, im));
    }
    return make_double2(re, im);
  };
  // ch 0: T1 = L X2, T2 = L X1;  ch 1: T1 = L X1 (U1), T2 = L X2 (U2)
  for (int e = tid; e < BB; e += blockDim.x) {
    const int i = e / B, j = e - (e / B) * B;
    T1[e] = mm(L, ch == 0 ? X2 : X1, i, j);
    T2[e] = mm(L, ch == 0 ? X1 : X2, i, j);
  }
  __syncthreads();
  for (int e = tid; e < BB; e += blockDim.x) {
    const int i = e / B, j = e - (e / B) * B;
    if (ch == 0) {
      const double2 u = mm(X1, T1, i, j), v = mm(X2, T2, i, j);
      dp[off + e] = make_double2(-f * (u.x + v.x), -f * (u.y + v.y));
    } else {
      const double2 a = mm(X1, T1, i, j), b = mm(X1, T2, i, j), c2 = mm(X2, T1, i, j), g = mm(X2, T2, i, j);
      dc[off + e] = make_double2(2.0 * f * (2.0 * a.x - b.x - c2.x), 2.0 * f * (2.0 * a.y - b.y - c2.y));
      dd[off + e] = make_double2(-2.0 * f * g.x, -2.0 * f * g.y);
    }
  }
}

hipError_t launch_su2_bundle(int B, int Nq, int nD, const int *didx, const double *Lc, const double *Va,
                             const double *Vax, const double *Vc, const double *Vd, double f, double *dp, double *dc,
                             double *dd, hipStream_t st) {
  if (B < 1 || B > 25) return hipErrorInvalidValue;
  const size_t lds = 5 * (size_t)B * B * sizeof(double2);
  hipLaunchKernelGGL(su2_bundle_kernel, dim3((unsigned)Nq, 2), dim3(256), lds, st, B, Nq, nD, didx,
                     (const double2 *)Lc, (const double2 *)Va, (const double2 *)Vax, (const double2 *)Vc,
                     (const double2 *)Vd, f, (double2 *)dp, (double2 *)dc, (double2 *)dd);
  return hipGetLastError();
}

}  // namespace tufrg
