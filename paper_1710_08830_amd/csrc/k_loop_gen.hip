// Form-factor projected orbital loops for NO > 2 spin-orbitals (hot path of
// multi-orbital models such as t2g with spin-orbit coupling).
//
// Same quantity as the two-orbital kernel (see k_loop.hip):
//   Lc(q)[dR][(a,b,c,d)] = 1/Nf sum_k e^{-ik.dR} M_q(k)[a,b,c,d],
//   M_q(k)[a,b,c,d] = sum_m Pi_m(k)_ac W_m(k)_bd,  W_m = sum_n L_mn X_n,
// with X_n = Pi_n(k') (pp, k' = q - k) or its transpose (ph, k' = k - q).
//
// Entry pairs.  Pi_m and W_m are Hermitian, so M[(c,d,a,b)] = conj M[(a,b,c,d)]
// and Lc[dR][(c,d,a,b)] = conj Lc[-dR][(a,b,c,d)].  A thread owns one pair of
// such entries (or a self-conjugate entry), listed by the host: it forms M for
// the first entry at every k and keeps its loop for every dR of the
// difference set D of the form factors; the partner follows at the end.
//
// Separable phases.  Over one kx row the thread accumulates S = sum M and, for
// dy = 1..NDY, A = sum cos(theta) M and B = sum -sin(theta) M with
// theta = 2 pi ky dy / Lf (table phy[ky][dy - 1], read by scalar loads), so that the row transform at +dy is A + iB and at
// -dy is A - iB.  At the end of the row Lc[(dx, dy)] += e^{-i kx dx} Y(dy) for
// every (dx, dy) in D.
//
// Staging.  Tiles of KT consecutive ky go through LDS in packed Hermitian form:
// the projectors Pi_m(k) and X_n(k'), the loop kernels L_mn and then W_m(k).  The
// inner loop reads the two reals of an entry per band and sums the four real
// products; the signs (conjugate entries, real diagonals) enter once per point.
// The steps of a tile run in four stages of a pipeline with one barrier per tile,
// the values from memory one tile ahead in registers: waiting for each tile's
// loads and at four barriers the kernel took 1.73 ms (t2g, 13 form factors, FP64,
// L 10 refined 6) and 1.45 ms (Zeeman, 9, FP32, L 11 refined 5), now 0.98 and
// 0.74 ms (the first 0.76 since its pairs around zero energy, Omega scheme, take the
// quotient): FP32 is then bound by vector issue and LDS reads, FP64 (13 form factors:
// 41 complex sums a thread, six waves a CU) by the latency of the stages.
//
// Kramers pairs (PAIR): when bands (0,1), (2,3), (4,5) are degenerate at every
// k, L_mn depends on the pairs only and the band sums group exactly into three
// bands with the pair sums of the projectors (energies and regulator values
// of the first band of each pair).
#include "common.h"
#include "kernels.h"
#include "loop_sym.h"

namespace tufrg {

namespace {

// points (dx, dy) of the difference set: the 9-vector shell gives the 5 x 5
// box (R = 2), the 13-vector shell the diamond |dx| + |dy| <= 4 (R = 4)
template <int R>
struct Shape;
template <>
struct Shape<2> {
  static constexpr int N = 25;
  __device__ static constexpr int dx(int i) { return i / 5 - 2; }
  __device__ static constexpr int dy(int i) { return i % 5 - 2; }
};
template <>
struct Shape<4> {
  static constexpr int N = 41;
  __device__ static constexpr int row_len(int x) { return 2 * (4 - (x < 0 ? -x : x)) + 1; }
  __device__ static constexpr int row_start(int x) {
    int s = 0;
    for (int r = -4; r < x; ++r) s += row_len(r);
    return s;
  }
  __device__ static constexpr int dx(int i) {
    int x = -4;
    while (x < 4 && row_start(x + 1) <= i) ++x;
    return x;
  }
  __device__ static constexpr int dy(int i) { return i - row_start(dx(i)) - (row_len(dx(i)) - 1) / 2; }
};

// entry (r, c) of a packed Hermitian NO x NO matrix (NO diagonal reals, then Re
// and Im of (lo, hi) for lo < hi in row-major order): offset of its real part,
// sign of the imaginary part behind it (0: real)
template <int NO>
__device__ inline int packed_of(int r, int c, int &sign) {
  sign = r < c ? 1 : r > c ? -1 : 0;
  if (r == c) return r;
  const int lo = min(r, c), hi = max(r, c);
  return NO + 2 * (lo * (2 * NO - 1 - lo) / 2 + hi - lo - 1);
}

}  // namespace

// One workgroup per (part, item, kx chunk): part selects NTHR of the entry pairs,
// the item a channel and a coarse q; the kx rows of a halved sum as in loop_sym.h.
template <typename T, int NO, int NDY, int SCHEME, int NTHR, int KT, bool PAIR>
__global__ __launch_bounds__(NTHR) void loop_gen_kernel(const T *__restrict__ band, const T *__restrict__ pir,
                                                        const T *__restrict__ kv, const T *__restrict__ cvp,
                                                        const double *__restrict__ tw, const T *__restrict__ phy,
                                                        const int *__restrict__ pairs,
                                                        int n_pairs, int Lq, int n_ref, int Lf, int nparts, int kxper,
                                                        int nkxc, int half, const int *__restrict__ items, int n_pp,
                                                        int n_ph, int ndx_out,
                                                        T lam, int deriv, T *__restrict__ partial) {
  using SH = Shape<NDY>;
  constexpr int NPT = SH::N;
  constexpr int NO2 = NO * NO, NO4 = NO2 * NO2;
  constexpr int NB = PAIR ? NO / 2 : NO;  // bands summed (pairs)
  constexpr int PK = NB * NO2;      // packed reals of the summed bands' projectors at one k
  constexpr int NC = NO + NO * NO2; // band values per k-point: e_m, then the packed projectors
  constexpr bool SHELL = SCHEME == CUT_SHELL;
  // band m of the sums in the arrays of all bands (paired: the first of the pair)
  constexpr int MS = PAIR ? 2 : 1;
  const int tid = threadIdx.x;
  int w = blockIdx.x;
  const int part = w % nparts;
  w /= nparts;
  // kx chunk: the pp items' chunks come first, then the ph items'
  const int w_pp = n_pp * ((loop_rows_max(Lf, half & 1) + kxper - 1) / kxper), ch = w >= w_pp ? 1 : 0;
  w -= ch ? w_pp : 0;
  const int n_it = ch ? n_ph : n_pp, kxc = w / n_it, it = (ch ? n_pp : 0) + w % n_it;
  const int qi = items[it] & LOOP_ITEM_Q;
  const int qfx = (qi / Lq) * n_ref, qfy = (qi % Lq) * n_ref;
  const int pidx = part * NTHR + tid;
  const bool active = pidx < n_pairs;
  const int tau = active ? pairs[2 * pidx] : 0, taub = active ? pairs[2 * pidx + 1] : 0;
  // Pi_m at (a, c), W_m at (b, d); ph takes the transpose of Pi_n(k')
  int sgx, sgy;
  const int xo = packed_of<NO>(tau / (NO * NO2), (tau / NO) % NO, sgx);
  const int yo = packed_of<NO>((tau / NO2) % NO, tau % NO, sgy);
  const T sx = T(sgx), sy = T(ch == 0 ? sgy : -sgy), sxy = sx * sy;

  constexpr int PU = PK / 2;                       // pairs of reals of a point's projectors
  constexpr int EKV = 2 * NB + (SHELL ? 2 * NB : 0);  // e, K (a, b of the shell) of a point
  constexpr int NSL = (KT * PU + NTHR - 1) / NTHR, NSE = (KT * 2 * EKV + NTHR - 1) / NTHR;
  typedef T T2 __attribute__((ext_vector_type(2)));
  __shared__ T2 sP[2][KT][PU];  // Pi_m(k) packed
  __shared__ T2 sX[2][KT][PU];  // X_n(k') packed
  __shared__ T2 sW[2][KT][PU];  // W_m(k) packed
  __shared__ T sE[2][KT][2][EKV];
  __shared__ T sL[2][KT][NB][NB];
  const T sg = (ch == 0) ? T(1) : T(-1);

  cx<T> Z[NPT];
#pragma unroll
  for (int i = 0; i < NPT; ++i) Z[i] = cmake(T(0), T(0));

  int r0, nr, hx0, hx1;
  loop_rows(Lf, qfx, (half >> ch) & 1, r0, nr, hx0, hx1);
  nr = min(nr, (kxc + 1) * kxper) - kxc * kxper;
  r0 += kxc * kxper;
  const int ntk = (Lf + KT - 1) / KT, ntile = nr * ntk;
  const unsigned magic = 0xffffffffu / (unsigned)ntk + 1u;  // t / ntk, exact for t < 2^32 / ntk
  struct Pos {
    int kx, kpx, ky0;
  };
  auto pos = [&](int t) __attribute__((always_inline)) {
    t = min(t, ntile - 1);
    const int r = ntk == 1 ? t : (int)__umulhi((unsigned)t, magic);
    Pos p;
    p.kx = r0 + r >= Lf ? r0 + r - Lf : r0 + r;
    p.kpx = ch == 0 ? qfx - p.kx : p.kx - qfx;
    p.kpx += p.kpx < 0 ? Lf : 0;
    p.ky0 = (t - r * ntk) * KT;
    return p;
  };
  auto column = [&](int side, int ky) __attribute__((always_inline)) {
    ky = min(ky, Lf - 1);
    int kp = ch == 0 ? qfy - ky : ky - qfy;
    kp += kp < 0 ? Lf : 0;
    return side ? kp : ky;
  };
  // a tile's values on their way from memory, in registers
  T2 rp[NSL], rx[NSL];
  T re[NSE];
  auto load_pi = [&](int t, int side, T2 (&v)[NSL]) __attribute__((always_inline)) {
    const Pos p = pos(t);
#pragma unroll
    for (int u = 0; u < NSL; ++u) {
      const int i = min(tid + NTHR * u, KT * PU - 1), j = i / PU, o = i - j * PU;
      const size_t k = (size_t)(side ? p.kpx : p.kx) * Lf + column(side, p.ky0 + j);
      v[u] = ((const T2 *)(PAIR ? pir + k * PK : band + k * NC + NO))[o];
    }
  };
  auto store_pi = [&](T2 (*dst)[PU], const T2 (&v)[NSL]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NSL; ++u) {
      const int i = tid + NTHR * u;
      if (i < KT * PU) (&dst[0][0])[i] = v[u];
    }
  };
  auto load_e = [&](int t) __attribute__((always_inline)) {
    const Pos p = pos(t);
#pragma unroll
    for (int u = 0; u < NSE; ++u) {
      const int i = min(tid + NTHR * u, KT * 2 * EKV - 1), j = i / (2 * EKV), v = i - j * 2 * EKV;
      const int side = v / EKV, r = v - side * EKV;
      const size_t k = (size_t)(side ? p.kpx : p.kx) * Lf + column(side, p.ky0 + j);
      const T *src = r < NB ? band + k * NC + MS * r : kv + k * NO + MS * (r - NB);
      if (SHELL && r >= 2 * NB) {
        const int c = r - 2 * NB;  // (a_m, b_m) of summed band c / 2
        src = cvp + k * 2 * NO + 2 * MS * (c >> 1) + (c & 1);
      }
      re[u] = *src;
    }
  };
  auto store_e = [&](int bf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NSE; ++u) {
      const int i = tid + NTHR * u;
      if (i < KT * 2 * EKV) (&sE[bf][0][0][0])[i] = re[u];
    }
  };
  // loop kernels L_mn = sg * DD[K](e_m(k), -sg e_n(k')), the row's weight included
  auto loop_kernels = [&](int t, int bf) __attribute__((always_inline)) {
    // from wave 2 on: of six waves, 2 and 3 have a SIMD of their own
    for (int i = tid >= 128 ? tid - 128 : tid + NTHR - 128; i < KT * NB * NB; i += NTHR) {
      const int j = i / (NB * NB), m = (i / NB) % NB, n = i % NB, kx = pos(t).kx;
      const T(&e0)[EKV] = sE[bf][j][0], (&e1)[EKV] = sE[bf][j][1];
      T l = (kx == hx0 || kx == hx1 ? T(0.5) * sg : sg) *
            divided_difference(e0[m], -sg * e1[n], e0[NB + m], -sg * e1[NB + n], lam, dd_scheme(SCHEME), deriv);
      // shell scheme: times a_m(k) b_n(k') + b_m(k) a_n(k')
      if constexpr (SHELL)
        l *= fma(e0[2 * NB + 2 * m], e1[2 * NB + 2 * n + 1], e0[2 * NB + 2 * m + 1] * e1[2 * NB + 2 * n]);
      sL[bf][j][m][n] = l;
    }
  };
  // W_m = sum_n L_mn X_n
  auto weights = [&](int bf) __attribute__((always_inline)) {
    for (int i = tid; i < KT * PU; i += NTHR) {
      const int j = i / PU, mp = i - j * PU, m = mp / (NO2 / 2), o = mp - m * (NO2 / 2);
      T2 acc = T2{T(0), T(0)};
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const T l = sL[bf][j][m][n];
        const T2 x = sX[bf][j][n * (NO2 / 2) + o];
        acc[0] = fma(l, x[0], acc[0]);
        acc[1] = fma(l, x[1], acc[1]);
      }
      sW[bf][j][mp] = acc;
    }
  };
  cx<T> S = cmake(T(0), T(0)), A[NDY], B[NDY];
#pragma unroll
  for (int j = 0; j < NDY; ++j) A[j] = B[j] = cmake(T(0), T(0));
  if (ntile > 0) load_e(0);  // none: a last chunk past the rows of this item
  // one barrier per tile: products of tile t, W of t + 1, loop kernels of t + 2;
  // the values of t + 1 (Pi), t + 2 (X), t + 3 (e, K) from registers into LDS, the
  // next ones on their way meanwhile
  for (int t = ntile > 0 ? -3 : ntile; t < ntile; ++t) {
    store_e((t + 3) & 1);
    if (t >= -2) store_pi(sX[t & 1], rx);
    if (t >= -1) store_pi(sP[(t + 1) & 1], rp);
    load_e(t + 4);
    load_pi(t + 3, 1, rx);
    load_pi(max(t + 2, 0), 0, rp);
    if (t >= -2 && t + 2 < ntile) loop_kernels(t + 2, t & 1);
    if (t >= -1 && t + 1 < ntile) weights((t + 1) & 1);
    if (t >= 0) {
      const Pos p = pos(t);
      const int kt = min(KT, Lf - p.ky0);
      const T *P = (const T *)sP[t & 1] + xo, *W = (const T *)sW[t & 1] + yo;
#pragma unroll 2
      for (int j = 0; j < kt; ++j, P += PK, W += PK) {
        // the same for every lane: scalar loads (through LDS: 1.00 -> 1.20 ms)
        const T *ph = phy + (size_t)(p.ky0 + j) * (2 * NDY);
        T rr = T(0), ii = T(0), ri = T(0), ir = T(0);
#pragma unroll
        for (int m = 0; m < NB; ++m) {
          const T pr = P[m * NO2], pi = P[m * NO2 + 1], wr = W[m * NO2], wi = W[m * NO2 + 1];
          rr = fma(pr, wr, rr);
          ii = fma(pi, wi, ii);
          ri = fma(pr, wi, ri);
          ir = fma(pi, wr, ir);
        }
        const cx<T> M = cmake(fma(-sxy, ii, rr), fma(sy, ri, sx * ir));
        S.re += M.re;
        S.im += M.im;
#pragma unroll
        for (int dy = 0; dy < NDY; ++dy) {
          const T cs = ph[2 * dy], sn = ph[2 * dy + 1];
          A[dy].re = fma(cs, M.re, A[dy].re);
          A[dy].im = fma(cs, M.im, A[dy].im);
          B[dy].re = fma(sn, M.re, B[dy].re);
          B[dy].im = fma(sn, M.im, B[dy].im);
        }
      }
      if (p.ky0 + KT >= Lf) {
        // row transform at +dy: A + iB, at -dy: A - iB; then the kx phase,
        // one |dx| at a time
#pragma unroll
        for (int adx = 0; adx <= NDY; ++adx) {
          const int jj = (p.kx * adx) % Lf;
          const cx<T> f = cmake((T)tw[2 * jj], (T)tw[2 * jj + 1]);
#pragma unroll
          for (int i = 0; i < NPT; ++i) {
            const int dx = SH::dx(i), dy = SH::dy(i);
            if ((dx < 0 ? -dx : dx) != adx) continue;
            cx<T> Yv;
            if (dy == 0) {
              Yv = S;
            } else {
              const cx<T> Av = A[(dy > 0 ? dy : -dy) - 1], Bv = B[(dy > 0 ? dy : -dy) - 1];
              Yv = dy > 0 ? cmake(Av.re - Bv.im, Av.im + Bv.re) : cmake(Av.re + Bv.im, Av.im - Bv.re);
            }
            cfma(Z[i], dx < 0 ? cmake(f.re, -f.im) : f, Yv);
          }
        }
        S = cmake(T(0), T(0));
#pragma unroll
        for (int j = 0; j < NDY; ++j) A[j] = B[j] = cmake(T(0), T(0));
      }
    }
    __syncthreads();
  }
  if (!active) return;
  // partial[item][kx chunk][dx][dy + NDY][tau] for dx >= 0; the partner entry from
  // Lc[dR][partner] = conj Lc[-dR][tau]
  const int ndy2 = 2 * NDY + 1;
  const size_t pbase = ((size_t)it * nkxc + kxc) * (size_t)(ndx_out * ndy2 * NO4);
#pragma unroll
  for (int i = 0; i < NPT; ++i) {
    const int dx = SH::dx(i), dy = SH::dy(i);
    if (dx >= 0) {
      const size_t idx = pbase + (size_t)(dx * ndy2 + dy + NDY) * NO4 + tau;
      partial[2 * idx] = Z[i].re;
      partial[2 * idx + 1] = Z[i].im;
    }
    if (dx <= 0 && taub != tau) {
      const size_t idx = pbase + (size_t)(-dx * ndy2 - dy + NDY) * NO4 + taub;
      partial[2 * idx] = Z[i].re;
      partial[2 * idx + 1] = -Z[i].im;
    }
  }
}

template <typename T, int NDY>
static hipError_t launch_gen(const LoopArgs &a, hipStream_t st) {
  // FP32: every pair of a (q, channel) in one workgroup of 11 waves (three
  // per SIMD); FP64 needs twice the registers: workgroups of 6 waves
  constexpr bool f64 = sizeof(T) == 8;
  constexpr int NTHR = f64 ? 384 : 704, KT = f64 ? 8 : 16;
  if (a.ndx != NDY + 1) return hipErrorInvalidValue;
  const int NP = (a.n_pairs + NTHR - 1) / NTHR;
  if (!a.items || a.n_pp + a.n_ph < 1 || a.nkyb != 1) return hipErrorInvalidValue;
  auto work = [&](int n, int h) { return (long long)n * ((loop_rows_max(a.Lf, h) + a.kxper - 1) / a.kxper); };
  const long long nw = NP * (work(a.n_pp, a.half & 1) + work(a.n_ph, (a.half >> 1) & 1));
  if (nw > 0x7fffffffLL) return hipErrorInvalidValue;
  dim3 grid((unsigned)nw), block(NTHR);
  const T *band = (const T *)a.band, *kv = (const T *)a.kv, *phy = (const T *)a.phy, *cvp = (const T *)a.cv;
  const T *pir = f64 ? (const T *)a.pir64 : (const T *)a.pir;
  if (a.scheme == CUT_SHELL && !cvp) return hipErrorInvalidValue;
  if (a.pair && !pir) return hipErrorInvalidValue;
#define TUFRG_GEN_LAUNCH(S, P)                                                                                   \
  hipLaunchKernelGGL((loop_gen_kernel<T, 6, NDY, S, NTHR, KT, P>), grid, block, 0, st, band, pir, kv, cvp, a.tw, \
                     phy, a.pairs, a.n_pairs, a.Lq, a.n_ref, a.Lf, NP, a.kxper, a.nparts, a.half, a.items, a.n_pp, \
                     a.n_ph, a.ndx, (T)a.lam, a.deriv, (T *)a.partial)
#define TUFRG_GEN_SCHEMES(P)               \
  if (a.scheme == CUT_TEMPERATURE)         \
    TUFRG_GEN_LAUNCH(CUT_TEMPERATURE, P);  \
  else if (a.scheme == CUT_OMEGA)          \
    TUFRG_GEN_LAUNCH(CUT_OMEGA, P);        \
  else if (a.scheme == CUT_SHELL)          \
    TUFRG_GEN_LAUNCH(CUT_SHELL, P);        \
  else                                     \
    return hipErrorInvalidValue;
  if (a.pair) {
    TUFRG_GEN_SCHEMES(true)
  } else {
    TUFRG_GEN_SCHEMES(false)
  }
#undef TUFRG_GEN_SCHEMES
#undef TUFRG_GEN_LAUNCH
  return hipGetLastError();
}

hipError_t launch_loop_gen(const LoopArgs &a, hipStream_t st) {
  if (a.n_o != 6 || !a.pairs || a.n_pairs <= 0) return hipErrorInvalidValue;
  const bool f64 = (a.prec == 0);
  if (a.ndx == 5 && a.ndy == 4) return f64 ? launch_gen<double, 4>(a, st) : launch_gen<float, 4>(a, st);
  if (a.ndx == 3 && a.ndy == 2) return f64 ? launch_gen<double, 2>(a, st) : launch_gen<float, 2>(a, st);
  return hipErrorInvalidValue;
}

}  // namespace tufrg
