// Symmetries of the loop sums that every loop kernel uses.
//
// The sum over k of an item (channel ch, coarse q) is
//   Lc(q)[dR][(a,b,c,d)] = 1/Nf sum_k e^{-ik.dR} sum_mn Pi_m(k)_ac X_n(k')_bd L_mn,
// X_n = Pi_n(q - k) (pp) or Pi_n(k - q)^T (ph), L symmetric in its two energies.
// Relabelling k gives, for every model:
//   pp, k -> q - k:  the term of q - k is e^{-iq.dR} conj(term of k [dR][(d,c,b,a)]);
//   ph, k -> k + q:  Lc(-q)[dR][(a,b,c,d)] = e^{iq.dR} Lc(q)[dR][(d,c,b,a)].
// With time reversal, Pi_m(-k) = T Pi_m(k)^* T^t and e_m(-k) = e_m(k), T real
// with one entry t_a = +-1 per row a (column a'):
//   both channels, k -> -k: Lc(-q)[dR][(a,b,c,d)] = tttt conj(Lc(q)[dR][(a',b',c',d')]);
//   ph, k -> q - k: the term of q - k is e^{-iq.dR} tttt conj(term of k [dR][(d',c',b',a')]).
// trs = 0: no time reversal; 1: T = 1 (a' = a); 2: a' = a ^ 1, t_a = (-1)^a
// (T = i sigma_y in each orbital, the spin index fastest).
//
// Rows.  With one of each pair (k, q - k) the kx rows run from ceil(qx / 2) to
// floor((qx + Lf) / 2) (mod Lf); a row that is its own partner counts half.
#pragma once

#include <hip/hip_runtime.h>

namespace tufrg {

constexpr int LOOP_ITEM_Q = 0x3fffffff, LOOP_ITEM_CH = 30;

struct LoopSym {
  int trs, half, Lq;
  const double2 *twq;  // exp(+2 pi i j / Lq)
};

// largest number of kx rows of an item
__host__ __device__ inline int loop_rows_max(int Lf, int half) { return half ? Lf / 2 + 1 : Lf; }

// kx rows r0 .. r0 + n - 1 (mod Lf) of an item, and its rows of weight 1/2 (-1: none)
__host__ __device__ inline void loop_rows(int Lf, int qfx, int half, int &r0, int &n, int &h0, int &h1) {
  r0 = 0;
  n = Lf;
  h0 = h1 = -1;
  if (!half) return;
  r0 = (qfx + 1) / 2;
  const int r1 = (qfx + Lf) / 2;
  n = r1 - r0 + 1;
  if (!(qfx & 1)) h0 = r0;
  if (!((qfx + Lf) & 1)) h1 = r1 >= Lf ? r1 - Lf : r1;
}

// twice the weight of row kx in the halved sum: 2, 1 or 0
__host__ __device__ inline int loop_row_weight2(int Lf, int qfx, int kx) {
  int r = 2 * kx - qfx;
  r += r < 0 ? 2 * Lf : 0;
  return (r == 0 || r == Lf) ? 1 : (r < Lf ? 2 : 0);
}

// entry (a, b, c, d) with its indices reversed (rev) and/or replaced by their
// time-reversal partners (bar, with the sign t_a t_b t_c t_d)
__device__ inline int loop_tau(int n_o, int tau, bool rev, bool bar, double &sgn) {
  int d = tau % n_o, c = (tau / n_o) % n_o, b = (tau / (n_o * n_o)) % n_o, a = tau / (n_o * n_o * n_o);
  sgn = 1.0;
  if (bar) {
    sgn = ((a + b + c + d) & 1) ? -1.0 : 1.0;
    a ^= 1;
    b ^= 1;
    c ^= 1;
    d ^= 1;
  }
  return rev ? ((d * n_o + c) * n_o + b) * n_o + a : ((a * n_o + b) * n_o + c) * n_o + d;
}

// the entry of the halved sum whose conjugate completes entry tau
__device__ inline int loop_partner_tau(const LoopSym &s, int n_o, int ch, int tau, double &sgn) {
  return loop_tau(n_o, tau, true, ch == 1 && s.trs == 2, sgn);
}

// e^{iq.dR}
__device__ inline double2 loop_phase(const LoopSym &s, int q, int dx, int dy) {
  int j = ((q / s.Lq) * dx + (q % s.Lq) * dy) % s.Lq;
  j += j < 0 ? s.Lq : 0;
  return s.twq[j];
}

// v += e^{-iq.dR} sgn conj(h)
__device__ inline void loop_add_partner(const LoopSym &s, int q, int dx, int dy, double sgn, double2 h, double2 &v) {
  const double2 p = loop_phase(s, q, dx, dy);
  const double hr = sgn * h.x, hi = sgn * h.y;
  // (p.x - i p.y) (hr - i hi)
  v.x += p.x * hr - p.y * hi;
  v.y -= p.x * hi + p.y * hr;
}

// entry t of the block of -q from the entries v of that of q (the maps of the
// entries are their own inverses, and the signs square to one)
__device__ inline double2 loop_mirror(const LoopSym &s, int n_o, int q, int dx, int dy, int t, const double2 *v) {
  double sgn;
  if (s.trs) {
    const double2 x = v[loop_tau(n_o, t, false, s.trs == 2, sgn)];
    return make_double2(sgn * x.x, -sgn * x.y);
  }
  const double2 x = v[loop_tau(n_o, t, true, false, sgn)], p = loop_phase(s, q, dx, dy);
  return make_double2(p.x * x.x - p.y * x.y, p.x * x.y + p.y * x.x);
}

// stores entry tau of the item's block (at element off of the blocks of blk
// elements) to the slot of q, and transformed to the slot of -q
__device__ inline void loop_store(const LoopSym &s, int n_o, int ch, int q, int dx, int dy, int tau, double2 v,
                                  int2 dst, int chrel, int n_q_out, size_t blk, size_t off,
                                  double2 *__restrict__ out) {
  if (dst.x >= 0) out[((size_t)chrel * n_q_out + dst.x) * blk + off + tau] = v;
  if (dst.y >= 0) {
    double sgn;
    double2 m;
    int t;
    if (s.trs) {
      // a' of a' is a and the signs square to one: entry tau of q gives entry tau' of -q
      t = loop_tau(n_o, tau, false, s.trs == 2, sgn);
      m = make_double2(sgn * v.x, -sgn * v.y);
    } else {
      t = loop_tau(n_o, tau, true, false, sgn);
      const double2 p = loop_phase(s, q, dx, dy);
      m = make_double2(p.x * v.x - p.y * v.y, p.x * v.y + p.y * v.x);
    }
    out[((size_t)chrel * n_q_out + dst.y) * blk + off + t] = m;
  }
}

}  // namespace tufrg
