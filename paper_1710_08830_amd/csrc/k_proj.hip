// Truncated-unity cross projections (hot path, HBM-bound).
//
// Matrix layouts (B = n_ff n_o^2, flat index r n_o^2 + a n_o + b):
//   P[q][(R,a,b),(R',c,d)] = P^{RR'}_{a b d c}(q),  C[q][(R,a,b),(R',c,d)] = C^{RR'}_{a d b c}(q).
// The projections of the paper's Sec. 3.3 read, in these layouts and with
// X(rho) = 1/Nq sum_q e^{i q.rho} X(q):
//   P[V^C](s)[(R,a,b),(R',c,d)] =  sum_rho e^{is.rho} C(rho)[(R+rho,a,d),(R'-rho,c,b)]
//   P[V^D](s)[(R,a,b),(R',c,d)] = -sum_rho e^{is.rho} C(rho-R')[(R+rho-R',a,c),(-rho,d,b)]
//   C[V^P](u)[(R,a,b),(R',c,d)] =  sum_rho e^{iu.rho} P(rho)[(R+rho,a,d),(R'-rho,c,b)]
//   C[V^D](u)[(R,a,b),(R',c,d)] = -sum_rho e^{iu.rho} C(-R')[(R-R'+rho,a,c),(rho,b,d)]
// (the P[V^D] line substitutes rho = R' + R'' in the paper's form, which carries
// an extra e^{is.R'}), every term whose form-factor labels leave S being dropped.
// So each projected vertex is X(q) + X[V0] + sum_rho e^{iq.rho} G_X(rho), with
// G_X gathered in rho-space:
//   ft_kernel        X(q) -> X(rho)              (HBM read of both states)
//   assemble_kernel  X(rho) -> G(rho) -> VP, VC  (HBM read of the states, write of V)
// On the q-mesh q = 2 pi (qx, qy) / Lq the phase factorises,
// e^{iq.rho} = e^{2 pi i qx rho_x / Lq} e^{2 pi i qy rho_y / Lq}, and rho_y takes
// at most nine values over D, 0 and pairs +-y (D = S - S):
//   ft:       M(qx, y) = sum_qy e^{2 pi i qy y / Lq} X(qx, qy);
//             X(rho) = 1/Nq sum_qx e^{2 pi i qx rho_x / Lq} M(qx, rho_y)
//   assemble: h(qx, y) = sum_{rho: rho_y = y} e^{2 pi i qx rho_x / Lq} G(rho);
//             VX(qx, qy) = X + X[V0] + sum_y e^{2 pi i qy y / Lq} h(qx, y)
// A pair +-y shares its products with the cosine and the sine.  Neither M nor h
// leaves the workgroup: it owns EW matrix elements e at all q, its 256 threads
// being EW elements times 256 / EW units (a qx row, or one of `parts` pieces of
// one).  In ft the units meet in LDS, where the threads of an element share out
// its rho; in assemble the G of the workgroup's elements lie in LDS and a thread
// forms the h of its own unit.  Eight loads per thread are in flight; ft has the
// next eight on their way across its barriers (2.4 -> 1.5 ms at the size below).
// Bound by HBM: t2g 32 x 32, 13 form factors (7.2 GB a state): ft 1.5 ms (4.8
// TB/s), assemble 2.9 ms (5.0 TB/s, the rate of a copy).  With M and h (2 GB
// each) and G in memory, in five launches, it was 7.4 ms.
// EW = 64 reads whole 1 KB lines per wave, with wave-uniform phases; fewer
// elements per workgroup give small states more workgroups (below).
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace tufrg {

namespace {

constexpr int NTHR = 256, NU = 8;  // threads; loads in flight
constexpr int NDS = 44;            // most rho of a small set (41 for form factors up to |R| = 2)

// rho sums per thread of sets up to NDS or 81
constexpr int rho_per_thread(int EW, int big) {
  return big ? (81 + NTHR / EW - 1) / (NTHR / EW) : (NDS + NTHR / EW - 1) / (NTHR / EW);
}

// Element block of this workgroup: each XCD walks a range of its own (the gathers
// of neighbouring elements share lines in its L2), in reverse for the assembly.
// nb is a multiple of eight.
__device__ inline int xcd_block(int nb, bool reverse = false) {
  const int per = nb >> 3, i = blockIdx.x >> 3;
  return (blockIdx.x & 7) * per + (reverse ? per - 1 - i : i);
}

// v mod Lq for v < Lq^2, Lq <= 4096, magic = ceil(2^32 / Lq): the quotient is at
// most one too large
__device__ inline int mod_lq(unsigned v, unsigned Lq, unsigned magic) {
  const int r = (int)(v - __umulhi(v, magic) * Lq);
  return r + (r < 0 ? (int)Lq : 0);
}

// cos and sin of the qy phases of a q: per wave from memory (EW = 64) or LDS
template <int NP>
struct Phases {
  double2 p[NP ? NP : 1];
  __device__ inline void read(const double2 *t, int qy) {
#pragma unroll
    for (int y = 0; y < NP; ++y) p[y] = t[qy * NP + y];
  }
};

// real[w][iD][e] = scale sum_q e^{iq.rho} X_w(q)[e]
template <int EW, int NP, int NJ>
__global__ __launch_bounds__(NTHR) void ft_kernel(int BB, int Lq, int nD, int parts, double scale,
                                                  const double2 *__restrict__ phy, const double2 *__restrict__ twq,
                                                  const int *__restrict__ dtab, const double2 *__restrict__ P,
                                                  const double2 *__restrict__ C, double2 *__restrict__ real) {
  constexpr int NG = NTHR / EW, NY = 2 * NP + 1;
  __shared__ double2 sM[NG * NY * EW];
  extern __shared__ double2 psm[];  // [Lq] qx phases, for EW < 64 [Lq][NP] qy phases
  const int tid = threadIdx.x, el = tid % EW;
  const int g = EW == 64 ? __builtin_amdgcn_readfirstlane(tid / 64) : tid / EW;
  const int blk = xcd_block(gridDim.x), nb = (BB + EW - 1) / EW;
  if (blk >= 2 * nb) return;
  const int w = blk / nb, e = (blk - w * nb) * EW + el;
  double2 *sY = psm + Lq;
  for (int i = tid; i < Lq; i += NTHR) psm[i] = twq[i];
  if (EW < 64)
    for (int i = tid; i < Lq * NP; i += NTHR) sY[i] = phy[i];
  const double2 *ph = EW < 64 ? sY : phy;
  // the thread's rho: g, g + NG, ... (past the list: the last again, not stored)
  int xv[NJ], ix[NJ], sl[NJ];
  double ar[NJ], ai[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int t = dtab[min(g + NG * j, nD - 1)];
    xv[j] = t & 0xffff;
    sl[j] = (t >> 16) * EW + el;
    ix[j] = 0;
    ar[j] = ai[j] = 0.0;
  }
  const int rows = NG / parts, rl = g / parts, pt = g % parts;
  const int q0 = pt * Lq / parts, q1 = (pt + 1) * Lq / parts;
  const double2 *X = (w == 0 ? P : C) + min(e, BB - 1);
  double2 xn[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) xn[u] = X[((size_t)min(rl, Lq - 1) * Lq + min(q0 + u, q1 - 1)) * BB];
  __syncthreads();
  for (int r0 = 0; r0 < Lq; r0 += rows) {
    if (r0 + rl < Lq) {
      const double2 *Xr = X + (size_t)(r0 + rl) * Lq * BB;
      double zr = 0.0, zi = 0.0, cr[NP + 1], ci[NP + 1], sr[NP + 1], si[NP + 1];
#pragma unroll
      for (int y = 0; y < NP; ++y) cr[y] = ci[y] = sr[y] = si[y] = 0.0;
      for (int q = q0; q < q1; q += NU) {
        double2 x[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) x[u] = xn[u];
        // the next loads, of the unit's next row after its last ones
        const bool last = q + NU >= q1;
        const int qn = last ? q0 : q + NU;
        const double2 *Xn = last ? X + (size_t)min(r0 + rows + rl, Lq - 1) * Lq * BB : Xr;
#pragma unroll
        for (int u = 0; u < NU; ++u) xn[u] = Xn[(size_t)min(qn + u, q1 - 1) * BB];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          if (u && q + u >= q1) break;
          Phases<NP> f;
          f.read(ph, q + u);
          zr += x[u].x;
          zi += x[u].y;
#pragma unroll
          for (int y = 0; y < NP; ++y) {
            cr[y] = fma(f.p[y].x, x[u].x, cr[y]);
            ci[y] = fma(f.p[y].x, x[u].y, ci[y]);
            sr[y] = fma(f.p[y].y, x[u].x, sr[y]);
            si[y] = fma(f.p[y].y, x[u].y, si[y]);
          }
        }
      }
      double2 *m = sM + g * NY * EW + el;
      m[0] = make_double2(zr, zi);
#pragma unroll
      for (int y = 0; y < NP; ++y) {
        m[(2 * y + 1) * EW] = make_double2(cr[y] - si[y], ci[y] + sr[y]);
        m[(2 * y + 2) * EW] = make_double2(cr[y] + si[y], ci[y] - sr[y]);
      }
    }
    __syncthreads();
    const int nr = min(rows, Lq - r0);
    for (int r = 0; r < nr; ++r) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const double2 *m = sM + r * parts * NY * EW + sl[j];
        double2 v = m[0];
        for (int p = 1; p < parts; ++p) {
          const double2 o = m[p * NY * EW];
          v.x += o.x;
          v.y += o.y;
        }
        const double2 t = psm[ix[j]];
        ar[j] = fma(t.x, v.x, fma(-t.y, v.y, ar[j]));
        ai[j] = fma(t.x, v.y, fma(t.y, v.x, ai[j]));
        ix[j] += xv[j];
        ix[j] -= ix[j] >= Lq ? Lq : 0;
      }
    }
    __syncthreads();
  }
  if (e >= BB) return;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int iD = g + NG * j;
    if (iD < nD) real[((size_t)w * nD + iD) * BB + e] = make_double2(ar[j] * scale, ai[j] * scale);
  }
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// two floats to packed BF16 pairs (round to nearest even): hi and the BF16 of the remainders
__device__ inline void split2(float a, float b, unsigned &hi, unsigned &lo) {
  hi = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, bf16x2));
  const float ra = a - __uint_as_float(hi << 16), rb = b - __uint_as_float(hi & 0xffff0000u);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){ra, rb}, bf16x2));
}

struct GatherTables {
  int n_o, n_ff, B, nD;
  const int *ff, *dlist, *ffgrid, *dgrid;
};
constexpr int GRID = 17 * 17;

// G[w][iD][e]: w = 0 feeds VP (from C), w = 1 feeds VC (from P and C); grid the
// form-factor and D indices of (x, y) in [-8, 8]^2, one after the other
__device__ inline double2 gather_one(const GatherTables &t, const int *grid, int w, int iD, int row, int col,
                                     const double2 *__restrict__ real) {
  const int no2 = t.n_o * t.n_o, B = t.B;
  const long long BB = (long long)B * B;
  const int r = row / no2, a = (row % no2) / t.n_o, b = row % t.n_o;
  const int rp = col / no2, c = (col % no2) / t.n_o, d = col % t.n_o;
  const int Rx = t.ff[2 * r], Ry = t.ff[2 * r + 1], Rpx = t.ff[2 * rp], Rpy = t.ff[2 * rp + 1];
  const int px = t.dlist[2 * iD], py = t.dlist[2 * iD + 1];
  auto idx = [&](const int *g, int x, int y) {
    const bool in = x >= -8 && x <= 8 && y >= -8 && y <= 8;
    const int v = g[in ? (x + 8) * 17 + (y + 8) : 0];
    return in ? v : -1;
  };
  const double2 *Pr = real, *Cr = real + (size_t)t.nD * BB;
  const int A = idx(grid, Rx + px, Ry + py), Bi = idx(grid, Rpx - px, Rpy - py);
  int A2, B2, D2, r2, c2;
  if (w == 0) {
    A2 = idx(grid, Rx + px - Rpx, Ry + py - Rpy), B2 = idx(grid, -px, -py);
    D2 = idx(grid + GRID, px - Rpx, py - Rpy);
    r2 = A2 * no2 + a * t.n_o + c, c2 = B2 * no2 + d * t.n_o + b;
  } else {
    A2 = idx(grid, Rx - Rpx + px, Ry - Rpy + py), B2 = idx(grid, px, py);
    D2 = idx(grid + GRID, -Rpx, -Rpy);
    r2 = A2 * no2 + a * t.n_o + c, c2 = B2 * no2 + b * t.n_o + d;
  }
  // both loads always, from element 0 where the term is dropped
  const bool in1 = A >= 0 && Bi >= 0, in2 = A2 >= 0 && B2 >= 0 && D2 >= 0;
  const int r1 = A * no2 + a * t.n_o + d, c1 = Bi * no2 + c * t.n_o + b;
  const double2 v1 = (w == 0 ? Cr : Pr)[in1 ? iD * BB + (long long)r1 * B + c1 : 0];
  const double2 v2 = Cr[in2 ? D2 * BB + (long long)r2 * B + c2 : 0];
  return make_double2((in1 ? v1.x : 0.0) - (in2 ? v2.x : 0.0), (in1 ? v1.y : 0.0) - (in2 ? v2.y : 0.0));
}

// VX(qx, qy)[e] = X[e] + X[V0][e] + sum_rho e^{iq.rho} G_X(rho)[e]; G gathered
// from X(rho) or given (SRC 2); V in FP64, or in the form of the bundle products
// that read it: SRC 1 split planes of BF16, SRC 3 FP32.  The element blocks run in reverse: the
// last ones that ft read are still in the last-level cache.
template <int EW, int NP, int SRC>
__global__ __launch_bounds__(NTHR) void assemble_kernel(int BB, int Lq, int nD, int nw, int parts,
                                                        unsigned magic, GatherTables gt, const double2 *__restrict__ phy,
                                                        const double2 *__restrict__ twq,
                                                        const int *__restrict__ dslot,
                                                        const double2 *__restrict__ src,
                                                        const double2 *__restrict__ P, const double2 *__restrict__ C,
                                                        const double2 *__restrict__ v0p,
                                                        const double2 *__restrict__ v0c, void *__restrict__ VP,
                                                        void *__restrict__ VC) {
  constexpr bool GATHER = SRC != 2;
  constexpr int NG = NTHR / EW, NY = 2 * NP + 1;
  extern __shared__ double2 psm[];  // [nD][EW] G, [Lq] qx phases, for EW < 64 [Lq][NP] qy phases
  __shared__ int grid[GATHER ? 2 * GRID : 1];
  const int tid = threadIdx.x, el = tid % EW;
  const int g = EW == 64 ? __builtin_amdgcn_readfirstlane(tid / 64) : tid / EW;
  const int blk = xcd_block(gridDim.x, true), nb = (BB + EW - 1) / EW;
  if (blk >= nw * nb) return;
  const int w = blk / nb, e = (blk - w * nb) * EW + el;
  const int ec = min(e, BB - 1);
  double2 *sG = psm, *sX = psm + nD * EW, *sY = sX + Lq;
  for (int i = tid; i < Lq; i += NTHR) sX[i] = twq[i];
  if (EW < 64)
    for (int i = tid; i < Lq * NP; i += NTHR) sY[i] = phy[i];
  const double2 *ph = EW < 64 ? sY : phy;
  if constexpr (GATHER) {
    for (int i = tid; i < GRID; i += NTHR) {
      grid[i] = gt.ffgrid[i];
      grid[GRID + i] = gt.dgrid[i];
    }
    __syncthreads();
    const int row = ec / gt.B, col = ec % gt.B;
#pragma unroll 4
    for (int i = g; i < nD; i += NG) sG[i * EW + el] = gather_one(gt, grid, w, i, row, col, src);
  } else {
    for (int i = g; i < nD; i += NG) sG[i * EW + el] = src[((size_t)w * nD + i) * BB + ec];
  }
  __syncthreads();
  const double2 v0 = (w == 0 ? v0p : v0c)[ec];
  const double2 *X = (w == 0 ? P : C) + ec;
  double2 *V = (double2 *)(w == 0 ? VP : VC) + ec;
  float2 *F = (float2 *)(w == 0 ? VP : VC) + ec;
  unsigned short *S = (unsigned short *)(w == 0 ? VP : VC) + (ec & ~3) + (size_t)(el & 3) * BB;  // BB a multiple of four
  const bool valid = e < BB;
  for (int unit = g; unit < Lq * parts; unit += NG) {
    const int row = unit / parts, pt = unit % parts;
    const int q0 = pt * Lq / parts, q1 = (pt + 1) * Lq / parts;
    double hr[NY], hi[NY];
#pragma unroll
    for (int y = 0; y < NY; ++y) {
      hr[y] = hi[y] = 0.0;
      for (int j = 0; j < 9; ++j) {
        const int t = dslot[9 * y + j];
        if (t < 0) break;
        const double2 v = sG[(t & 0xffff) * EW + el], f = sX[mod_lq((unsigned)row * (unsigned)(t >> 16), Lq, magic)];
        hr[y] = fma(f.x, v.x, fma(-f.y, v.y, hr[y]));
        hi[y] = fma(f.x, v.y, fma(f.y, v.x, hi[y]));
      }
    }
    // c (h+ + h-) + i s (h+ - h-)
    hr[0] += v0.x;
    hi[0] += v0.y;
#pragma unroll
    for (int y = 1; y < NY; y += 2) {
      const double pr = hr[y], pi = hi[y], mr = hr[y + 1], mi = hi[y + 1];
      hr[y] = pr + mr;
      hi[y] = pi + mi;
      hr[y + 1] = pr - mr;
      hi[y + 1] = pi - mi;
    }
    const size_t base = (size_t)row * Lq * BB;
    for (int q = q0; q < q1; q += NU) {
      double2 x[NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) x[u] = X[base + (size_t)min(q + u, q1 - 1) * BB];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if (u && q + u >= q1) break;
        Phases<NP> f;
        f.read(ph, q + u);
        double vr = x[u].x + hr[0], vi = x[u].y + hi[0];
#pragma unroll
        for (int y = 0; y < NP; ++y) {
          vr = fma(f.p[y].x, hr[2 * y + 1], fma(-f.p[y].y, hi[2 * y + 2], vr));
          vi = fma(f.p[y].x, hi[2 * y + 1], fma(f.p[y].y, hr[2 * y + 2], vi));
        }
        if constexpr (SRC == 1) {
          // the four lanes of a quad hold four elements in a row: lane j stores
          // plane j of all four, eight bytes (2-byte stores instead: 783 us,
          // with these 767, with the XCDs on ranges of their own 704; t2g 16 x 16, 13
          // form factors)
          unsigned hi, lo;
          split2((float)vr, (float)vi, hi, lo);
          const bool odd = el & 1, upper = el & 2;
          const unsigned o1 = __builtin_amdgcn_mov_dpp((int)(odd ? hi : lo), 0xB1, 0xf, 0xf, true);  // lane ^ 1
          const unsigned w0 = odd ? o1 : hi, w1 = odd ? lo : o1;  // hi (odd lanes: lo) of elements 0, 1 of the pair
          const unsigned re = __builtin_amdgcn_perm(w1, w0, 0x05040100), im = __builtin_amdgcn_perm(w1, w0, 0x07060302);
          const unsigned o2 = __builtin_amdgcn_mov_dpp((int)(upper ? re : im), 0x4E, 0xf, 0xf, true);  // lane ^ 2
          if (valid) *(uint2 *)(S + 4 * (base + (size_t)(q + u) * BB)) = upper ? make_uint2(o2, im) : make_uint2(re, o2);
        } else if constexpr (SRC == 3) {
          if (valid) F[base + (size_t)(q + u) * BB] = make_float2((float)vr, (float)vi);
        } else {
          if (valid) V[base + (size_t)(q + u) * BB] = make_double2(vr, vi);
        }
      }
    }
  }
}

// Elements per workgroup and pieces per qx row.  64 elements once that gives the
// chip several workgroups per CU; fewer elements otherwise (ft + assemble at BB =
// 2704, Lq 15: 28 us with 16 elements, 40 with 4; at 1296, Lq 24: 37 with 16, 32
// with 4; at 81: 30 with 16, 15 with 4).  Pieces: the fewest rounds of loads over
// the units of a workgroup, a round costing the unit's own work (its rho sums)
// besides.
struct ProjSplit {
  int ew, parts;
};
ProjSplit proj_split(const ProjArgs &a) {
  const int BB = a.B * a.B;
  ProjSplit s;
  s.ew = BB >= 32768 && a.nD <= NDS ? 64 : BB >= 2000 ? 16 : 4;
  const int ng = NTHR / s.ew;
  int best = 0;
  s.parts = 1;
  for (int p = 1; p <= ng && p <= a.Lq; p *= 2) {
    const int rounds = (a.Lq * p + ng - 1) / ng, cost = rounds * ((a.Lq + p - 1) / p + 8);
    if (p == 1 || cost < best) best = cost, s.parts = p;
  }
  return s;
}

bool proj_ok(const ProjArgs &a) {
  return (a.np == 0 || a.np == 2 || a.np == 4) && a.Nq == a.Lq * a.Lq && a.nD >= 1 && a.nD <= 81 && a.Lq <= 4096;
}

}  // namespace

template <int EW, int NP>
static void ft_launch(const ProjArgs &a, int parts, const double *P, const double *C, double *real, hipStream_t st) {
  const int BB = a.B * a.B;
  const dim3 grid((2 * ((BB + EW - 1) / EW) + 7) / 8 * 8);
  const size_t lds = sizeof(double2) * ((size_t)a.Lq + (EW < 64 ? a.Lq * NP : 0));
  const double scale = 1.0 / (double)a.Nq;
#define TUFRG_FT(BIG)                                                                                              \
  hipLaunchKernelGGL((ft_kernel<EW, NP, rho_per_thread(EW, BIG)>), grid, dim3(NTHR), lds, st, BB, a.Lq, a.nD, parts, \
                     scale, (const double2 *)a.phy, (const double2 *)a.twq, a.dtab, (const double2 *)P,            \
                     (const double2 *)C, (double2 *)real)
  if (a.nD <= NDS)
    TUFRG_FT(0);
  else if constexpr (EW < 64)
    TUFRG_FT(1);
#undef TUFRG_FT
}

template <int EW, int NP, int SRC>
static void assemble_launch(const ProjArgs &a, int parts, const double *P, const double *C, const double *src,
                            const double *v0p, const double *v0c, void *VP, void *VC, int nw, hipStream_t st) {
  const int BB = a.B * a.B;
  const dim3 grid((nw * ((BB + EW - 1) / EW) + 7) / 8 * 8);
  const size_t lds = sizeof(double2) * ((size_t)a.nD * EW + a.Lq + (EW < 64 ? a.Lq * NP : 0));
  const unsigned magic = (unsigned)((((unsigned long long)1 << 32) + a.Lq - 1) / a.Lq);
  const GatherTables gt{a.n_o, a.n_ff, a.B, a.nD, a.ff, a.dlist, a.ffgrid, a.dgrid};
  hipLaunchKernelGGL((assemble_kernel<EW, NP, SRC>), grid, dim3(NTHR), lds, st, BB, a.Lq, a.nD, nw, parts, magic, gt,
                     (const double2 *)a.phy, (const double2 *)a.twq, a.dslot, (const double2 *)src, (const double2 *)P,
                     (const double2 *)C, (const double2 *)v0p, (const double2 *)v0c, VP, VC);
}

// the rho_y of a set within |R| <= 2 closed under R -> -R: 0, two or four pairs
#define TUFRG_PROJ_NP(EW, CALL) \
  if (a.np == 0)                \
    CALL(EW, 0);                \
  else if (a.np == 2)           \
    CALL(EW, 2);                \
  else                          \
    CALL(EW, 4);
#define TUFRG_PROJ(CALL)       \
  if (sp.ew == 64) {           \
    TUFRG_PROJ_NP(64, CALL)    \
  } else if (sp.ew == 16) {    \
    TUFRG_PROJ_NP(16, CALL)    \
  } else {                     \
    TUFRG_PROJ_NP(4, CALL)     \
  }

hipError_t launch_ft(const ProjArgs &a, const double *P, const double *C, double *real, hipStream_t st) {
  if (!proj_ok(a)) return hipErrorInvalidValue;
  const ProjSplit sp = proj_split(a);
#define TUFRG_FT_CALL(EW, NP) ft_launch<EW, NP>(a, sp.parts, P, C, real, st)
  TUFRG_PROJ(TUFRG_FT_CALL)
#undef TUFRG_FT_CALL
  return hipGetLastError();
}

hipError_t launch_assemble(const ProjArgs &a, const double *P, const double *C, const double *real,
                           const double *v0p, const double *v0c, void *VP, void *VC, VForm form, hipStream_t st) {
  if (!proj_ok(a)) return hipErrorInvalidValue;
  const ProjSplit sp = proj_split(a);
#define TUFRG_AS_CALL(EW, NP)                                                                                 \
  form == V_PLANES ? assemble_launch<EW, NP, V_PLANES>(a, sp.parts, P, C, real, v0p, v0c, VP, VC, 2, st)    \
  : form == V_FP32 ? assemble_launch<EW, NP, V_FP32>(a, sp.parts, P, C, real, v0p, v0c, VP, VC, 2, st)      \
                   : assemble_launch<EW, NP, V_FP64>(a, sp.parts, P, C, real, v0p, v0c, VP, VC, 2, st)
  TUFRG_PROJ(TUFRG_AS_CALL)
#undef TUFRG_AS_CALL
  return hipGetLastError();
}

hipError_t launch_assemble_gathered(const ProjArgs &a, const double *P, const double *C, const double *G,
                                    const double *v0p, const double *v0c, double *VP, double *VC, hipStream_t st,
                                    int nw) {
  if (!proj_ok(a) || nw < 1 || nw > 2) return hipErrorInvalidValue;
  const ProjSplit sp = proj_split(a);
#define TUFRG_AS_CALL(EW, NP) assemble_launch<EW, NP, 2>(a, sp.parts, P, C, G, v0p, v0c, VP, VC, nw, st)
  TUFRG_PROJ(TUFRG_AS_CALL)
#undef TUFRG_AS_CALL
  return hipGetLastError();
}
#undef TUFRG_PROJ
#undef TUFRG_PROJ_NP

// D[q][(R,a,b)][(R',c,d)] = -C[q][(R,a,c)][(R',b,d)]: the third channel in the
// layout of C, D_{n1n2n3n4} = -C_{n1n2n4n3}; a pure gather, exact
__global__ void channel_d_kernel(int n_o, int B, long long n, const double2 *__restrict__ C,
                                 double2 *__restrict__ D) {
  const int no2 = n_o * n_o;
  const long long BB = (long long)B * B;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const int col = (int)(i % B), row = (int)((i / B) % B);
    const long long q = i / BB;
    const int r = row / no2, a = (row % no2) / n_o, b = row % n_o;
    const int rp = col / no2, c = (col % no2) / n_o, d = col % n_o;
    const double2 v = C[q * BB + (long long)(r * no2 + a * n_o + c) * B + (rp * no2 + b * n_o + d)];
    D[i] = make_double2(-v.x, -v.y);
  }
}

hipError_t launch_channel_d(int n_o, int B, int Nq, const double *C, double *D, hipStream_t st) {
  const long long n = (long long)Nq * B * B;
  const long long blocks = std::min<long long>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(channel_d_kernel, dim3((unsigned)std::max<long long>(blocks, 1)), dim3(256), 0, st, n_o, B, n,
                     (const double2 *)C, (double2 *)D);
  return hipGetLastError();
}

}  // namespace tufrg
