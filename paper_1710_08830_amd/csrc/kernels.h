// Host-side launchers of the TU-fRG kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>

namespace tufrg {

// a0: band data on the fine mesh (eigenvalues minus mu, packed projectors)
// unit_pi: band basis, Pi_m(k) = e_m e_m^T (eigenvalues as always)
hipError_t launch_band(int n_o, int Lf, int n_hop, const int *hop_R, const double *hop_t, double mu, int unit_pi,
                       double *e, double *pi, float *e32, float *pi32, hipStream_t st);
hipError_t launch_kval(int n, int Nf, int aos_no, const double *e, double lam, int scheme, int deriv, double *kv,
                       float *kv32, hipStream_t st);
// two orbitals: ekv[k] = (e_0, e_1, K(e_0), K(e_1)) and the static pi4[k], k-major 4-vectors
hipError_t launch_ekv4(int Nf, const double *band, double lam, int scheme, int deriv, double *ekv, float *ekv32,
                       hipStream_t st);
hipError_t launch_pi4(int Nf, const double *band, double *pi4, float *pi4_32, hipStream_t st);
// shell scheme: factors (a, b) of every band value e[m][k] (component-major);
// two orbitals [Nf][4] = (a_0, a_1, b_0, b_1), more orbitals [Nf][n_o][2]
hipError_t launch_shell_ab(int n_o, int Nf, const double *e, double lam, int deriv, double *cv, float *cv32,
                           hipStream_t st);
// component-major [nc][Nf] -> k-major [Nf][nc] (FP64 and FP32)
hipError_t launch_to_kmajor(int nc, int Nf, const double *src, double *dst, float *dst32, hipStream_t st);

// a1-a3: form-factor projected orbital loops
struct LoopArgs {
  int n_o, Lq, n_ref, Lf, Nq;
  int ndx, ndy;        // computed box: dx in [0, ndx), dy in [-ndy, ndy]
  int nkyb, kxper;     // ky blocks of 64 lanes, kx rows per chunk
  int nparts;          // partial sums kept per item (at least ky blocks x kx chunks)
  int kxr = 2;         // six spin-orbitals on the matrix cores: kx rows per work item (1..8)
  // items: the (channel, coarse q) whose k sums are taken, q | ch << 30, n_pp of
  // channel 0 then n_ph of channel 1; dst per item: the output slots of q and of
  // -q (-1: none) among the n_q_out of its channel (see loop_sym.h)
  const int *items = nullptr;
  const int2 *dst = nullptr;
  int n_pp = 0, n_ph = 0, n_q_out = 0;
  int half = 0;        // bit ch: one of each pair of kx rows (kx, qx - kx) is summed
  int trs = 0;         // time reversal of the bands (see loop_sym.h)
  const double *twq = nullptr;  // exp(+2 pi i j / Lq), [Lq][2]
  int scheme, deriv, prec;
  double lam;
  const void *band;    // band data (FP64 or FP32 by prec): two orbitals component-major
                       // [n_o + n_o^3][Nf], more orbitals k-major [Nf][n_o + n_o^3]
  const void *kv;      // regulator values, [n_o][Nf] or [Nf][n_o] like the band data
  const double *tw;    // exp(-2 pi i j / Lf), [Lf][2]
  const float *tw32 = nullptr;  // the same in FP32
  void *partial;       // [items][nparts][ndx][2 ndy + 1][n_o^4][2] in the arithmetic type
                       // (FP64 for TUFRG_FP64, else FP32: the partials carry no more)
  const int *pairs = nullptr;  // more than two orbitals: [n_pairs][2] entry and its conjugate partner
  int n_pairs = 0;
  const void *phy = nullptr;   // more than two orbitals: exp(-2 pi i ky dy / Lf), [Lf][ndy][2], like band
  const void *ekv = nullptr;   // two orbitals: [Nf][4] = (e_0, e_1, K(e_0), K(e_1)), like band
  const void *pi4 = nullptr;   // two orbitals: [Nf][4] = (Pi_0[00], Pi_0[11], Re Pi_0[01], Im Pi_0[01])
  const void *cv = nullptr;    // shell scheme: shell factors, two orbitals [Nf][4] = (a_0, a_1, b_0, b_1),
                               // more orbitals [Nf][n_o][2] = (a_m, b_m); like band
  int pair = 0;                // six spin-orbitals on the matrix cores: bands (0,1), (2,3), (4,5)
                               // degenerate at every k, summed by pairs
  const float *pir = nullptr;     // with pair: [Nf][3][36] pair sums of the packed projectors (FP32)
  const double *pir64 = nullptr;  // the same in FP64 (six spin-orbitals on the vector units, FP64)
};
hipError_t launch_loop(const LoopArgs &a, hipStream_t st);
// several two-orbital instances of one precision in fused launches (one per
// kernel shape and regulator): instance i sums all its items of both channels
// into a[i].partial, with the work items of its own launch_loop.
// desc_h (pinned host) and desc_d (device) hold n descriptors; desc_h is
// rewritten, so the previous call's copies must be complete.
struct No2Inst {
  const void *ekv, *pi4, *cvp, *twk;
  const double *tw;
  const int *items;
  void *partial;
  double lam;
  int Lq, n_ref, Lf, nkyb, kxper, nparts, half, n_pp, n_ph, deriv, work0, pad;
};
hipError_t launch_loop_batch(const LoopArgs *a, int n, No2Inst *desc_h, No2Inst *desc_d, hipStream_t st);
// more than two spin-orbitals (six: t2g with spin-orbit coupling)
hipError_t launch_loop_gen(const LoopArgs &a, hipStream_t st);
// six spin-orbitals on the matrix cores in the real basis of Hermitian
// matrices (one channel): row buffers Y of loop_rb_rowbuf_floats(ndy, Lf)
// floats per group of four coarse q, then (sums) the compact loops; the
// half-plane points of the computed shape from loop_rb_half_points.  The A
// operand (phases times projectors, split; independent of q, Lambda and the
// channel) is computed once into loop_rb_apre_bytes(ndy, Lf) bytes.
size_t loop_rb_apre_bytes(int ndy, int Lf, int pair);
hipError_t launch_loop_rb_apre(int ndy, int pair, const float *band, const float *pir, const float *phy, int Lf,
                               void *apre, hipStream_t st);
// pair sums of the packed projectors into pir (FP32) and/or pir64 (FP64; either may be null)
hipError_t launch_pair_pi(int Nf, const double *band, float *pir, double *pir64, hipStream_t st);
// (the items of one channel: n_pp or n_ph is zero)
hipError_t launch_loop_rb(const LoopArgs &a, const void *apre, float *Y, hipStream_t st);
hipError_t launch_loop_rb_sums(const LoopArgs &a, const float *Y, double *lamb, const int *hmap, const int *dlist,
                               int nD, double *out, hipStream_t st);
size_t loop_rb_rowbuf_floats(int ndy, int Lf);
int loop_rb_half_points(int ndy, int *dx, int *dy);
// the same in 15 coordinates per pair sum, for models with time reversal times
// inversion (k_loop_kr.hip): pair sums x, per-evaluation energies and regulator
// values ek (16 floats per k with shell factors, else 8), A operand, row buffers
// and coordinates lam per item
size_t kr_x_floats(int Lf);
hipError_t launch_kr_x(int Lf, const double *band, float *x, hipStream_t st);
size_t kr_apre_bytes(int ndy, int Lf);
hipError_t launch_kr_apre(int ndy, const double *bandk, const float *phy, int Lf, void *apre, hipStream_t st);
hipError_t launch_kr_ek(int Nf, int shell, const double *band, double vlam, int vscheme, int vderiv, double lam,
                        int deriv, float *ek, hipStream_t st);
size_t kr_rowbuf_floats(int ndy, int Lf);
size_t kr_lam_doubles(int ndy);
hipError_t launch_loop_kr(const LoopArgs &a, const float *x, const float *ek, const void *apre, float *Y,
                          hipStream_t st);
hipError_t launch_loop_kr_sums(const LoopArgs &a, const float *Y, double *lam, const int *hmap, const int *dlist, int nD,
                               double *out, hipStream_t st);
// sums partials, applies 1/Nf, fills dx < 0 by hermiticity and the other half
// of the sum and of the coarse q by symmetry
hipError_t launch_loop_finalize(const LoopArgs &a, int nD, const int *dlist, double *compact, hipStream_t st);
// compact [n_ch][n_q][nD][n_o^4] -> full [n_q][B][B] for one channel
hipError_t launch_loop_expand(int n_o, int n_ff, int nD, int n_q, const int *didx, const double *compact,
                              double *out, hipStream_t st);

// a4-a5: real-space transform, gathers, assembly of projected vertices
struct ProjArgs {
  int n_o, n_ff, B, Lq, Nq, nD;
  const int *dlist;    // [nD][2]
  const int *ffgrid;   // [17][17] form-factor index of (x, y) in [-8, 8]^2, -1 outside S
  const int *dgrid;    // [17][17] index into dlist, -1 outside D
  const int *ff;       // [n_ff][2]
  const double *twq;   // exp(+2 pi i j / Lq), [Lq][2]
  int np;              // the rho_y of D are 0 (slot 0) and np <= 4 pairs +-y (slots 2 y + 1, 2 y + 2)
  const double *phy;   // (cos, sin)(2 pi qy y / Lq) of the pairs, [Lq][np][2]
  const int *dtab;     // per rho of dlist: (rho_x mod Lq) | (slot of rho_y) << 16
  const int *dslot;    // [9][9] per slot the rho of D with that rho_y: iD | (rho_x mod Lq) << 16, else -1
};
// real [2][nD][B][B]: P(rho), C(rho)
hipError_t launch_ft(const ProjArgs &a, const double *P, const double *C, double *real, hipStream_t st);
// D [Nq][B][B] (layout of C) from C: D_{n1n2n3n4} = -C_{n1n2n4n3}
hipError_t launch_channel_d(int n_o, int B, int Nq, const double *C, double *D, hipStream_t st);
// VP, VC from the transforms P(rho), C(rho) at real, in the form the bundle
// products take them: complex FP64 or FP32, or split planes [Nq][4][B][B] of BF16
// (Re hi, Re lo, Im hi, Im lo; x = hi + lo)
enum VForm { V_FP64 = 0, V_PLANES = 1, V_FP32 = 3 };
hipError_t launch_assemble(const ProjArgs &a, const double *P, const double *C, const double *real,
                           const double *v0p, const double *v0c, void *VP, void *VC, VForm form, hipStream_t st);
// the same from the gathers G [nw][nD][B][B]; nw = 1: only VP from P and G[0]
hipError_t launch_assemble_gathered(const ProjArgs &a, const double *P, const double *C, const double *G,
                                    const double *v0p, const double *v0c, double *VP, double *VC, hipStream_t st,
                                    int nw = 2);

// a6: bundle products  out = f * V L V  per q, L expanded from compact form, of
// n_ch channels; bundles larger than 64 need a workspace tmp of n_q * B * B complex
struct BundleArgs {
  const void *V;  // complex FP64 for prec 0, FP32 otherwise (launch_assemble)
  const double *Lc;
  double f;
  double *out;
};
hipError_t launch_bundle(int prec, int n_o, int n_ff, int B, int nD, int n_q, const int *didx, const BundleArgs *a,
                         int n_ch, double *tmp, hipStream_t st);
// the same on the matrix cores with BF16 split operands (k_bundle_mfma.hip), V in
// split planes (launch_assemble), in chunks of q that fit the workspace ws (at
// least bundle_split_bytes_per_q)
size_t bundle_split_bytes_per_q(int n_o, int B, int nD);
hipError_t launch_bundle_bf16x3(int n_o, int n_ff, int B, int nD, int n_q, const int *didx, const void *V,
                                const double *Lc, double factor, double *out, void *ws, size_t ws_bytes,
                                hipStream_t st);

// SU(2)-reduced flow of one orbital (k_su2.hip): one-band loops (partial sums
// like the two-orbital ones, finished by launch_loop_finalize); X -> X^x; the
// gathers G[3][nD][B][B] of a~, c~, d~ from rA = (p, c)(rho), rB = (p^x, d)(rho);
// the reduced products per q (B <= 25)
hipError_t launch_loop1(const LoopArgs &a, hipStream_t st);
hipError_t launch_su2_exch(int n_ff, int Nq, int Lq, const int *ff, const int *fneg, const double *twq,
                           const double *X, double *Xx, hipStream_t st);
hipError_t launch_su2_gather(int B, int nD, const int *ff, const int *dlist, const int *ffgrid, const int *dgrid,
                             const double *rA, const double *rB, double *G, hipStream_t st);
hipError_t launch_su2_bundle(int B, int Nq, int nD, const int *didx, const double *Lc, const double *Va,
                             const double *Vax, const double *Vc, const double *Vd, double f, double *dp, double *dc,
                             double *dd, hipStream_t st);

// orbital <-> band basis (k_basis.hip): compact basis matrix [Nq][nD][n_o^4] of one
// channel (0: pp, U matrix; 1: ph, X matrix) from U[Nf][n_o][n_o] (orbital rows, band
// columns); box: D inside [-box, box]^2 (2 or 4); dlist [nD][2]; tw = exp(-2 pi i j /
// Lf), [Lf][2]; rows: workspace of basis_rows_doubles(n_o, Lf, box, q_chunk) doubles
// (the coarse q are processed q_chunk at a time)
size_t basis_rows_doubles(int n_o, int Lf, int box, int nq);
hipError_t launch_basis_compact(int channel, int n_o, int Lq, int n_ref, int nD, int box, const int *dlist,
                                const double *U, const double *tw, double *rows, int q_chunk, double *out,
                                hipStream_t st);
// Y[q] = (A (x) 1) X[q] (A (x) 1)^H in the form-factor index, A [n_ff][n_ff] complex on the device
hipError_t launch_ff_apply(int n_ff, int no2, int n_q, const double *A, const double *X, double *Y, hipStream_t st);
// C[q] = opA(A[q]) opB(B[q]), n x n complex, op 1 = conjugate transpose (not both)
hipError_t launch_zgemm_batched(int n, int n_q, int opA, int opB, const double *A, const double *Bm, double *C,
                                hipStream_t st);

// a7: ODE updates and reductions
struct StepArrays {
  const double *x[3], *dx[3];
  double *y[3];
};
// y = x + h dx per array (null dx: no update; null y: no result), max |y| and the
// non-finite flag over all to out_bits, out_flag; bits, flag, ticket zero between launches
hipError_t launch_step_max(long long n, const StepArrays &a, int n_arr, double h, unsigned long long *bits,
                           unsigned int *flag, unsigned int *ticket, unsigned long long *out_bits,
                           unsigned int *out_flag, hipStream_t st);
hipError_t launch_lincomb(long long n, const double *x, int nk, const double *const *k, const double *coef,
                          double h, double *y, hipStream_t st);
hipError_t launch_dp_error(long long n, const double *x0, const double *x1, int nk, const double *const *k,
                           const double *ecoef, double h, double rtol, double atol, unsigned long long *errbits,
                           unsigned int *flag, hipStream_t st);
hipError_t launch_clear_reduce(unsigned long long *bits, unsigned int *flag, hipStream_t st);
hipError_t launch_scale(long long n, const double *x, double s, double *y, hipStream_t st);
// y = a + b over n doubles (n even: complex arrays)
hipError_t launch_add(long long n, const double *a, const double *b, double *y, hipStream_t st);

// loop surrogate network (k_mlp.hip)
// FP32 product C[M][N] = A B on the matrix cores (see k_mlp.hip): A(m, k) = tA ?
// A[k lda + m] : A[m lda + k], B(k, n) = tB ? B[n ldb + k] : B[k ldb + n]
enum { GEMM_PLAIN = 0, GEMM_BIAS, GEMM_GELU, GEMM_GELU_BWD, GEMM_LOSS };
struct GemmF32 {
  int M = 0, N = 0, K = 0, lda = 0, ldb = 0, tA = 0, tB = 0;
  int splits = 1;  // K ranges over workgroups, each to its own C [splits][M][N] (and db [splits][M])
  int epi = GEMM_PLAIN;
  const float *A = nullptr, *B = nullptr;
  float *C = nullptr;
  const float *bias = nullptr;  // [N]: BIAS, GELU, LOSS
  float *Z = nullptr;           // [M][N]: GELU writes the pre-activation, GELU_BWD multiplies by GELU'(Z)
  float *db = nullptr;          // [M]: sums over k of A
  const float *T = nullptr;     // LOSS: C = 2 inv (y - T), loss_part[workgroup] = inv sum (y - T)^2
  double *loss_part = nullptr;
  double inv = 0.0;
};
int gemm_f32_blocks(const GemmF32 &p);
// a forward product (tB), and the weight (tA) and data gradients of a layer in one launch
hipError_t launch_gemm_f32(const GemmF32 &p, hipStream_t st);
hipError_t launch_gemm_f32_bwd(const GemmF32 &w, const GemmF32 *d, hipStream_t st);
// sums of split gradients, dst[i] = sum_s src[s len + i], and loss += sum of loss_part
struct GradParts {
  static constexpr int MAX = 32;
  int n = 0;
  struct {
    const float *src;
    float *dst;
    long long len;
    int splits, block0;
  } part[MAX];
};
hipError_t launch_grad_reduce(GradParts gp, const double *loss_part, int n_loss, double *loss, hipStream_t st);
hipError_t launch_adam(long long n, float *p, const float *g, float *m, float *v, float lr, float b1, float b2,
                       float eps, int t, hipStream_t st);
hipError_t launch_gather_rows(int rows, int len, const int *idx, const float *src, float *dst, hipStream_t st);
hipError_t launch_sur_features(long long n, const int *ql, const int *cl, const int *dl, int Lq, int nD, double lam,
                               float *X, hipStream_t st);
hipError_t launch_sur_targets(long long n, const int *ql, const int *cl, const int *dl, int Nq, int nD, int no4,
                              double s, const double *Lc, float *T, unsigned int *bits, hipStream_t st);
hipError_t launch_sur_scatter(long long n, int no4, double s, const float *Y, double *Lc, unsigned int *bad,
                              hipStream_t st);
hipError_t launch_sur_compare(long long n, const double *a, const double *b, unsigned long long *bits,
                              hipStream_t st);

}  // namespace tufrg
