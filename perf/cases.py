"""The work that a user of this library has it do, as measurable cases.

A case is a plain dict.  ``op`` names the call, the other keys its sizes:

* ``rhs``      one right-hand side dP, dC of a state P, C (``tufrg_rhs``): what
               an own integrator, or a study of one scale, calls;
* ``flow``     an Euler flow from the bare vertex (``tufrg_flow``);
* ``su2``      one SU(2)-reduced right-hand side of one orbital per site
               (``tufrg_su2_rhs``);
* ``batch``    a lockstep flow of uneven Rashba instances
               (``tufrg_batch_flow``): a scan over parameters;
* ``loops``    the training data of the loop surrogate at one scale: compact
               loops, their scale, features and targets
               (``tufrg_loops_compact``, ``tufrg_sur_features``,
               ``tufrg_sur_targets``);
* ``project``  the projected vertices of a state (``tufrg_project``);
* ``grad``     loss and gradient of the surrogate network over one batch
               (``tufrg_mlp_loss_grad``), for an optimiser of the caller's.

``prec`` is the arithmetic the context is created with.  Right-hand sides and
states of FP32 and BF16X3 contexts are handed on in complex64, as a program
that asked for single-precision arithmetic records them (six spin-orbitals:
several GB per state in complex128); FP64 ones in complex128.

Chemical potential, scale, interaction strength and state come from the seed.
"""

import math

import numpy as np
import torch

from paper_1710_08830_amd import tufrg as T

DEV = "cuda"

_SHELL = [(0, 0), (1, 0), (-1, 0), (0, 1), (0, -1), (1, 1), (-1, -1), (1, -1), (-1, 1),
          (2, 0), (-2, 0), (0, 2), (0, -2)]


def listed():
    return [
        # the smallest problem: an 8 x 8 Hubbard lattice, where launches and latency count
        dict(name="hubbard_s5_rhs", op="rhs", model="hubbard", S=5, L=8, n_ref=12, cutoff="temperature", prec="fp64"),
        # the same lattice as a whole call: 20 Euler steps with the stop test after each
        dict(name="hubbard_s5_flow", op="flow", model="hubbard", S=5, L=8, n_ref=12, cutoff="temperature",
             prec="fp64", steps=20),
        # the spin-rotation-invariant form of a larger lattice
        dict(name="su2_s9_L24", op="su2", model="hubbard1", S=9, L=24, n_ref=12, cutoff="temperature", prec="fp64"),
        # double precision on odd meshes with the momentum-shell regulator
        dict(name="rashba_s13_L15_shell", op="rhs", model="rashba", S=13, L=15, n_ref=7, cutoff="shell", prec="fp64"),
        # the Rashba model of the paper on the mesh that the benchmark uses
        dict(name="rashba_s9_L24_fp32", op="rhs", model="rashba", S=9, L=24, n_ref=24, cutoff="omega", prec="fp32"),
        # a parameter scan: uneven instances in lockstep
        dict(name="rashba_batch12", op="batch", model="rashba", n=12, n_ref=12, cutoff="temperature", prec="fp32",
             steps=4),
        # the largest: loops of the t2g model with spin-orbit coupling on the benchmark's 32 x 32 mesh
        dict(name="t2g_s13_L32_loops", op="loops", model="t2g", S=13, L=32, n_ref=16, cutoff="temperature",
             prec="bf16x3"),
        # a right-hand side of that model at an ordinary size
        dict(name="t2g_s13_L16_bf16x3", op="rhs", model="t2g", S=13, L=16, n_ref=8, cutoff="temperature",
             prec="bf16x3"),
        # the double-precision run that such results are checked with
        dict(name="t2g_s13_L10_fp64", op="rhs", model="t2g", S=13, L=10, n_ref=6, cutoff="omega", prec="fp64"),
        # the model in a magnetic field (no degenerate bands), odd meshes, FP32
        dict(name="t2g_zeeman_s9_L11_fp32", op="rhs", model="zeeman", S=9, L=11, n_ref=5, cutoff="temperature",
             prec="fp32"),
        # the projections alone on the benchmark's mesh: states of 3.6 GB
        dict(name="t2g_s13_L32_project", op="project", model="t2g", S=13, L=32, n_ref=2, cutoff="temperature",
             prec="fp32"),
        # one gradient of the surrogate of the t2g loops
        dict(name="t2g_net_grad", op="grad", n_in=52, width=256, n_out=2592, rows=2048),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["rhs2", "rhs2", "rhs6", "rhs6", "loops2", "loops6", "flow", "su2", "batch", "project", "grad"])
    S = rng.choice([5, 9, 13])
    lo = 9 if S == 13 else 5
    cut = rng.choice(["temperature", "omega", "shell"])
    if op in ("rhs2", "loops2"):
        L = _logint(rng, lo, 32)
        return dict(op=op[:-1], model=rng.choice(["hubbard", "rashba"]), S=S, L=L,
                    n_ref=rng.randint(2, max(2, min(24, 600 // L))), cutoff=cut, prec=rng.choice(["fp64", "fp32"]))
    if op == "rhs6":
        L = _logint(rng, lo, 18)
        return dict(op="rhs", model=rng.choice(["t2g", "t2g", "zeeman"]), S=S, L=L,
                    n_ref=rng.randint(2, max(2, 90 // L)), cutoff=cut, prec=rng.choice(["bf16x3", "fp32", "fp64"]))
    if op == "loops6":
        L = _logint(rng, lo, 30)
        return dict(op="loops", model=rng.choice(["t2g", "t2g", "zeeman"]), S=S, L=L,
                    n_ref=rng.randint(2, max(2, 240 // L)), cutoff=cut, prec="bf16x3")
    if op == "flow":
        L = _logint(rng, lo, 16)
        return dict(op="flow", model=rng.choice(["hubbard", "rashba"]), S=S, L=L, n_ref=rng.randint(4, 12),
                    cutoff=rng.choice(["temperature", "omega"]), prec="fp64", steps=rng.randint(10, 30))
    if op == "su2":
        return dict(op="su2", model="hubbard1", S=S, L=_logint(rng, lo, 32), n_ref=rng.randint(3, 16),
                    cutoff=rng.choice(["temperature", "omega"]), prec="fp64")
    if op == "batch":
        return dict(op="batch", model="rashba", n=rng.randint(3, 12), n_ref=rng.randint(6, 12), cutoff="temperature",
                    prec="fp32", steps=rng.randint(2, 5))
    if op == "project":
        return dict(op="project", model=rng.choice(["rashba", "t2g"]), S=S, L=_logint(rng, lo, 30), n_ref=2,
                    cutoff="temperature", prec="fp32")
    n_dR = {5: 13, 9: 25, 13: 41}[S]
    return dict(op="grad", n_in=11 + n_dR, width=rng.choice([128, 200, 256]), n_out=rng.choice([32, 2592]),
                rows=_logint(rng, 100, 4096))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

_PAULI = np.array([[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]], dtype=np.complex128)


def _hoppings(model, alpha=0.3):
    """(hop_R, hop_t) of the square-lattice models, H(k) = sum_R t(R) e^{ik.R}."""
    if model in ("hubbard", "hubbard1"):
        one = np.eye(2 if model == "hubbard" else 1)
        ent = [(r, -one) for r in _SHELL[1:5]] + [(r, 0.25 * one) for r in _SHELL[5:9]]
    elif model == "rashba":
        one, sx, sy = np.eye(2), _PAULI[0], _PAULI[1]
        ent = [((1, 0), -one + alpha * sy / 2j), ((-1, 0), -one - alpha * sy / 2j),
               ((0, 1), -one - alpha * sx / 2j), ((0, -1), -one + alpha * sx / 2j)]
    else:  # three t2g orbitals with spin-orbit coupling; "zeeman": in a field along z
        rng = np.random.default_rng(1)
        iu = np.triu_indices(3)
        ent = []
        for j, d in enumerate([(1, 0), (0, 1), (1, 1), (1, -1)]):
            lo, hi = (0.2, 1.0) if j < 2 else (0.0, 0.2)
            t = np.zeros((3, 3))
            t[iu] = rng.uniform(lo, hi, size=6)
            t = np.kron(t + np.triu(t, 1).T, np.eye(2))
            ent += [(d, -t), ((-d[0], -d[1]), -t.T)]
        on = np.zeros((6, 6), dtype=np.complex128)
        for i in range(3):
            l = np.zeros((3, 3), dtype=np.complex128)
            l[(i + 1) % 3, (i + 2) % 3], l[(i + 2) % 3, (i + 1) % 3] = -1j, 1j
            on += 0.1 * np.kron(l, _PAULI[i])
        if model == "zeeman":
            on = on + 0.05 * np.kron(np.eye(3), _PAULI[2])
        ent.append(((0, 0), on))
    return np.array([r for r, _ in ent], dtype=np.int32), np.array([t for _, t in ent], dtype=np.complex128)


def _vertex(n_o, U):
    """Antisymmetric onsite vertex: Hubbard (one orbital), Kanamori with J = 0.15 U (three), or
    the onsite coefficient of the SU(2)-reduced form."""
    if n_o == 1:
        return np.full((1, 1, 1, 1), 0.5 * U, dtype=np.complex128)
    J, no = 0.15 * U, n_o // 2
    I = np.zeros((no,) * 4)
    for a in range(no):
        for b in range(no):
            if a == b:
                I[a, a, a, a] = U
            else:
                I[a, b, a, b], I[a, b, b, a], I[a, a, b, b] = U - 2 * J, J, J
    d = np.eye(2)
    W = np.einsum("abcd,st,uv->asbuctdv", I, d, d).reshape((n_o,) * 4)
    return (0.5 * (W - W.transpose(0, 1, 3, 2))).astype(np.complex128)


def _problem(case, seed):
    """Model and scale of a case, from the seed."""
    rng = np.random.default_rng(seed)
    hop_R, hop_t = _hoppings(case["model"])
    n_o = hop_t.shape[1]
    mu = {"hubbard": -0.6, "hubbard1": -0.6, "rashba": -0.4}.get(case["model"], 0.35) + rng.uniform(-0.2, 0.2)
    return dict(hop_R=hop_R, hop_t=hop_t, n_o=n_o, mu=mu, V0=_vertex(n_o, rng.uniform(1.5, 3.0)),
                ff=np.array(_SHELL[:case["S"]], dtype=np.int32), Lq=case["L"], n_ref=case["n_ref"],
                cutoff=case["cutoff"], temperature=0.06 if case["cutoff"] == "shell" else None, prec=case["prec"],
                lam=math.exp(rng.uniform(math.log(0.1), 0.0)))


def _instances(case, seed):
    """Uneven Rashba instances, as a scan over filling, coupling, interaction, mesh and shell has them."""
    rng = np.random.default_rng(seed)
    out = []
    for i in range(case["n"]):
        hop_R, hop_t = _hoppings("rashba", rng.uniform(0.0, 0.5))
        out.append(dict(hop_R=hop_R, hop_t=hop_t, n_o=2, mu=rng.uniform(-1.0, 0.0), V0=_vertex(2, rng.uniform(1.5, 3.5)),
                        ff=np.array(_SHELL[:(5, 9, 13)[i % 3]], dtype=np.int32), Lq=(16, 24, 32)[(i // 3) % 3],
                        n_ref=case["n_ref"], cutoff=case["cutoff"], temperature=None))
    return out


def _state(n, Nq, B, seed):
    """n random Hermitian [Nq][B][B] bundles of the size that couplings have in a flow."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    out = []
    for _ in range(n):
        x = torch.randn((Nq, B, B, 2), generator=g, device=DEV, dtype=torch.float64)
        x = torch.view_as_complex(x.mul_(0.1))
        out.append((x + x.mH).contiguous())
    return out


def _network(case, seed):
    sizes = [case["n_in"]] + [case["width"]] * 3 + [case["n_out"]]
    rng = np.random.default_rng(seed)
    par = []
    for i, o in zip(sizes[:-1], sizes[1:]):
        a = math.sqrt(6.0 / (i + o))
        par += [rng.uniform(-a, a, size=i * o), np.zeros(o)]
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    X = torch.randn((case["rows"], sizes[0]), generator=g, device=DEV)
    Y = 0.2 * torch.randn((case["rows"], sizes[-1]), generator=g, device=DEV)
    return sizes, np.concatenate(par).astype(np.float32), X, Y


def _context(p):
    return T.Context(p["hop_R"], p["hop_t"], p["mu"], p["V0"], p["ff"], p["Lq"], p["n_ref"], p["cutoff"], p["prec"],
                     temperature=p["temperature"])


def prepare(case, seed):
    s = dict(case=case, op=case["op"])
    if case["op"] == "grad":
        sizes, par, X, Y = _network(case, seed)
        s.update(net=T.Mlp(sizes, par), X=X, Y=Y)
        s["grad"] = torch.empty(s["net"].n_params, device=DEV)
        return s
    if case["op"] == "batch":
        s["batch"] = T.Batch(_instances(case, seed), precision=case["prec"])
        shapes = [(d["Nq"], d["B"], d["B"]) for d in s["batch"].dims]
        s["P"] = [torch.empty(x, dtype=torch.complex128, device=DEV) for x in shapes]
        s["C"] = [torch.empty(x, dtype=torch.complex128, device=DEV) for x in shapes]
        return s
    p = _problem(case, seed)
    ctx = _context(p)
    s.update(ctx=ctx, lam=p["lam"])
    if case["op"] == "loops":
        n = 2 * ctx.Nq * ctx.n_dR
        s.update(n=n, Lc=torch.empty((2, ctx.Nq, ctx.n_dR, ctx.n_o ** 4), dtype=torch.complex128, device=DEV),
                 X=torch.empty((n, 11 + ctx.n_dR), device=DEV), Y=torch.empty((n, 2 * ctx.n_o ** 4), device=DEV))
        return s
    s["x"] = _state(3 if case["op"] == "su2" else 2, ctx.Nq, ctx.B, seed)
    s["y"] = [torch.empty_like(x) for x in s["x"]]
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _recorded(case, arrays):
    return list(arrays) if case["prec"] == "fp64" else [x.to(torch.complex64) for x in arrays]


def run(s):
    case, op = s["case"], s["op"]
    if op == "grad":
        return dict(loss=T.tufrg_mlp_loss_grad(s["net"], s["X"], s["Y"], s["grad"]), grad=s["grad"])
    if op == "batch":
        for x in s["P"] + s["C"]:
            x.zero_()
        r = T.tufrg_batch_flow(s["batch"], s["P"], s["C"], 1.0, 0.5, case["steps"])
        return dict(PC=_recorded(case, s["P"] + s["C"]), n_steps=[x["n_steps"] for x in r])
    if op == "loops":
        T.tufrg_loops_compact(s["ctx"], s["lam"], 1, s["Lc"])
        scale = T.tufrg_sur_targets(s["ctx"], s["n"], 1.0, s["Lc"], s["Y"])
        T.tufrg_sur_features(s["ctx"], s["n"], s["lam"], s["X"])
        T.tufrg_sur_targets(s["ctx"], s["n"], scale, s["Lc"], s["Y"])
        return dict(X=s["X"], Y=s["Y"])
    if op == "flow":
        P, C = s["y"]
        P.zero_()
        C.zero_()
        r = T.tufrg_flow(s["ctx"], P, C, 5.0, 0.2, n_steps=case["steps"])
        return dict(P=P, C=C, max_coupling=r["max_coupling"], n_steps=r["n_steps"])
    if op == "su2":
        T.tufrg_su2_rhs(s["ctx"], s["lam"], *s["x"], *s["y"])
        return list(s["y"])
    if op == "project":
        T.tufrg_project(s["ctx"], *s["x"], *s["y"])
        return list(s["y"])
    T.tufrg_rhs(s["ctx"], s["lam"], *s["x"], *s["y"])
    return _recorded(case, s["y"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _differences(S):
    s = _SHELL[:S]
    return sorted({(a[0] - b[0], a[1] - b[1]) for a in s for b in s})


def _loop_work(n_o, S, L, n_ref):
    """Both channels: per (q, k) the block of U distinct entries (one of each Hermitian pair, a
    complex product of n_o bands) and its separable Fourier sum; one of k and q -+ k suffices."""
    U = (n_o ** 4 + n_o ** 2) / 2
    n_dy = len({d[1] for d in _differences(S)})
    Nf = (L * n_ref) ** 2
    return dict(bytes=8.0 * Nf * (n_o + n_o ** 3) + 32.0 * L * L * len(_differences(S)) * n_o ** 4,
                flops=L * L * Nf * U * 8.0 * (n_o + n_dy))


def _state_work(n_o, S, L, products):
    B = S * n_o ** 2
    n_dx = len({d[0] for d in _differences(S)})
    return dict(bytes=4 * 16.0 * L * L * B * B, flops=L * L * (2 * 2 * 8.0 * n_dx * B * B + products * 8.0 * B ** 3))


def _add(*ws):
    return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}


def work(case):
    op = case["op"]
    if op == "grad":
        s = [case["n_in"]] + [case["width"]] * 3 + [case["n_out"]]
        n = sum(a * b for a, b in zip(s[:-1], s[1:]))
        return dict(bytes=4.0 * (case["rows"] * (s[0] + s[-1]) + 2 * n), flops=6.0 * case["rows"] * n)
    if op == "batch":
        ws = []
        for i in range(case["n"]):
            S, L = (5, 9, 13)[i % 3], (16, 24, 32)[(i // 3) % 3]
            ws += [_loop_work(2, S, L, case["n_ref"]), _state_work(2, S, L, 4)] * case["steps"]
        return _add(*ws)
    n_o = {"hubbard": 2, "rashba": 2, "hubbard1": 1}.get(case["model"], 6)
    S, L = case["S"], case["L"]
    loops = _loop_work(n_o, S, L, case["n_ref"])
    if op == "loops":
        rows = 2 * L * L * len(_differences(S))
        return dict(bytes=8.0 * (L * case["n_ref"]) ** 2 * (n_o + n_o ** 3)
                    + 4.0 * rows * (2 * n_o ** 4 + 11 + len(_differences(S))), flops=loops["flops"])
    if op == "project":
        return _state_work(n_o, S, L, 0)
    if op == "su2":
        w = _state_work(1, S, L, 8)
        return _add(loops, dict(bytes=1.5 * w["bytes"], flops=1.5 * w["flops"]))
    return _add(*[loops, _state_work(n_o, S, L, 4)] * case.get("steps", 1))


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch and numpy
# ---------------------------------------------------------------------------

_GX, _GW = np.polynomial.legendre.leggauss(8)


def _sech2(x):
    s = torch.exp(-2.0 * x.abs())
    return 4.0 * s / (1.0 + s) ** 2


def _g(e, lam, scheme):
    """K = dJ/dLambda (temperature, Omega) or J at fixed T (the shell's bubbles)."""
    if scheme == "shell":
        return 0.5 * torch.tanh(e / (2.0 * lam))
    if scheme == "temperature":
        return -e / (4.0 * lam ** 2) * _sech2(e / (2.0 * lam))
    a = e.abs()
    return -e * (3.0 * a + lam) / (4.0 * (a + lam) ** 3)


def _dg(e, lam, scheme):
    x = e / (2.0 * lam)
    if scheme == "shell":
        return 0.25 / lam * _sech2(x)
    if scheme == "temperature":
        return -(1.0 - 2.0 * x * torch.tanh(x)) / (4.0 * lam ** 2) * _sech2(x)
    a = e.abs()
    return (3.0 * e * e - 4.0 * a * lam - lam * lam) / (4.0 * (a + lam) ** 4)


def _divided(x, y, lam, scheme):
    """(g(x) - g(y)) / (x - y); the mean of g' where x is close to y (in two parts where 0 lies between)."""
    x, y = torch.broadcast_tensors(x, y)
    d = x - y
    near = d.abs() <= 1e-2 * lam
    out = (_g(x, lam, scheme) - _g(y, lam, scheme)) / torch.where(near, 1.0, d)
    a, b = x[near], y[near]

    def mean(u, v):
        return sum(0.5 * w * _dg(0.5 * (u + v) + 0.5 * t * (v - u), lam, scheme) for t, w in zip(_GX, _GW))

    if a.numel():
        w = a.abs() / (a.abs() + b.abs()).clamp_min(1e-300)
        z = torch.zeros_like(a)
        out[near] = torch.where(a * b < 0, w * mean(a, z) + (1.0 - w) * mean(z, b), mean(a, b))
    return out


class _Exact:
    def __init__(self, p):
        self.p, self.n, self.L = p, p["n_o"], p["Lq"]
        self.Lf, self.S = p["Lq"] * p["n_ref"], [tuple(int(v) for v in r) for r in p["ff"]]
        self.D = sorted({(a[0] - b[0], a[1] - b[1]) for a in self.S for b in self.S})
        k = np.arange(self.Lf)
        kx, ky = (v.ravel() for v in np.meshgrid(k, k, indexing="ij"))
        H = np.zeros((self.Lf ** 2, self.n, self.n), dtype=np.complex128)
        for R, t in zip(p["hop_R"], p["hop_t"]):
            H += np.exp(2j * np.pi * ((kx * int(R[0]) + ky * int(R[1])) % self.Lf) / self.Lf)[:, None, None] * t
        E, U = np.linalg.eigh(H)
        self.e = torch.from_numpy(E - p["mu"]).to(DEV)
        U = torch.from_numpy(U).to(DEV)
        # Pi[k][m][a c]
        self.Pi = (U.transpose(1, 2)[:, :, :, None] * U.conj().transpose(1, 2)[:, :, None, :]).reshape(-1, self.n, self.n ** 2)
        self.kx, self.ky = torch.from_numpy(kx).to(DEV), torch.from_numpy(ky).to(DEV)
        self.phases = {}
        q = np.arange(self.L)
        self.qx, self.qy = (torch.from_numpy(v.ravel()).to(DEV) for v in np.meshgrid(q, q, indexing="ij"))

    def phase(self, R):
        """e^{i q.R} on the coarse mesh."""
        if R not in self.phases:
            x = (self.qx * R[0] + self.qy * R[1]) % self.L
            self.phases[R] = torch.exp(2j * math.pi * x.to(torch.complex128) / self.L)
        return self.phases[R]

    def loops(self, lam):
        """Compact loops [2][Nq][n_dR][a b c d]: sum over k of e^{-ik.dR} Pi_m(k)_ac X_n(k')_bd L_mn / Nf, with
        k' = q - k and X = Pi (particle-particle) or k' = k - q and X = Pi^T."""
        n, Nf, Nq, nD = self.n, self.Lf ** 2, self.L ** 2, len(self.D)
        ph = torch.stack([torch.exp(-2j * math.pi * ((self.kx * d[0] + self.ky * d[1]) % self.Lf).to(torch.complex128)
                                    / self.Lf) for d in self.D])
        A = (ph[:, None, :, None] * self.Pi.permute(2, 0, 1)[None]).reshape(nD * n * n, Nf * n) / Nf
        out = torch.empty((2, Nq, nD, n, n, n, n), dtype=torch.complex128, device=DEV)
        step = max(1, min(Nq, int(1e8) // (Nf * n ** 3)))
        scheme, p = self.p["cutoff"], self.p
        if scheme == "shell":
            e2 = self.e ** 2
            chi, dchi = e2 / (e2 + lam ** 2), -2.0 * lam * e2 / (e2 + lam ** 2) ** 2
        for ch in (0, 1):
            s = 1 if ch == 0 else -1
            X = self.Pi if ch == 0 else self.Pi.reshape(Nf, n, n, n).transpose(2, 3).reshape(Nf, n, n * n)
            for q0 in range(0, Nq, step):
                cx, cy = (v[q0:q0 + step] * p["n_ref"] for v in (self.qx, self.qy))
                nq = cx.numel()
                kp = (s * (cx - self.kx[:, None])) % self.Lf * self.Lf + (s * (cy - self.ky[:, None])) % self.Lf  # [k][q]
                Lmn = s * _divided(self.e[:, :, None, None], -s * self.e.t()[:, kp].permute(1, 0, 2)[:, None],
                                   p["temperature"] if scheme == "shell" else lam, scheme)  # [k][m][n][q]
                if scheme == "shell":
                    cp, dp = (v.t()[:, kp].permute(1, 0, 2)[:, None] for v in (chi, dchi))
                    Lmn = Lmn * (dchi[:, :, None, None] * cp + chi[:, :, None, None] * dp)
                W = torch.zeros((Nf, n, nq, n * n), dtype=torch.complex128, device=DEV)
                for j in range(n):
                    W.addcmul_(Lmn[:, :, j, :, None].to(torch.complex128), X[:, j][kp][:, None])
                r = (A @ W.reshape(Nf * n, nq * n * n)).reshape(nD, n, n, nq, n, n)  # dR a c q b d
                out[ch, q0:q0 + nq] = r.permute(3, 0, 1, 4, 2, 5)
        return out.reshape(2, Nq, nD, n ** 4)

    def full(self, Lc):
        """[Nq][B][B] of one channel's compact loops."""
        n, at = self.n, {d: i for i, d in enumerate(self.D)}
        S = self.S
        idx = torch.tensor([[at[(a[0] - b[0], a[1] - b[1])] for b in S] for a in S], device=DEV)
        x = Lc.reshape(-1, len(self.D), n * n, n * n)[:, idx]  # q R R' ab cd
        return x.permute(0, 1, 3, 2, 4).reshape(x.shape[0], len(S) * n * n, -1)

    # the tensors X[q][R][R'][n1][n2][n3][n4] of P (rows n1 n2, columns n4 n3) and C (rows n1 n3, columns n4 n2)
    def _tensor(self, M, kind):
        n, f = self.n, len(self.S)
        return M.reshape(-1, f, n, n, f, n, n).permute(*((0, 1, 4, 2, 3, 6, 5) if kind == "P" else (0, 1, 4, 2, 6, 3, 5)))

    def _matrix(self, X, kind):
        B = len(self.S) * self.n ** 2
        return X.permute(*((0, 1, 3, 4, 2, 6, 5) if kind == "P" else (0, 1, 3, 5, 2, 6, 4))).reshape(-1, B, B)

    def real(self, X):
        return {d: torch.tensordot(self.phase(d), X, 1) / self.L ** 2 for d in self.D}

    def cross(self, real, which):
        """Generator of (i, j, term) of one cross projection; see the header's Sec. 3.3 passages."""
        at = {r: i for i, r in enumerate(self.S)}
        for i, R in enumerate(self.S):
            for j, Q in enumerate(self.S):
                if which == "CD":
                    for b, r in enumerate(self.S):
                        a = at.get((R[0] - Q[0] + r[0], R[1] - Q[1] + r[1]))
                        if a is not None:
                            yield i, j, self.phase(r), real[(-Q[0], -Q[1])][a, b]
                    continue
                sg = -1 if which == "PD" else 1
                for r in self.D:
                    a = at.get((R[0] + r[0], R[1] + r[1]))
                    b = at.get((sg * Q[0] - r[0], sg * Q[1] - r[1]))
                    if a is not None and b is not None:
                        ph = self.phase((r[0] + Q[0], r[1] + Q[1])) if which == "PD" else self.phase(r)
                        yield i, j, ph, real[r][a, b]

    def _added(self, X, terms, sign=1, swap=False):
        for i, j, ph, x in terms:
            x = x.transpose(-1, -2) if swap else x
            X[:, i, j] += sign * ph.reshape((-1,) + (1,) * x.dim()) * x[None]

    def project(self, P, C):
        P, C = self._tensor(P, "P"), self._tensor(C, "C")
        V0 = torch.from_numpy(self.p["V0"]).to(DEV)
        Pr, Cr = self.real(P), self.real(C)
        VP, VC = P.clone(), C.clone()
        VP[:, 0, 0] += V0
        VC[:, 0, 0] += V0
        self._added(VP, self.cross(Cr, "PC"))
        self._added(VP, self.cross(Cr, "PD"), -1, True)
        self._added(VC, self.cross(Pr, "PC"))
        self._added(VC, self.cross(Cr, "CD"), -1, True)
        return self._matrix(VP, "P"), self._matrix(VC, "C")

    def rhs(self, lam, P, C, Lc=None):
        VP, VC = self.project(P, C)
        Lc = self.loops(lam) if Lc is None else Lc
        return VP @ (self.full(Lc[0]) @ VP), 2.0 * (VC @ (self.full(Lc[1]) @ VC))

    def flow(self, lam0, lam1, n):
        B = len(self.S) * self.n ** 2
        P = torch.zeros((self.L ** 2, B, B), dtype=torch.complex128, device=DEV)
        C = P.clone()
        grid = lam0 * (lam1 / lam0) ** (np.arange(n + 1) / n)
        for a, b in zip(grid[:-1], grid[1:]):
            dP, dC = self.rhs(float(a), P, C)
            P, C = P + (b - a) * dP, C + (b - a) * dC
        return P, C

    def su2(self, lam, p, c, d):
        at = {r: i for i, r in enumerate(self.S)}
        neg = [at[(-r[0], -r[1])] for r in self.S]
        ph = torch.stack([self.phase(r) for r in self.S], 1)[:, None, :]
        x = lambda m: ph * m[:, :, neg]  # noqa: E731
        v = complex(self.p["V0"].ravel()[0])
        rp, rx, rc, rd = (self.real(m) for m in (p, x(p), c, d))
        a, cc, dd = p.clone(), c.clone(), d.clone()
        for m in (a, cc, dd):
            m[:, 0, 0] += v
        self._added(a, self.cross(rc, "PC"))
        self._added(a, self.cross(rd, "PD"))
        self._added(cc, self.cross(rp, "PC"))
        self._added(cc, self.cross(rd, "CD"))
        self._added(dd, self.cross(rx, "PC"))
        self._added(dd, self.cross(rc, "CD"))
        Lc = self.loops(lam)
        pp, ph_ = self.full(Lc[0]), self.full(Lc[1])
        ax = x(a)
        return [-(a @ pp @ ax + ax @ pp @ a), 2.0 * (2.0 * cc @ ph_ @ cc - cc @ ph_ @ dd - dd @ ph_ @ cc),
                -2.0 * dd @ ph_ @ dd]


def _exact_targets(ex, lam):
    Lc = ex.loops(lam)
    n, Nq, nD = ex.n, ex.L ** 2, len(ex.D)
    Y = torch.view_as_real(Lc).reshape(2 * Nq * nD, 2 * n ** 4)
    Y = Y / Lc.abs().max()
    qx, qy = (2.0 * math.pi * v.to(torch.float64) / ex.L for v in (ex.qx, ex.qy))
    f = torch.stack([qx.sin(), qx.cos(), qy.sin(), qy.cos(), (2 * qx).sin(), (2 * qx).cos(), (2 * qy).sin(),
                     (2 * qy).cos(), torch.full_like(qx, math.log(lam) / 5.0)], 1)
    X = torch.zeros((2, Nq, nD, 11 + nD), dtype=torch.float64, device=DEV)
    X[..., :9] = f[None, :, None]
    X[0, ..., 9] = 1.0
    X[1, ..., 10] = 1.0
    X[..., 11:] = torch.eye(nD, dtype=torch.float64, device=DEV)
    return dict(X=X.reshape(2 * Nq * nD, -1), Y=Y)


def exact(case, seed):
    op = case["op"]
    if op == "grad":
        sizes, par, X, Y = _network(case, seed)
        w = torch.from_numpy(par).to(DEV).double().requires_grad_()
        at, h = 0, X.double()
        for l, (i, o) in enumerate(zip(sizes[:-1], sizes[1:])):
            h = h @ w[at:at + i * o].reshape(o, i).t() + w[at + i * o:at + i * o + o]
            at += i * o + o
            h = torch.nn.functional.gelu(h) if l < len(sizes) - 2 else h
        loss = ((h - Y.double()) ** 2).mean()
        loss.backward()
        return dict(loss=float(loss.detach()), grad=w.grad)
    if op == "batch":
        r = [_Exact(p).flow(1.0, 0.5, case["steps"]) for p in _instances(case, seed)]
        return dict(PC=[x for x, _ in r] + [x for _, x in r], n_steps=[None] * case["n"])
    # the loops of the largest six-orbital meshes take minutes in this form
    n_o = {"hubbard": 2, "rashba": 2, "hubbard1": 1}.get(case["model"], 6)
    if op != "project" and n_o == 6 and case["L"] ** 4 * case["n_ref"] ** 2 > 3e7:
        return None
    p = _problem(case, seed)
    ex = _Exact(p)
    if op == "loops":
        return _exact_targets(ex, p["lam"])
    if op == "flow":
        P, C = ex.flow(5.0, 0.2, case["steps"])
        return dict(P=P, C=C, max_coupling=max(float(P.abs().max()), float(C.abs().max())), n_steps=None)
    x = _state(3 if op == "su2" else 2, ex.L ** 2, len(ex.S) * ex.n ** 2, seed)
    if op == "su2":
        return ex.su2(p["lam"], *x)
    if op == "project":
        return list(ex.project(*x))
    return list(ex.rhs(p["lam"], *x))
