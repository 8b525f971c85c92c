"""Relabellings of the loop sum that the library's loop kernels use to leave
half (with time reversal three quarters) of the points out.

CPU: the oracle's loops obey them, for models with and without time reversal.
GPU: the loops of models with either time reversal (real hoppings; i sigma_y in
each orbital), of models without, and in the band basis, on even and odd coarse
and fine meshes (rows that are their own partners or not; coarse q equal to
their negative or not), against the oracle at the bars of the arithmetic."""

import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

from oracle import tufrg as otu  # noqa: E402
from synth import PAULI, ff_shell, hubbard_hoppings, kanamori_V0, onsite_V0, rashba_hoppings, t2g_soc_hoppings  # noqa: E402
from tests._layout import ph_loop_to_matrix, pp_loop_to_matrix  # noqa: E402


def _onsite(hop, m):
    """hop with the onsite matrix m added."""
    R, t = hop
    return np.concatenate([np.asarray(R), [[0, 0]]]).astype(np.int32), np.concatenate([t, m[None]])


def _bonds(n_o, seed):
    """Random complex Hermitian hoppings: no symmetry at all."""
    rng = np.random.default_rng(seed)
    R, t = [], []
    for r in ((1, 0), (0, 1), (1, 1)):
        m = rng.standard_normal((n_o, n_o)) + 1j * rng.standard_normal((n_o, n_o))
        R += [r, (-r[0], -r[1])]
        t += [m, m.conj().T]
    return np.array(R, dtype=np.int32), 0.4 * np.array(t)


def _quaternionic(seed):
    """Random hoppings with time reversal times inversion and neither alone:
    H(k) real in the 15 Hermitian 6 x 6 matrices that commute with T K."""
    rng = np.random.default_rng(seed)
    one, isg = np.eye(2), [1j * p for p in PAULI]
    Q = [np.kron(np.diag(np.eye(3)[i]), one).astype(np.complex128) for i in range(3)]
    for i, j in ((0, 1), (0, 2), (1, 2)):
        e = np.zeros((3, 3))
        e[i, j] = 1.0
        Q += [np.kron(e + e.T, one)] + [np.kron(e - e.T, g) for g in isg]
    R, t = [(0, 0)], [np.tensordot(rng.standard_normal(15), np.array(Q), 1)]
    for r in ((1, 0), (0, 1), (1, 1), (1, -1)):
        m = np.tensordot(rng.standard_normal(15) + 1j * rng.standard_normal(15), np.array(Q), 1)
        R += [r, (-r[0], -r[1])]
        t += [m, m.conj().T]
    return np.array(R, dtype=np.int32), 0.3 * np.array(t)


# name -> (hoppings, kind of time reversal: 0 none, 1 T = 1, 2 T = i sigma_y)
MODELS = {
    "hubbard": (hubbard_hoppings(), 1),
    "rashba": (rashba_hoppings(1.0, 0.3), 2),
    "rashba in a field": (_onsite(rashba_hoppings(1.0, 0.3), 0.2 * PAULI[2]), 0),
    "random2": (_bonds(2, 4), 0),
    "t2g": (t2g_soc_hoppings(0.2, seed=1), 2),
    "t2g in a field": (_onsite(t2g_soc_hoppings(0.2, seed=1), 0.05 * np.kron(np.eye(3), PAULI[2])), 0),
    "random6": (_bonds(6, 5), 0),
    "quaternionic": (_quaternionic(7), 0),
}


def _setup(model, S, Lq, n_ref, cutoff, basis="orbital"):
    hop = MODELS[model][0]
    n_o = hop[1].shape[1]
    V0 = onsite_V0(2.0) if n_o == 2 else kanamori_V0(2.0, 0.3)
    T = 0.06 if cutoff == "shell" else None
    return dict(hop=hop, V0=V0, ff=ff_shell(S), Lq=Lq, n_ref=n_ref, cutoff=cutoff, temperature=T, basis=basis, n_o=n_o,
                mu=-0.3)


def _oracle(c):
    return otu.TUSetup(*c["hop"], c["mu"], c["V0"], c["ff"], c["Lq"], c["n_ref"], c["cutoff"],
                       temperature=c["temperature"], basis=c["basis"])


def _compact(c, M):
    """[q][dR] -> n_o^4 entries (a, b, c, d) of the matrix form M [q][B][B]."""
    n, ff = c["n_o"], [tuple(int(v) for v in r) for r in c["ff"]]
    X = M.reshape(-1, len(ff), n, n, len(ff), n, n)
    return {(a[0] - b[0], a[1] - b[1]): X[:, i, :, :, j] for i, a in enumerate(ff) for j, b in enumerate(ff)}


@pytest.mark.parametrize("model", ["hubbard", "rashba", "rashba in a field", "random2", "t2g", "random6", "quaternionic"])
@pytest.mark.parametrize("Lq,n_ref", [(5, 1), (6, 2)])
def test_the_oracle_loops_obey_the_relabellings(model, Lq, n_ref):
    c = _setup(model, 5, Lq, n_ref, "temperature")
    st, kind = _oracle(c), MODELS[model][1]
    n = c["n_o"]
    q = np.arange(Lq * Lq)
    qx, qy = q // Lq, q % Lq
    neg = (-qx % Lq) * Lq + (-qy % Lq)
    bar = np.arange(n) ^ 1 if kind == 2 else np.arange(n)
    t = (-1.0) ** np.arange(n) if kind == 2 else np.ones(n)
    sgn = np.einsum("a,b,c,d->abcd", t, t, t, t)
    for ch, to in (("pp", pp_loop_to_matrix), ("ph", ph_loop_to_matrix)):
        L = _compact(c, to(otu.loops(st, ch, 0.3)))
        for d, X in L.items():
            ph = np.exp(2j * np.pi * (qx * d[0] + qy * d[1]) / Lq)[:, None, None, None, None]
            rev = X.transpose(0, 4, 3, 2, 1)
            tol = 1e-12 * np.abs(X).max() + 1e-15
            if ch == "pp":  # the sum over the other half of the points completes the sum
                assert np.abs(X - ph.conj() * rev.conj()).max() < tol
            else:
                assert np.abs(X[neg] - ph * rev).max() < tol
            if kind:
                B = sgn * X[:, bar][:, :, bar][:, :, :, bar][:, :, :, :, bar].conj()
                assert np.abs(X[neg] - B).max() < tol
                if ch == "ph":
                    assert np.abs(X - ph.conj() * B.transpose(0, 4, 3, 2, 1)).max() < tol


BAR = {"fp64": 1e-10, "fp32": 1e-5, "bf16x3": 1e-4}
CASES = [("hubbard", 5, 6, 3, "temperature", "fp64"), ("hubbard", 9, 5, 3, "omega", "fp32"),
         ("rashba", 9, 7, 11, "omega", "fp64"), ("rashba", 13, 9, 2, "shell", "fp32"),
         ("rashba in a field", 9, 6, 4, "temperature", "fp64"), ("rashba in a field", 5, 5, 13, "shell", "fp32"),
         ("random2", 13, 10, 1, "omega", "fp64"), ("random2", 5, 8, 12, "temperature", "fp32"),
         ("t2g", 9, 5, 3, "temperature", "fp64"), ("t2g", 5, 6, 3, "shell", "bf16x3"),
         ("t2g in a field", 9, 6, 2, "omega", "fp32"), ("t2g in a field", 5, 7, 3, "temperature", "bf16x3"),
         # 15 real coordinates per pair sum: tiles of 32 ky (one short, one and a bit, two whole), groups of 16 q
         ("t2g", 5, 5, 2, "omega", "bf16x3"), ("t2g", 13, 9, 4, "temperature", "bf16x3"),
         ("t2g", 5, 5, 8, "shell", "bf16x3"), ("t2g", 9, 8, 8, "omega", "bf16x3"),
         ("quaternionic", 9, 6, 3, "temperature", "bf16x3"), ("quaternionic", 5, 5, 8, "shell", "bf16x3"),
         ("quaternionic", 9, 5, 3, "omega", "bf16x3"), ("quaternionic", 5, 6, 3, "temperature", "fp64"),
         ("random6", 5, 5, 3, "temperature", "fp64"), ("random6", 9, 6, 3, "omega", "bf16x3")]


@pytest.mark.gpu
@pytest.mark.parametrize("model,S,Lq,n_ref,cutoff,prec", CASES)
@pytest.mark.parametrize("basis", ["orbital", "band"])
def test_loops_against_the_oracle(model, S, Lq, n_ref, cutoff, prec, basis):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg as T
    if basis == "band" and (model, prec, n_ref) not in (("rashba", "fp64", 11), ("t2g", "fp64", 3), ("random2", "fp32", 12),
                                                        ("t2g", "bf16x3", 3)):
        pytest.skip("the band basis once per kernel")
    c = _setup(model, S, Lq, n_ref, cutoff, basis)
    print(f"loop symmetry: {model} S{S} {Lq}x{Lq} refined {n_ref}x {cutoff} {prec} {basis}", flush=True)
    ctx = T.Context(*c["hop"], c["mu"], c["V0"], c["ff"], Lq, n_ref, cutoff, prec, temperature=c["temperature"],
                    basis=basis)
    st = _oracle(c)
    both = torch.empty((2, ctx.Nq, ctx.n_dR, ctx.n_o ** 4), dtype=torch.complex128, device="cuda")
    T.tufrg_loops_compact(ctx, 0.4, 1, both)
    for ch, name, to in ((T.PP, "pp", pp_loop_to_matrix), (T.PH, "ph", ph_loop_to_matrix)):
        L = torch.empty((ctx.Nq, ctx.B, ctx.B), dtype=torch.complex128, device="cuda")
        T.tufrg_bubble(ctx, ch, 0.4, 1, L)
        got, ref = L.cpu().numpy(), to(otu.loops(st, name, 0.4))
        err = np.abs(got - ref).max() / np.abs(ref).max()
        print(name, f"{err:.2e}", flush=True)
        assert err < BAR[prec]
        # one channel alone is that channel of both
        dR = [tuple(r) for r in T.tufrg_dR(ctx)]
        X = _compact(c, got)
        for i, d in enumerate(dR):
            assert np.array_equal(both[ch, :, i].cpu().numpy(), X[d].reshape(ctx.Nq, -1))
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("Lq,n_ref,S", [(6, 3, 5), (7, 10, 9), (10, 7, 13), (16, 4, 9)])
@pytest.mark.parametrize("cutoff", ["temperature", "omega"])
@pytest.mark.parametrize("kind", ["real", "complex"])
def test_one_orbital_loops_against_the_oracle(Lq, n_ref, S, cutoff, kind):
    """The one-band kernel with time reversal (real hoppings) and without."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg as T
    hop = _bonds(1, 6)
    if kind == "real":
        hop = (hop[0], hop[1].real.astype(np.complex128))
    V0 = np.full((1, 1, 1, 1), 1.0, dtype=np.complex128)
    print(f"one-orbital loops: {Lq}x{Lq} refined {n_ref}x S{S} {cutoff} {kind}", flush=True)
    ctx = T.Context(*hop, 0.1, V0, ff_shell(S), Lq, n_ref, cutoff, "fp64")
    st = otu.TUSetup(*hop, 0.1, V0, ff_shell(S), Lq, n_ref, cutoff)
    for ch, name in ((T.PP, "pp"), (T.PH, "ph")):
        L = torch.empty((ctx.Nq, ctx.B, ctx.B), dtype=torch.complex128, device="cuda")
        T.tufrg_bubble(ctx, ch, 0.4, 1, L)
        ref = otu.loops(st, name, 0.4).reshape(L.shape)
        assert np.abs(L.cpu().numpy() - ref).max() < 1e-10 * np.abs(ref).max()
    ctx.close()
