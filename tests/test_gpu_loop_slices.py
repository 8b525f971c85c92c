"""Loops whose partial sums are taken in slices of the coarse q (one and six
spin-orbitals; the workspace is bounded): the values of every slice and of both
slots of an item, and the memory a context takes."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import PAULI, ff_shell, kanamori_V0, t2g_soc_hoppings  # noqa: E402


@pytest.fixture(scope="module")
def T():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg
    return tufrg


def _free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("kind", ["real", "complex"])
def test_one_orbital_slices(T, kind):
    """448 x 448, 13 form factors: without time reversal 301057 items of two chunks and
    seven ky blocks, 3.0 GB of partial sums in one piece; the workspace is 1 GB."""
    Lq, lam = 448, 0.5
    R = np.array([[1, 0], [-1, 0], [0, 1], [0, -1]], dtype=np.int32)
    z = 1.0 if kind == "real" else np.exp(0.3j)
    t = np.array([z, np.conj(z), 0.8, 0.8], dtype=np.complex128).reshape(-1, 1, 1)
    V0 = np.full((1, 1, 1, 1), 1.0, dtype=np.complex128)
    ff = ff_shell(13)
    print(f"one-orbital slices: {Lq}x{Lq} {kind}", flush=True)
    before = _free()
    ctx = T.Context(R, t, 0.2, V0, ff, Lq, 1, "temperature", "fp64")
    used = before - _free()
    Nq = Lq * Lq
    # compact loops (both channels), VP and VC, the bounded workspace, and 0.3 GB of tables
    assert used < 16 * (2 * Nq * 41 + 2 * Nq * 13 ** 2) + 2 ** 30 + 3e8
    L = torch.empty((2, ctx.Nq, ctx.n_dR, 1), dtype=torch.complex128, device="cuda")
    T.tufrg_loops_compact(ctx, lam, 1, L)
    dR = np.asarray(T.tufrg_dR(ctx)).reshape(-1, 2)
    k = 2 * np.pi * np.arange(Lq) / Lq
    e = sum(t[h, 0, 0] * np.exp(1j * (k[:, None] * R[h, 0] + k[None] * R[h, 1])) for h in range(4)).real - 0.2

    def K(x):
        return -x / (4 * lam ** 2) / np.cosh(x / (2 * lam)) ** 2

    ph = [np.exp(-1j * (k[:, None] * d[0] + k[None] * d[1])) for d in dR]
    i = np.arange(Lq)
    for q in (0, 1, 5 * Lq + 300, 149 * Lq + 77, 150 * Lq, Nq // 3, Nq // 2 + 3, 300 * Lq + 447, Nq - 1):
        qx, qy = divmod(q, Lq)
        for ch, s in ((0, 1), (1, -1)):
            ep = e[(s * (qx - i)) % Lq][:, (s * (qy - i)) % Lq]
            d = e + s * ep
            near = np.abs(d) < 1e-4
            m = 0.5 * (e - s * ep)  # both arguments of the divided difference
            h = 1e-4
            l = np.where(near, (K(m + h) - K(m - h)) / (2 * h), (K(e) - K(-s * ep)) / np.where(near, 1, d)) * s
            ref = np.array([(p * l).sum() for p in ph]) / Nq
            got = L[ch, q, :, 0].cpu().numpy()
            # the reference's own quotient next to its switch: 1e-16 / 1e-4 per term
            assert np.abs(got - ref).max() < 1e-8 * np.abs(ref).max(), (q, ch)
    ctx.close()


@pytest.mark.parametrize("model,prec", [("t2g", "fp64"), ("field", "fp64"), ("field", "fp32")])
def test_six_orbital_slices(T, model, prec):
    """20 x 20 refined 32x, 13 form factors: 402 items of 7 chunks (2.5 GB of partial
    sums) or 602 of 6 and 14 (3.1 and 3.7 GB), in two slices of each channel; against
    the BF16X3 kernels, which keep row buffers instead."""
    R, t = t2g_soc_hoppings(0.2, seed=1)
    if model == "field":
        R = np.concatenate([np.asarray(R), [[0, 0]]]).astype(np.int32)
        t = np.concatenate([t, 0.05 * np.kron(np.eye(3), PAULI[2])[None]])
    print(f"six-orbital slices: {model} S13 20x20 refined 32x {prec}", flush=True)
    out = []
    for p in (prec, "bf16x3"):
        ctx = T.Context(R, t, 0.35, kanamori_V0(2.0, 0.3), ff_shell(13), 20, 32, "omega", p)
        x = torch.empty((2, ctx.Nq, ctx.n_dR, 6 ** 4), dtype=torch.complex128, device="cuda")
        T.tufrg_loops_compact(ctx, 0.3, 1, x)
        torch.cuda.synchronize()
        out.append(x)
        ctx.close()
    for ch in (0, 1):
        assert float((out[0][ch] - out[1][ch]).abs().max() / out[0][ch].abs().max()) < 1e-5
