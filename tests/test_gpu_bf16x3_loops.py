"""BF16X3 loops of six spin-orbitals against the FP64 loops of the library (held
to the oracle elsewhere), at a bar that follows from the arithmetic: every kind
of kernel (six bands; pairs; pairs in 15 coordinates), with and without time
reversal, on both shapes of difference vectors, loops and bubbles.

A term of the k sum is off by at most 3 * 2^-18 (both operands split, the product
of the low parts dropped) plus 3e-6 (the FP32 quotient next to the switch to the
mean of the derivative).  Taken as independent uniform errors over the tenth of
the points that the peak of the loop kernel holds, five standard deviations of
the sum are 5 / sqrt(3 * 0.1 Lf^2) of that, relative to the largest entry."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import PAULI, ff_shell, kanamori_V0, t2g_soc_hoppings  # noqa: E402
from tests.test_loop_symmetry import MODELS  # noqa: E402

R, TT = t2g_soc_hoppings(0.2, seed=1)
SLOW = [0, 2, 4, 1, 3, 5]  # spin index slowest: bands paired, no pairing within an orbital to find
HOP = {"t2g": (R, TT), "t2g, spin slowest": (R, np.ascontiguousarray(TT[:, SLOW][:, :, SLOW])),
       "t2g in a field": MODELS["t2g in a field"][0], "quaternionic": MODELS["quaternionic"][0]}

# kind 0: six bands (no pairs, pairing off or an odd mesh)
CASES = [(0, "t2g in a field", 13, 9, 7, "temperature"), (0, "t2g in a field", 9, 16, 4, "omega"),
         (0, "t2g", 5, 9, 7, "shell"), (0, "t2g", 13, 9, 8, "omega"),
         (1, "t2g, spin slowest", 13, 9, 8, "temperature"), (1, "t2g, spin slowest", 9, 8, 8, "shell"),
         # one form factor: few final blocks, shared by several workgroups
         (0, "t2g in a field", 1, 4, 16, "omega"), (0, "t2g", 1, 3, 21, "temperature"),
         (1, "t2g, spin slowest", 1, 5, 12, "shell"), (2, "t2g", 1, 4, 16, "temperature"),
         # a last tile of 8, 10, 16 and 32 ky; 13 to 85 items in groups of 16; few final blocks and many
         (2, "t2g", 13, 9, 8, "temperature"), (2, "t2g", 5, 5, 14, "omega"), (2, "t2g", 9, 10, 10, "shell"),
         (2, "t2g", 9, 13, 6, "temperature"), (2, "quaternionic", 5, 5, 20, "shell"),
         (2, "quaternionic", 13, 9, 10, "omega"), (2, "quaternionic", 9, 8, 8, "temperature")]


@pytest.mark.parametrize("kind,model,S,Lq,n_ref,cutoff", CASES)
def test_loops_against_fp64(kind, model, S, Lq, n_ref, cutoff):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg as T
    print(f"bf16x3 loops: kind {kind} {model} S{S} {Lq}x{Lq} refined {n_ref}x {cutoff}", flush=True)
    Lf = Lq * n_ref
    bar = 5.0 * (3.0 * 2.0 ** -18 + 3e-6) / np.sqrt(3.0 * 0.1 * Lf * Lf)
    L = []
    # the random model's bands are three times as wide: a third of the points at the peak
    bar *= np.sqrt(3.0) if model == "quaternionic" else 1.0
    for prec in ("fp64", "bf16x3"):
        ctx = T.Context(*HOP[model], -0.3, kanamori_V0(2.0, 0.3), ff_shell(max(S, 5))[:S], Lq, n_ref, cutoff, prec,
                        temperature=0.1 if cutoff == "shell" else None)
        if prec == "bf16x3":
            assert T.tufrg_pair_bands(ctx, kind > 0) is (kind > 0)
        for deriv in (1, 0):
            x = torch.empty((2, ctx.Nq, ctx.n_dR, 6 ** 4), dtype=torch.complex128, device="cuda")
            T.tufrg_loops_compact(ctx, 0.4, deriv, x)
            L.append(x)
        torch.cuda.synchronize()
        ctx.close()
    for deriv, ref, got in ((1, L[0], L[2]), (0, L[1], L[3])):
        for ch in (0, 1):
            err = float((got[ch] - ref[ch]).abs().max() / ref[ch].abs().max())
            print(f"deriv {deriv} channel {ch}: {err:.2e}, bar {bar:.2e}", flush=True)
            assert err < bar


def test_switching_the_pairs_leaves_no_stale_operand():
    """Pairs off and on again, at another scale in between: the loops of a context that never switched."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg as T
    for cutoff in ("temperature", "shell"):
        print(f"bf16x3 loops: pairs switched, t2g S5 6x6 refined 4x {cutoff}", flush=True)
        ctx = [T.Context(R, TT, -0.3, kanamori_V0(2.0, 0.3), ff_shell(5), 6, 4, cutoff, "bf16x3",
                         temperature=0.1 if cutoff == "shell" else None) for _ in range(2)]
        x = [torch.empty((2, c.Nq, c.n_dR, 6 ** 4), dtype=torch.complex128, device="cuda") for c in ctx]
        T.tufrg_loops_compact(ctx[0], 0.7, 1, x[0])
        T.tufrg_pair_bands(ctx[0], False)
        T.tufrg_loops_compact(ctx[0], 0.5, 1, x[0])
        assert T.tufrg_pair_bands(ctx[0], True)
        for c, y in zip(ctx, x):
            T.tufrg_loops_compact(c, 0.4, 1, y)
        torch.cuda.synchronize()
        assert torch.equal(x[0], x[1])
        for c in ctx:
            c.close()
