"""Vector loops of six spin-orbitals at the edges of their ky tiles, and the
two-orbital loops at the end of a kx chunk, against the FP64 oracle.

Six orbitals: rows shorter than one tile (8 ky in FP64, 16 in FP32), of exactly
one and two tiles, with a remainder of one, with and without the pair sums, a
momentum shell, and chunks past the rows of an item.  Two orbitals: 64 ky a wave
(the contraction with the ky phases), one below, at and above, with the boxes of
difference vectors 1, 2 and 4.  Bars of the arithmetic as in the other loop tests.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import tufrg as otu  # noqa: E402
from tests._layout import ph_loop_to_matrix, pp_loop_to_matrix  # noqa: E402
from tests.test_loop_symmetry import BAR, _oracle, _setup  # noqa: E402

CASES = [("t2g", 5, 5, 1, "temperature", "fp64"), ("t2g", 5, 8, 1, "omega", "fp64"),
         ("t2g", 13, 9, 1, "temperature", "fp64"), ("random6", 13, 9, 2, "omega", "fp64"),
         ("random6", 5, 8, 2, "shell", "fp32"), ("t2g in a field", 9, 17, 1, "temperature", "fp32"),
         ("t2g", 9, 8, 4, "omega", "fp32"), ("random6", 13, 9, 1, "temperature", "fp32"),
         ("random2", 1, 7, 9, "temperature", "fp32"), ("random2", 5, 8, 8, "omega", "fp64"),
         ("rashba", 13, 13, 5, "temperature", "fp64"), ("random2", 9, 16, 8, "temperature", "fp32")]


@pytest.mark.parametrize("model,S,Lq,n_ref,cutoff,prec", CASES)
def test_loops_at_the_edges_of_the_tiles(model, S, Lq, n_ref, cutoff, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg as T
    c = _setup(model, max(S, 5), Lq, n_ref, cutoff)
    c["ff"] = np.asarray(c["ff"])[:1] if S == 1 else c["ff"]
    ctx = T.Context(c["hop"][0], c["hop"][1], c["mu"], c["V0"], c["ff"], Lq, n_ref, cutoff, prec,
                    temperature=c["temperature"])
    st, lam = _oracle(c), 0.3
    B = len(c["ff"]) * c["n_o"] ** 2
    for ch, name, to in ((T.PP, "pp", pp_loop_to_matrix), (T.PH, "ph", ph_loop_to_matrix)):
        out = torch.full((Lq * Lq, B, B), float("nan"), dtype=torch.complex128, device="cuda")
        T.tufrg_bubble(ctx, ch, lam, 1, out)
        torch.cuda.synchronize()
        ref = to(otu.loops(st, name, lam))
        assert np.abs(out.cpu().numpy() - ref).max() <= BAR[prec] * np.abs(ref).max()
    ctx.close()
