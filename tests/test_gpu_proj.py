"""The projection kernels at the edges of their splits, against the FP64 oracle.

Form-factor sets with no, two and four pairs of rho_y and up to 81 difference
vectors; 4, 16 and 64 matrix elements per workgroup with a ragged last block;
meshes of one point, below, at and above the eight loads in flight, and with
more rows than units.  Tolerance: a projected entry sums at most Nq n_D terms in
FP64, the oracle's in another order; 1e-12 of the largest entry.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import tufrg as otu  # noqa: E402
from synth import (ff_shell, hubbard_hoppings, kanamori_V0, onsite_V0, random_exchange_state,  # noqa: E402
                   t2g_soc_hoppings)
from tests._layout import c_to_matrix, p_to_matrix  # noqa: E402

ONE = np.array([(0, 0)])
XLINE = np.array([(0, 0), (1, 0), (-1, 0)])
YLINE = np.array([(0, 0), (0, 2), (0, -2)])
BOX = np.array([(0, 0)] + [(x, y) for x in range(-2, 3) for y in range(-2, 3) if (x, y) != (0, 0)])


@pytest.mark.parametrize("n_o,ff,Lq", [
    (2, ONE, 1), (2, ONE, 37), (2, XLINE, 5), (2, YLINE, 9), (2, ff_shell(5), 8),
    (2, BOX, 9), (2, BOX, 17), (6, ONE, 7), (6, ff_shell(5), 6), (6, ff_shell(9), 10)])
def test_projections_at_the_edges_of_the_splits(n_o, ff, Lq):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg as T
    hop = hubbard_hoppings(1.0, -0.25) if n_o == 2 else t2g_soc_hoppings(0.2, seed=1)
    V0 = onsite_V0(3.0) if n_o == 2 else kanamori_V0(2.0, 0.3)
    ff = np.asarray(ff)
    ctx = T.Context(hop[0], hop[1], -0.3, V0, ff, Lq, 1, "temperature", "fp64")
    st = otu.TUSetup(*hop, -0.3, V0, ff, Lq, 1, "temperature")
    P = random_exchange_state(st.Nq, st.n_ff, st.n_o, seed=3)
    C = random_exchange_state(st.Nq, st.n_ff, st.n_o, seed=4)
    dev = torch.device("cuda:0")
    Pd, Cd = torch.from_numpy(p_to_matrix(P)).to(dev), torch.from_numpy(c_to_matrix(C)).to(dev)
    VP, VC = torch.full_like(Pd, float("nan")), torch.full_like(Cd, float("nan"))
    T.tufrg_project(ctx, Pd, Cd, VP, VC)
    torch.cuda.synchronize()
    rVP, rVC = otu.projected_vertices(st, P, C)
    for got, ref in ((VP, p_to_matrix(rVP)), (VC, c_to_matrix(rVC))):
        assert np.abs(got.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
    ctx.close()
