"""An Euler step's update, maximum and non-finite flag against torch.

One workgroup (a mesh of one point), a ragged last one, and more elements than
the 512 workgroups have threads.  Two steps in a row: the second finds the
accumulators of the first cleared.  Tolerance: the update is one FP64 fused
multiply-add per real number, the maximum one square root; a few ulp, 1e-15 of
the largest entry.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import ff_shell, hubbard_hoppings, onsite_V0  # noqa: E402

ONE = np.array([(0, 0)])


@pytest.mark.parametrize("ff,Lq", [(ONE, 1), (ff_shell(5), 6), (ff_shell(9), 12)])
def test_step_and_maximum(ff, Lq):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg as T
    hop = hubbard_hoppings(1.0, -0.25)
    ctx = T.Context(hop[0], hop[1], -0.6, onsite_V0(3.0), np.asarray(ff), Lq, 2, "temperature", "fp64")
    g = torch.Generator().manual_seed(5)
    P, C = (torch.view_as_complex(torch.randn(ctx.Nq, ctx.B, ctx.B, 2, generator=g, dtype=torch.float64)).cuda() * s
            for s in (0.02, 0.01))
    for l0, l1 in ((0.9, 0.8), (0.8, 0.75)):
        dP, dC = torch.empty_like(P), torch.empty_like(C)
        T.tufrg_rhs(ctx, l0, P, C, dP, dC)
        refP, refC = P + (l1 - l0) * dP, C + (l1 - l0) * dC
        res = T.tufrg_flow(ctx, P, C, l0, l1, n_steps=1, v_max=1e9)
        torch.cuda.synchronize()
        big = max(refP.abs().max().item(), refC.abs().max().item())
        assert (P - refP).abs().max().item() <= 1e-15 * big and (C - refC).abs().max().item() <= 1e-15 * big
        assert abs(res["max_coupling"] - big) <= 1e-15 * big
        assert res["n_steps"] == 1
    C.view(-1)[-1] = float("nan")
    with pytest.raises(Exception, match="non-finite"):
        T.tufrg_flow(ctx, P, C, 0.75, 0.7, n_steps=1, v_max=1e9)
    ctx.close()
