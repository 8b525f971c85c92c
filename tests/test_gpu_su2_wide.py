"""The SU(2)-reduced right-hand side with every form factor of |R_x|, |R_y| <= 2 (25, 81
difference vectors), the most that the library takes, against the oracle."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import su2  # noqa: E402
from oracle import tufrg as otu  # noqa: E402


@pytest.mark.parametrize("cutoff", ["temperature", "omega"])
def test_reduced_rhs_with_25_form_factors(cutoff):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg as T
    print(f"su2 rhs: S25 {cutoff}", flush=True)
    r = range(-2, 3)
    ff = np.array([(0, 0)] + [(x, y) for x in r for y in r if (x, y) != (0, 0)], dtype=np.int32)
    R = np.array([[1, 0], [-1, 0], [0, 1], [0, -1], [1, 1], [-1, -1]], dtype=np.int32)
    t = np.array([-1, -1, -1, -1, 0.25, 0.25], dtype=np.complex128).reshape(-1, 1, 1)
    V0 = np.full((1, 1, 1, 1), 1.5, dtype=np.complex128)
    args = (R, t, -0.6, V0, ff, 9, 2, cutoff)
    st, ctx = otu.TUSetup(*args), T.Context(*args, "fp64")
    rng = np.random.default_rng(3)
    x = [rng.standard_normal((81, 25, 25)) + 1j * rng.standard_normal((81, 25, 25)) for _ in range(3)]
    out = [torch.zeros((81, 25, 25), dtype=torch.complex128, device="cuda") for _ in range(3)]
    T.tufrg_su2_rhs(ctx, 0.4, *[torch.from_numpy(v).cuda() for v in x], *out)
    for got, ref in zip(out, su2.rhs(st, 0.4, *x)):
        # the bar of the narrower sets
        assert np.abs(got.cpu().numpy() - ref).max() < 1e-11 * np.abs(ref).max()
    ctx.close()
