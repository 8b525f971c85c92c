"""Targets of the surrogate and their largest magnitude: with and without block
lists, T on and off 16-byte boundaries, one workgroup and many, and what an
invalid block does to the maximum.  Oracle: NumPy on the same loops (the
targets are one FP64 product rounded to FP32: at most half an ulp away)."""

import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

pytestmark = pytest.mark.gpu

from synth import ff_shell, hubbard_hoppings, kanamori_V0, onsite_V0, t2g_soc_hoppings  # noqa: E402


@pytest.mark.parametrize("model,Lq", [("hubbard", 5), ("hubbard", 24), ("t2g", 9)])
@pytest.mark.parametrize("offset", [0, 1, 4])
@pytest.mark.parametrize("lists", [False, True])
def test_targets_and_their_maximum(model, Lq, offset, lists):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg as T
    hop, V0 = (hubbard_hoppings(), onsite_V0(2.0)) if model == "hubbard" else (t2g_soc_hoppings(0.2), kanamori_V0(2.0, 0.3))
    ctx = T.Context(*hop, 0.1, V0, ff_shell(5), Lq, 1, "omega", "fp32")
    n, no4 = 2 * ctx.Nq * ctx.n_dR, ctx.n_o ** 4
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    Lc = torch.view_as_complex(torch.randn((2, ctx.Nq, ctx.n_dR, no4, 2), generator=g, device="cuda", dtype=torch.float64))
    rows = Lc.reshape(n, no4)
    kw = {}
    if lists:
        b = torch.randperm(n, generator=g, device="cuda")[: max(1, n - 3)]
        kw = dict(q=(b // ctx.n_dR) % ctx.Nq, ch=b // (ctx.n_dR * ctx.Nq), iD=b % ctx.n_dR)
        kw = {k: v.to(torch.int32).contiguous() for k, v in kw.items()}
        rows, n = rows[b], len(b)
    buf = torch.full((n * 2 * no4 + offset,), 7.0, device="cuda")
    Y = buf[offset:]
    print(f"targets: {model} {Lq}x{Lq} offset {offset} lists {lists}", flush=True)
    big = T.tufrg_sur_targets(ctx, n, 0.7, Lc, Y, **kw)
    ref = torch.view_as_real(rows).reshape(-1).cpu().numpy() / 0.7
    got = Y.cpu().numpy()
    assert np.abs(got - ref).max() <= 2.0 ** -24 * np.abs(ref).max() + 1e-300
    assert big == float(np.abs(got).max()) * 0.7
    assert (buf[:offset] == 7.0).all()
    if lists and model == "t2g":
        kw["q"][1] = ctx.Nq  # whole runs of 64 NaN targets: the maximum is NaN
        assert np.isnan(T.tufrg_sur_targets(ctx, n, 0.7, Lc, Y, **kw))
        assert torch.isnan(Y.reshape(n, -1)[1]).all() and torch.isfinite(Y.reshape(n, -1)[2:]).all()
    elif lists:
        kw["q"][1] = -1  # 32 NaN targets: passed over
        assert np.isfinite(T.tufrg_sur_targets(ctx, n, 0.7, Lc, Y, **kw))
    ctx.close()
