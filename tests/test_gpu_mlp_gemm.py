"""The matrix-core products of the surrogate network at the edges of their
tiles (32 x 64, K steps of 64, split weight gradients from 512 rows): forward,
loss and gradient against the FP64 oracle, layer by layer.  The bound is that of
an FP32 sum of n terms with random rounding, a few sqrt(n) ulp of the largest
value: 1e-5 for the sums of at most 2600 terms here."""

import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

pytestmark = pytest.mark.gpu

from oracle import mlp as omlp  # noqa: E402
from synth import mlp_batch, mlp_init  # noqa: E402


def rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


@pytest.mark.parametrize("sizes", [[1, 1], [3, 5], [16, 64, 32], [17, 65, 33, 66], [52, 256, 256, 2592], [25, 200, 32]])
@pytest.mark.parametrize("n", [1, 31, 64, 513, 2048])
@pytest.mark.parametrize("shift", [0, 1])
def test_network_against_the_oracle(sizes, n, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if max(sizes) > 1000 and n not in (64, 513):
        pytest.skip("the wide network at two row counts")
    from paper_1710_08830_amd import tufrg as T
    print(f"network {sizes} rows {n} shift {shift}", flush=True)
    p = mlp_init(sizes, seed=3)
    X, Y = mlp_batch(n, sizes[0], sizes[-1], seed=7)
    net = T.Mlp(sizes, p)

    def put(a):  # optionally off a 16-byte boundary
        buf = torch.zeros(a.size + shift, dtype=torch.float32, device="cuda")
        buf[shift:] = torch.from_numpy(np.ascontiguousarray(a)).reshape(-1)
        return buf[shift:].reshape(a.shape)

    out = put(np.zeros((n, sizes[-1]), dtype=np.float32))
    T.tufrg_mlp_forward(net, put(X), out)
    ref, _, _ = omlp.forward(p, sizes, X)
    assert rel(out.cpu().numpy(), ref) < 1e-5
    grad = put(np.zeros(net.n_params, dtype=np.float32))
    loss = T.tufrg_mlp_loss_grad(net, put(X), put(Y), grad)
    loss2 = T.tufrg_mlp_loss_grad(net, put(X), put(Y))
    lref, gref = omlp.loss_and_grad(p, sizes, X, Y)
    assert abs(loss / lref - 1) < 1e-6 and loss2 == loss
    g, o = grad.cpu().numpy(), 0
    for ni, no in zip(sizes[:-1], sizes[1:]):
        for sz in (ni * no, no):
            assert rel(g[o:o + sz], gref[o:o + sz]) < 1e-5 * max(1.0, np.abs(gref).max() / np.abs(gref[o:o + sz]).max())
            o += sz
    net.close()
