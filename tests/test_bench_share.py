"""bench.py's share of the summed points and choice of the matrix-core count
follow the hopping table of the model that runs (CPU)."""

import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

from synth import PAULI, workload  # noqa: E402
from tests.test_loop_symmetry import MODELS  # noqa: E402


@pytest.mark.parametrize("model", sorted(MODELS))
def test_the_share_follows_time_reversal(model):
    import bench
    (R, t), kind = MODELS[model]
    assert bench.summed_share({"hop_R": R, "hop_t": t}) == (0.25 if kind else 0.5)


def test_the_workloads_and_the_fifteen_coordinates():
    import bench
    for name in ("hubbard_s5_L8", "rashba_s9_L24", "t2g_s13_L32", "t2g_s13_L48"):
        w = workload(name)
        assert bench.summed_share(w) == 0.25
        assert bench.fifteen_coordinates(w, True) is (w["n_o"] == 6) and not bench.fifteen_coordinates(w, False)
    w = dict(workload("t2g_s13_L32"))
    slow = [0, 2, 4, 1, 3, 5]
    assert not bench.fifteen_coordinates(dict(w, hop_t=np.asarray(w["hop_t"])[:, slow][:, :, slow]), True)
    field = dict(w, hop_R=np.concatenate([w["hop_R"], [[0, 0]]]),
                 hop_t=np.concatenate([w["hop_t"], 0.1 * np.kron(np.eye(3), PAULI[2])[None]]))
    assert bench.summed_share(field) == 0.5 and not bench.fifteen_coordinates(field, True)
    R, t = MODELS["quaternionic"][0]
    assert bench.fifteen_coordinates({"hop_R": R, "hop_t": t}, True)
