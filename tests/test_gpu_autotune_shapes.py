"""The autotuner on models without time reversal: one loop channel sums every kx
row there and the other half of them, so a chunk's rows do not follow from the
number of chunks.  The default shape is one of the candidates that are timed,
and a second context takes the cached shape bit for bit.  Models of equal sizes
whose loops do other work (time reversal; the kind of matrix-core loops) have
cache entries of their own."""

import json

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import PAULI, ff_shell, kanamori_V0, onsite_V0, rashba_hoppings, t2g_soc_hoppings  # noqa: E402


@pytest.fixture(scope="module")
def T():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg
    return tufrg


def _ctx(T, field, Lq, n_ref, prec):
    R, t = rashba_hoppings(1.0, 0.3)
    if field:
        R = np.concatenate([np.asarray(R), [[0, 0]]]).astype(np.int32)
        t = np.concatenate([t, field * PAULI[2][None]])
    return T.Context(R, t, -0.4, onsite_V0(2.5), ff_shell(5), Lq, n_ref, "temperature", prec)


def _loops(T, ctx):
    L = torch.empty((2, ctx.Nq, ctx.n_dR, 16), dtype=torch.complex128, device="cuda")
    T.tufrg_loops_compact(ctx, 0.3, 1, L)
    return L.cpu().numpy()


@pytest.mark.parametrize("Lq,n_ref", [(8, 4), (8, 8), (9, 7), (12, 12)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_the_default_shape_is_timed_without_time_reversal(T, tmp_path, Lq, n_ref, prec):
    print(f"autotune: rashba in a field S5 {Lq}x{Lq} refined {n_ref}x {prec}", flush=True)
    cache = tmp_path / "tune.json"
    ctx = _ctx(T, 0.2, Lq, n_ref, prec)
    r = T.tufrg_autotune(ctx, 0.3, str(cache))
    print(r)
    assert r["n_candidates"] >= 2 and 0 < r["loop_ms"] <= r["default_ms"]
    (entry,) = json.loads(cache.read_text())["entries"].values()
    assert entry["default_ms"] == r["default_ms"] and entry["loop_kx_chunks"] == r["loop_kx_chunks"]
    other = _ctx(T, 0.2, Lq, n_ref, prec)
    r2 = T.tufrg_autotune(other, 0.3, str(cache))
    assert r2["from_cache"] == 1 and r2["loop_kx_chunks"] == r["loop_kx_chunks"]
    assert np.array_equal(_loops(T, other), _loops(T, ctx))
    ctx.close()
    other.close()


def test_models_of_equal_sizes_do_not_share_an_entry(T, tmp_path):
    cache = tmp_path / "tune.json"
    for field in (0.0, 0.2):
        print(f"autotune: rashba field {field} S5 8x8 refined 6x fp32", flush=True)
        ctx = _ctx(T, field, 8, 6, "fp32")
        assert T.tufrg_autotune(ctx, 0.3, str(cache))["from_cache"] == 0
        ctx.close()
    # pairs in 15 coordinates; the same bands with the spin index slowest: pairs in 36; no pairs
    R, t = t2g_soc_hoppings(0.2, seed=1)
    p = [0, 2, 4, 1, 3, 5]
    for hop, paired in ((t, True), (np.ascontiguousarray(t[:, p][:, :, p]), True), (t, False)):
        print(f"autotune: t2g S5 6x6 refined 4x bf16x3, pairs {paired}", flush=True)
        ctx = T.Context(R, hop, 0.35, kanamori_V0(2.0, 0.3), ff_shell(5), 6, 4, "temperature", "bf16x3")
        assert T.tufrg_pair_bands(ctx, paired) is paired
        assert T.tufrg_autotune(ctx, 0.3, str(cache))["from_cache"] == 0
        ctx.close()
    assert len(json.loads(cache.read_text())["entries"]) == 5


def test_an_entry_from_before_the_rows_were_halved_is_not_applied(T, tmp_path):
    cache = tmp_path / "tune.json"
    ctx = _ctx(T, 0.0, 8, 8, "fp32")
    T.tufrg_autotune(ctx, 0.3, str(cache))
    (key,) = json.loads(cache.read_text())["entries"]
    old = key.split("|half=")[0] + "|pairs=0"
    for k in (key, old):
        cache.write_text(json.dumps({"version": 1, "entries": {
            k: {"loop_kx_chunks": 2, "loop_ms": 1.0, "default_ms": 1.0}}}))
        r = T.tufrg_autotune(ctx, 0.3, str(cache))
        assert r["from_cache"] == 0 and r["n_candidates"] >= 2
    ctx.close()
