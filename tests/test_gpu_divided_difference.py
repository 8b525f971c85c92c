"""The divided differences of the loop kernels at close energies, one pair of
energies at a time: on a 2 x 2 mesh with one hopping along x and bands without
spin the particle-hole loop at q = (pi, 0) is their divided difference alone (four
equal terms, sums and factors of two).

Against the exact mean of the derivative over the interval (Gauss-Legendre with ten
points in 80-bit arithmetic), and against the error of the two-point rule
evaluated in the kernel's own arithmetic at the same pairs: the kernel may not be
further off than the spread of such errors."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

X = np.longdouble
GX, GW = (v.astype(X) for v in np.polynomial.legendre.leggauss(10))


def _derivative(e, lam, cutoff, deriv):
    """K' (deriv) or J' in the type of its arguments, each quantity rounded to it."""
    T = type(lam)
    if cutoff == "temperature":
        x = e / (T(2) * lam)
        s = np.exp(T(-2) * np.abs(x))
        inv = T(1) / (T(1) + s)
        s2, th = T(4) * s * inv * inv, np.copysign((T(1) - s) * inv, x)
        return -s2 * (T(1) - T(2) * x * th) / (T(4) * lam * lam) if deriv else s2 / (T(4) * lam)
    a = np.abs(e)
    d = a + lam
    if deriv:
        return (T(3) * e * e - T(4) * a * lam - lam * lam) / (T(4) * (d * d) * (d * d))
    return lam * (T(3) * a + lam) / (T(4) * (d * d) * d)


def _pairs(prec, cutoff):
    rng = np.random.default_rng(5)
    T = np.float64 if prec == "fp64" else np.float32
    width = 1e-3 if prec == "fp64" else 2e-2
    out = []
    for i in range(160):
        lam = np.exp(rng.uniform(np.log(0.1), np.log(2.0)))
        x = lam * (rng.uniform(0.0, 4.0) if i % 4 else 0.01 * rng.uniform())
        w = 0.98 * width * (lam if cutoff == "temperature" else lam + 2.0 * x)
        out.append((T(lam), x, w * (1.0 if i % 2 else rng.uniform(0.3, 1.0))))
    for i in range(20):  # zero inside
        lam = np.exp(rng.uniform(np.log(0.1), np.log(2.0)))
        out.append((T(lam), -0.9 * width * lam * rng.uniform(0.01, 0.99), 0.9 * width * lam))
    return T, out


@pytest.mark.parametrize("prec,cutoff", [("fp64", "temperature"), ("fp32", "temperature"), ("fp32", "omega"),
                                         ("fp64", "omega")])
@pytest.mark.parametrize("deriv", [1, 0])
def test_the_mean_is_no_further_off_than_the_two_point_rule(prec, cutoff, deriv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_08830_amd import tufrg as TU
    T, pairs = _pairs(prec, cutoff)
    n_o = 1 if prec == "fp64" else 2
    worst = {"kernel": 0.0, "two-point": 0.0}
    for lam, x0, w in pairs:
        one = np.eye(n_o)
        # energies x0 + w and x0 at kx = 0 and pi
        R = np.array([[0, 0], [1, 0], [-1, 0]], dtype=np.int32)
        t = np.array([(x0 + 0.5 * w) * one, 0.25 * w * one, 0.25 * w * one]).astype(np.complex128)
        ctx = TU.Context(R, t, 0.0, np.zeros((n_o,) * 4, dtype=np.complex128), np.array([[0, 0]], dtype=np.int32), 2, 1,
                         cutoff, prec)
        e = torch.empty((n_o, 4), dtype=torch.float64, device="cuda")
        Pi = torch.empty((n_o, 4, n_o, n_o), dtype=torch.complex128, device="cuda")
        TU.tufrg_band_data(ctx, e, Pi)
        L = torch.empty((2, 4, 1, n_o ** 4), dtype=torch.complex128, device="cuda")
        TU.tufrg_loops_compact(ctx, float(lam), deriv, L)
        x, y = (T(v) for v in (e[0, 0].item(), e[0, 2].item()))
        got = X(-L[1, 2, 0, 0].real.item())
        ctx.close()
        mid, half = X(0.5) * (X(x) + X(y)), X(0.5) * (X(x) - X(y))
        if x * y < 0:  # K' of the Omega scheme has a kink at 0: both parts
            ref = sum(X(0.5) * g * (X(z) * _derivative(X(0.5) * X(z) * (1 + p), X(lam), cutoff, deriv))
                      for z in (abs(x), abs(y)) for p, g in zip(GX, GW)) / (X(abs(x)) + X(abs(y)))
        else:
            ref = sum(X(0.5) * g * _derivative(mid + p * half, X(lam), cutoff, deriv) for p, g in zip(GX, GW))
        c = T(0.57735026918962576451)
        m, h = T(0.5) * (x + y), T(0.5) * (y - x)
        two = T(0.5) * (_derivative(m - c * h, lam, cutoff, deriv) + _derivative(m + c * h, lam, cutoff, deriv))
        if x * y < 0 and cutoff == "omega":
            two = T(ref)  # the quotient of sums of one sign: rounding alone
        top = X(0.25) / (X(lam) ** 2 if deriv else X(lam))  # the largest |f|
        for name, v in (("kernel", got), ("two-point", X(two))):
            worst[name] = max(worst[name], float(abs(v - ref) / top))
    print(f"{prec} {cutoff} deriv {deriv}: kernel {worst['kernel']:.2e}, two-point rule {worst['two-point']:.2e}", flush=True)
    # 1.5: the spread of the largest of 180 rounding errors (FP64 Omega: it is that rule)
    assert worst["kernel"] <= 1.5 * worst["two-point"]
