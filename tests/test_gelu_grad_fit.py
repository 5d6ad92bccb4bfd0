"""The network kernels' GELU': GELU'(-y) = e (1/2 + y (t P(t) - 1 / sqrt(2 pi))), e = exp(-y^2 / 2), t = 1 / (1 + y / 4),
GELU'(y) = 1 - GELU'(-y), with the coefficients written in net.hip, checked on the host against scipy."""
import re

import numpy as np
import pytest

from tests.test_gelu_fit import SRC

special = pytest.importorskip("scipy.special")


def kernel_coefficients():
    body = open(SRC).read()
    body = body[body.index("__device__ __forceinline__ float gelu_grad_f(float x)"):]
    body = body[:body.index("}\n")]
    num = r"([-+0-9.e]+)f"
    c = float(re.search(r"rcpf\(fmaf\(" + num, body).group(1))
    P = [float(re.search(r"float p = " + num + ";", body).group(1))]
    P += [float(v) for v in re.findall(r"p = fmaf\(p, t, " + num + r"\);", body)]
    scale = float(re.search(r"exp2f\(y \* y \* " + num, body).group(1))
    k = float(re.search(r"fmaf\(t, p, " + num, body).group(1))
    return c, P, scale, k


def exact(x):
    return special.ndtr(x) + x * np.exp(-0.5 * x * x) / np.sqrt(2.0 * np.pi)


def test_fit_error():
    c, P, scale, k = kernel_coefficients()
    assert c == 0.25 and len(P) == 7
    assert abs(scale + 0.5 / np.log(2)) < 1e-12 and abs(k + 1.0 / np.sqrt(2.0 * np.pi)) < 1e-12
    y = np.linspace(0.0, 14.0, 400001)
    t = 1.0 / (1.0 + c * y)
    g = np.exp2(scale * y * y) * (0.5 + y * (t * np.polyval(P, t) + k))
    # half an FP32 ulp of values up to 1.13
    assert np.max(np.abs(g - exact(-y))) <= 2.0 ** -24


def test_fp32_error():
    c, P, scale, k = kernel_coefficients()
    f = np.float32

    def fma(a, b, d):
        return (a.astype(np.float64) * b + np.float64(d)).astype(f)

    x = np.concatenate([np.random.default_rng(3).normal(0, 2, 400000), np.linspace(-8, 8, 160001)]).astype(f)
    y = np.abs(x)
    t = (f(1) / fma(y, f(c), f(1))).astype(f)
    p = np.full_like(t, f(P[0]))
    for v in P[1:]:
        p = fma(p, t.astype(np.float64), f(v))
    e = np.exp2(((y * y).astype(f) * f(scale)).astype(f)).astype(f)
    d = fma(y, fma(t, p.astype(np.float64), f(k)).astype(np.float64), f(0.5))
    pos = x > 0
    g = (np.where(pos, -e, e).astype(np.float64) * d + pos).astype(f)
    # one rounding of a result in [1, 2) (6e-8), and those of e and d and the fit, each below 4e-8
    err = np.abs(g - exact(x.astype(np.float64)))
    assert np.max(err) <= 1.8e-7
    assert np.sqrt(np.mean(err ** 2)) <= 4e-8
