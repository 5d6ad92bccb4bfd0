"""Fits of the normal tail used by the GELU and GELU' epilogues of the network kernels.

Phi(-y) (y >= 0) is written as t * 2^(P(t) - y^2 / (2 ln 2)) with t = 1 / (1 + c y) and P a
polynomial of degree 6; P is fitted to log2(Phi(-y) / t) + y^2 / (2 ln 2) on y in [0, 14] by least
squares, reweighted iteratively toward the minimax solution, and its coefficients are rounded to
fp32.  Prints a C initialiser for the kernel source and the maximum relative error of Phi(-y)
(evaluated in FP64 with the rounded coefficients).

GELU'(-y) = Phi(-y) - y phi(y) is written as e (1/2 + y (t P(t) - 1 / sqrt(2 pi))), e = exp(-y^2 / 2),
t = 1 / (1 + y / 4), P of degree 6, fitted the same way to the absolute error of GELU' (the relative
error of the tail weighs in below e = 0.02).

    python paper_1904_03057_amd/fit_gelu.py
"""
import numpy as np
from scipy.special import log_ndtr

DEG = 6
YMAX = 14.0
L2E = 1.0 / np.log(2.0)


def fit(c, iters=40):
    y = np.linspace(0.0, YMAX, 200001)
    t = 1.0 / (1.0 + c * y)
    f = log_ndtr(-y) * L2E - np.log2(t) + 0.5 * y * y * L2E
    V = np.vander(t, DEG + 1)
    w = np.ones_like(t)
    for _ in range(iters):
        coef, *_ = np.linalg.lstsq(V * w[:, None], f * w, rcond=None)
        e = V @ coef - f
        w = w * (1.0 + 5.0 * np.abs(e) / np.abs(e).max())
        w /= w.mean()
    return coef.astype(np.float32)


def rel_error(c, coef):
    y = np.linspace(0.0, YMAX, 400001)
    t = 1.0 / (1.0 + np.float64(np.float32(c)) * y)
    P = np.polyval(coef.astype(np.float64), t)
    q = t * np.exp2(P - 0.5 * y * y * L2E)
    ref = np.exp(log_ndtr(-y))
    return float(np.max(np.abs(q / ref - 1.0)))


def fit_grad(c=0.25, iters=40):
    y = np.concatenate([np.linspace(1e-4, 6.0, 30001), np.linspace(6.0, YMAX, 4001)])
    t = 1.0 / (1.0 + c * y)
    f = (np.exp(log_ndtr(-y) + 0.5 * y * y) - 0.5) / (y * t)
    scale = y * t * np.maximum(np.exp(-0.5 * y * y), 2e-2)
    V = np.vander(t, DEG + 1)
    w = scale.copy()
    for _ in range(iters):
        coef, *_ = np.linalg.lstsq(V * w[:, None], f * w, rcond=None)
        e = np.abs((V @ coef - f) * scale)
        w = w * (1.0 + 5.0 * e / e.max())
        w /= w.mean()
    return coef.astype(np.float32)


def grad_error(coef, c=0.25):
    y = np.linspace(0.0, YMAX, 400001)
    t = 1.0 / (1.0 + c * y)
    e = np.exp(-0.5 * y * y)
    k = 1.0 / np.sqrt(2.0 * np.pi)
    d = e * (0.5 + y * (t * np.polyval(coef.astype(np.float64), t) - k))
    return float(np.max(np.abs(d - (np.exp(log_ndtr(-y)) - y * e * k))))


def main():
    best = None
    for c in np.linspace(0.25, 0.31, 25):
        coef = fit(c)
        err = rel_error(c, coef)
        if best is None or err < best[0]:
            best = (err, float(np.float32(c)), coef)
    err, c, coef = best
    print("c = %.9ef" % c)
    print("P (highest degree first) = {" + ", ".join("%.9ef" % v for v in coef) + "}")
    print("max relative error of Phi(-y): %.3e" % err)
    coef = fit_grad()
    print("GELU' P (highest degree first) = {" + ", ".join("%.9ef" % v for v in coef) + "}")
    print("max error of GELU'(-y): %.3e" % grad_error(coef))


if __name__ == "__main__":
    main()
