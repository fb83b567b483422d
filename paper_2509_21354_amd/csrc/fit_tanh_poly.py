"""Derives the constants of ``tanh_small`` in ``lstm_generic.hip``.

For |x| < X_MAX, tanh x = x + x^3 P(x^2) with P a polynomial: a least-squares fit of the relative error on Chebyshev
nodes, re-weighted by the error until the largest errors are alike (Lawson's iteration towards the minimax fit).  Run
``python fit_tanh_poly.py`` to print the coefficients and the error; ``coefficients()`` is what the test of the constants
imports.
"""
import numpy as np

X_MAX = 0.5625
DEGREE = 5          # number of coefficients of P


def coefficients(degree: int = DEGREE) -> np.ndarray:
    n = 4001
    x = X_MAX * 0.5 * (1.0 - np.cos(np.pi * (np.arange(n) + 0.5) / n))
    ratio = x / np.tanh(x)
    A = (x * x)[:, None] ** np.arange(1, degree + 1) * ratio[:, None]
    w = np.ones(n)
    coef = None
    for _ in range(200):
        coef, *_ = np.linalg.lstsq(A * np.sqrt(w)[:, None], (1.0 - ratio) * np.sqrt(w), rcond=None)
        err = np.abs(A @ coef - (1.0 - ratio))
        w = w * (err / err.max() + 1e-12)
        w /= w.sum()
    return coef


def relative_error(x, coef) -> np.ndarray:
    s = x * x
    return (x + x * s * np.polynomial.polynomial.polyval(s, coef)) / np.tanh(x) - 1.0


def tanh_f32(x: np.ndarray, coef) -> np.ndarray:
    """The kernel's evaluation order in float32 (its fused multiply-adds rounded once, through float64)."""
    f, d = np.float32, np.float64
    x, c = np.asarray(x).astype(f), np.asarray(coef).astype(f)
    s = x * x
    p = np.full_like(x, c[-1])
    for k in range(len(c) - 2, -1, -1):
        p = f(d(p) * d(s) + d(c[k]))
    return f(d(f(x * s)) * d(p) + d(x))


if __name__ == "__main__":
    c = coefficients()
    for k, v in enumerate(c):
        print(f"c{k} = {np.float32(v)!r:>16}  ({v:.17e})")
    xs = np.linspace(1e-4, X_MAX, 400001)
    print("largest relative error:", np.abs(relative_error(xs, c)).max())
