"""Coefficients of the rational approximation used by the fp32 acquisition
kernels for the normal partial expectation.

For x >= 0 let M(x) = P(Z > x) / phi(x) (the Mills ratio of the standard
normal) and g(x) = 1 - x M(x), so that h(-x) = phi(x) g(x) with
h(u) = u Phi(u) + phi(u).  g falls from 1 at 0 like 1 / x^2; it is fitted on
[0, 14] by R(s) = P4(s) / Q6(s), s = x / 4 (the denominator two degrees higher
to follow the 1 / x^2 tail), minimising the relative error: linearised least
squares iterated on the previous denominator (Sanathanan-Koerner), then
reweighted towards the largest errors (Lawson).  Prints the two coefficient
lists and the achieved relative error in double and in float32 Horner
evaluation.

For the fp64 kernels phi(0) g(x) (x + K)^2 is expanded in Chebyshev polynomials
of y, r = 1 / (x + K) mapped linearly from x = 0 .. 39 to 1 .. -1 (the rational
variable with which Shepherd and Laframboise, Math. Comp. 36 (1981), expand
erfcx), in 60 digits, and printed as powers of y.  K = 5 gives the fastest
decay: the first term left out is below 1e-17 of the value.

Run: python gen_normal_tail.py
"""
import mpmath as mp
import numpy as np
from scipy.special import erfcx

SCALE = 4.0
X_MAX = 14.0
DEG_P, DEG_Q = 4, 6


def g_exact(x):
    return 1.0 - x * erfcx(x / np.sqrt(2.0)) * np.sqrt(np.pi / 2.0)


def fit():
    x = np.concatenate([np.linspace(0.0, 1.0, 2000), np.linspace(1.0, X_MAX, 20000)[1:]])
    y = g_exact(x)
    s = x / SCALE
    w = 1.0 / y
    q_prev = np.ones_like(x)
    for it in range(80):
        A = np.hstack([np.vander(s, DEG_P + 1, increasing=True),
                       -y[:, None] * np.vander(s, DEG_Q + 1, increasing=True)[:, 1:]])
        W = (w / q_prev)[:, None]
        c, *_ = np.linalg.lstsq(A * W, y * W[:, 0], rcond=None)
        p = c[:DEG_P + 1]
        q = np.concatenate([[1.0], c[DEG_P + 1:]])
        q_prev = np.polyval(q[::-1], s)
        err = (np.polyval(p[::-1], s) / q_prev - y) / y
        if it > 20:
            w = w * (1.0 + 50.0 * np.abs(err) / np.max(np.abs(err)))
    return x, y, p, q, np.max(np.abs(err))


def eval_f32(p, q, x):
    s = (x.astype(np.float32) * np.float32(1.0 / SCALE)).astype(np.float32)
    P = np.float32(p[-1])
    for c in p[-2::-1]:
        P = (P * s + np.float32(c)).astype(np.float32)
    Q = np.float32(q[-1])
    for c in q[-2::-1]:
        Q = (Q * s + np.float32(c)).astype(np.float32)
    return (P / Q).astype(np.float32)


K64, X64, DEG64 = 5, 39, 24


def fit64():
    mp.mp.dps = 60
    r0, r1 = mp.mpf(1) / (X64 + K64), mp.mpf(1) / K64
    n = DEG64 + 16
    c = [mp.mpf(0)] * (DEG64 + 1)
    for i in range(n):
        a = mp.pi * (2 * i + 1) / (2 * n)
        r = (r0 + r1) / 2 + (r1 - r0) / 2 * mp.cos(a)
        x = 1 / r - K64
        g = 1 - x * mp.sqrt(mp.pi / 2) * mp.exp(x * x / 2) * mp.erfc(x / mp.sqrt(2))
        for k in range(DEG64 + 1):
            c[k] += (2 if k else 1) * g / r ** 2 / mp.sqrt(2 * mp.pi) * mp.cos(k * a) / n
    power = [mp.mpf(0)] * (DEG64 + 1)
    t0, t1 = [mp.mpf(1)], [mp.mpf(0), mp.mpf(1)]  # T_k in powers of y
    for k in range(DEG64 + 1):
        for e, v in enumerate(t0):
            power[e] += c[k] * v
        nxt = [mp.mpf(0)] + [2 * v for v in t1]
        for e, v in enumerate(t0):
            nxt[e] -= v
        t0, t1 = t1, nxt
    return 2 / (r1 - r0), -(r1 + r0) / (r1 - r0), power


if __name__ == "__main__":
    a64, b64, power64 = fit64()
    print("fp64: y = a r + b, a, b =", mp.nstr(a64, 20), mp.nstr(b64, 20))
    print("powers of y:", ", ".join(mp.nstr(v, 20) for v in power64))
    x, y, p, q, e = fit()
    e32 = np.max(np.abs((eval_f32(p, q, x).astype(np.float64) - y) / y))
    assert np.min(np.polyval(q[::-1], x / SCALE)) >= 1.0
    print("P:", ", ".join(f"{v:.9e}f" for v in p))
    print("Q:", ", ".join(f"{v:.9e}f" for v in q))
    print(f"max relative error on [0, {X_MAX}]: double {e:.2e}, float32 Horner {e32:.2e}")
