"""Accuracy of the fp32 posterior's split product, in units that tell six part
products from five.

With v = L^-1 k, q = |v|^2 and beta = K^-1 k, an error of one eps = 2^-24 in
every covariance, independent from entry to entry, moves q by 2 eps
sqrt(sum_i (beta_i k_i)^2), and one eps of rounding whenever 16 columns more have
been added to a v_i, whose sum is P_ij then, by 2 eps sqrt(sum_i v_i^2 sum_j
P_ij^2).  The unit is half their root mean square over the candidates, the
measure the root mean square of the error of q in that unit.
An error that all covariances share, e of themselves (the bias of the square
root and the exponential, up to four eps), moves q by 2 e q: it is fitted and
taken off.  What is left of the covariances' errors and the rounding is a few
eps: a correct kernel measures 2 to 3.6.  One part product of the six left out
measures 9 at least (test_posterior_split_host.py).  So: 5.  The mean,
alpha . k, has the unit eps sqrt(sum (alpha_i k_i)^2) the same way."""
import numpy as np

from oracle.gp import matern52

EPS = 2.0 ** -24
LIMIT = 5.0


def problem(m, d, tau2=1e-2):
    rng = np.random.default_rng(1000 * m + d)
    return rng.random((m, d)), rng.standard_normal(m), rng.uniform(0.3, 1.5, d), tau2


def factor(X, y, ls, tau2):
    Li = np.linalg.inv(np.linalg.cholesky(matern52(X, X, ls, 1.0) + tau2 * np.eye(len(X))))
    return Li, Li.T @ (Li @ y)


def units(Li, alpha, k):
    """(of q, of the mean) over the candidates that are the columns of k."""
    v = Li @ k
    beta = Li.T @ v
    part, rounding = np.zeros_like(v), np.zeros_like(v)
    for j in range(0, len(k), 16):
        part += Li[:, j:j + 16] @ k[j:j + 16]
        rounding += np.where(np.arange(len(k))[:, None] >= j, part * part, 0.0)
    rms = lambda x: float(np.sqrt(np.mean(x)))  # noqa: E731
    return (EPS * rms(((beta * k) ** 2).sum(0) + (v * v * rounding).sum(0)), EPS * rms(((alpha[:, None] * k) ** 2).sum(0)))


def measure(err, unit, shared=None):
    """shared: what an error of one, common to all covariances, does to the value."""
    if shared is not None:
        err = err - np.clip(err @ shared / (shared @ shared), -4 * EPS, 4 * EPS) * shared
    return float(np.sqrt(np.mean(np.square(err)))) / unit
