"""The polynomials in the sub-bin offset that the smooth kernels take, checked
on the host for every width that takes them (the edges of each class of term
counts included): the interpolant of N(d - t) through the n Chebyshev nodes of
[-1/2, 1/2] against the direct Gaussian samples over the support, for the
forward with n terms, and for the adjoint with n + 1 terms its value and its
derivative.  The bounds are the root mean square over the offset, relative
over the support: 2.5e-8 for the samples, 1e-7 for the derivative (which the
adjoint multiplies with an fp32 weight)."""
import math

import numpy as np
import pytest

# smallest width (bins) of each class of forward terms
CLASSES = [(1.2, 8), (1.6, 7), (2.5, 6), (4.9, 5)]
WIDTHS = [1.2, 1.4, 1.5999, 1.6, 1.858, 2.0, 2.4999, 2.5, 2.654, 3.185, 4.0, 4.8999, 4.9, 7.4, 20.0, 170.0]


def terms(sigma):
    return [n for lo, n in CLASSES if sigma >= lo][-1]


def fit(sigma, n):
    rs = math.ceil(6 * sigma)
    d = np.arange(-rs, rs + 1, dtype=np.float64)
    nodes = 0.5 * np.cos(np.pi * (2 * np.arange(n) + 1) / (2 * n))
    coef = np.linalg.inv(np.vander(nodes, n, increasing=True))     # [m][j]: s^m of node j's Lagrange polynomial
    return d, coef @ gauss(d[None, :] + nodes[:, None], sigma)


def gauss(x, sigma):
    return np.exp(-0.5 * (x / sigma) ** 2) / (sigma * math.sqrt(2 * math.pi))


@pytest.mark.parametrize("sigma", WIDTHS)
def test_forward_terms(sigma):
    d, K = fit(sigma, terms(sigma))
    err = []
    for s in np.linspace(-0.5, 0.5, 101):
        direct = gauss(d + s, sigma)
        err.append(np.linalg.norm(sum(s ** m * k for m, k in enumerate(K)) - direct) / np.linalg.norm(direct))
    assert np.sqrt(np.mean(np.square(err))) <= 2.5e-8


@pytest.mark.parametrize("sigma", WIDTHS)
def test_adjoint_terms(sigma):
    d, K = fit(sigma, terms(sigma) + 1)
    e0, e1 = [], []
    for s in np.linspace(-0.5, 0.5, 101):
        direct = gauss(d + s, sigma)
        slope = -(d + s) / sigma ** 2 * direct
        e0.append(np.linalg.norm(sum(s ** m * k for m, k in enumerate(K)) - direct) / np.linalg.norm(direct))
        e1.append(np.linalg.norm(sum(m * s ** (m - 1) * K[m] for m in range(1, len(K))) - slope) / np.linalg.norm(slope))
    assert np.sqrt(np.mean(np.square(e0))) <= 2.5e-8
    assert np.sqrt(np.mean(np.square(e1))) <= 1e-7
