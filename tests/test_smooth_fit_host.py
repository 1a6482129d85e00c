"""The polynomials that the library's host side hands to the smooth kernels --
its choice of terms, its nodes, its coefficients -- on a dense sweep of widths:
within 2.5e-8 of the Gaussian samples over the support (root mean square over
the sub-bin offset, relative over the support), 1e-7 for the adjoint's
derivative, and the coefficients reproduce every power below the number of
terms at any offset (1e-12: fp64 recurrences of at most nine terms)."""
import math

import numpy as np
import pytest

import host_plans

WIDTHS = sorted(set(np.round(np.geomspace(1.2, 170.0, 160), 6)) | {1.2, 1.5999999, 1.6, 2.4999999, 2.5, 4.8999999, 4.9})
# Gauss-Legendre points and weights of the mean over the bin (exact to degree 63)
S, W = np.polynomial.legendre.leggauss(32)
S, W = S / 2, W / 2


def _gauss(x, sigma):
    return np.exp(-0.5 * (x / sigma) ** 2) / (sigma * math.sqrt(2 * math.pi))


@pytest.mark.parametrize("adjoint", [False, True])
def test_polynomials_of_the_library(adjoint):
    terms = set()
    for sigma in WIDTHS:
        node, coef = (np.array(v) for v in host_plans.moment_fit(float(sigma), adjoint))
        n = len(node)
        terms.add(n)
        assert np.abs(node).max() <= 0.5
        powers = S[:, None] ** np.arange(n)
        for k in range(n):          # the interpolant of s^k is s^k
            np.testing.assert_allclose(powers @ (coef @ node ** k), S ** k, rtol=0, atol=1e-12)
        rs = math.ceil(6 * sigma)
        d = np.arange(-rs, rs + 1.0)
        K = coef @ _gauss(d[None, :] + node[:, None], sigma)
        direct = _gauss(d[None, :] + S[:, None], sigma)
        e0 = np.linalg.norm(powers @ K - direct, axis=1) / np.linalg.norm(direct, axis=1)
        assert np.sqrt(W @ e0 ** 2) <= 2.5e-8, (sigma, n)
        if adjoint:
            slope = -(d[None, :] + S[:, None]) / sigma ** 2 * direct
            got = (powers[:, :-1] * np.arange(1, n)) @ K[1:]
            e1 = np.linalg.norm(got - slope, axis=1) / np.linalg.norm(slope, axis=1)
            assert np.sqrt(W @ e1 ** 2) <= 1e-7, (sigma, n)
    assert terms == ({6, 7, 8, 9} if adjoint else {5, 6, 7, 8})


def test_narrow_widths_go_by_taps():
    for sigma in (0.05, 0.7, 1.19, 1.1999999):
        assert host_plans.moment_fit(sigma, False) is None and host_plans.moment_fit(sigma, True) is None
