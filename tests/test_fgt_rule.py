"""Host-side choice between the direct Hermite sum and the Taylor polynomials
at calls timed on both paths (microseconds in the comments: direct, Taylor);
the size of the workspace tells the choice."""
import math

import numpy as np
import pytest


def _takes_taylor(nt, depth, p, K, r):
    from paper_1009_3457_amd import _binding as B
    sigma = float(np.float32(2.0 ** -depth / (r * math.sqrt(2.0))))
    return int(B.load().fgt2d_hermite_eval_workspace(nt, depth, p, sigma, K)) > 0


@pytest.mark.parametrize("nt,p,r", [
    (1, 9, 1.0), (160, 9, 1.0), (640, 9, 0.5),   # 19, 32; 19, 32; 22, 33
    (48, 12, 1.0), (640, 12, 0.5),               # 24, 37; 26, 37
    (16, 16, 1.0), (640, 16, 0.5),               # 31, 43; 35, 44
])
def test_neighbourhoods_wider_than_the_grid_cost_the_grid(nt, p, r):
    """K = 3 on 4 x 4 boxes: 49 boxes by the neighbourhood's width, 16 there are."""
    assert not _takes_taylor(nt, 2, p, 3, r)


@pytest.mark.parametrize("nt,depth,p,K,r", [
    (204, 6, 16, 3, 0.5), (12288, 6, 16, 3, 0.5),    # 3100, 50 (unsorted)
    (3276, 8, 12, 16, 1.0),                          # 26600, 310
    (25600, 4, 9, 8, 0.5), (6553600, 8, 12, 8, 0.5),
])
def test_calls_that_gain_keep_the_polynomials(nt, depth, p, K, r):
    assert _takes_taylor(nt, depth, p, K, r)


def _order(depth, p, K, r):
    """The polynomials' order, from the layout of the workspace: a table of the
    offsets' fragments, and q p and q^2 floats a box."""
    from paper_1009_3457_amd import _binding as B
    sigma = float(np.float32(2.0 ** -depth / (r * math.sqrt(2.0))))
    have = int(B.load().fgt2d_hermite_eval_workspace(1000 * 4 ** depth, depth, p, sigma, K))
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    n, ks = 4 ** depth, (p + 3) // 4
    for q in range(4, 17, 2):
        if have == up((2 * K + 1) * ks * 256) + up(n * q * p * 4) + up(n * q * q * 4) + 256:
            return q
    assert have == 0
    return 0


def test_remainder_of_both_axes_is_within_the_stated_bound():
    """R (2 F + R) <= 2^-24 (1 + rho) for the order taken, with Cramer's bound
    |h_n| <= e_n = 1.0865 2^(n/2) sqrt(n!): R = sum_{m>=q} (r/2)^m/m! sum_{a<p}
    (r/2)^a/a! e_(a+m) on one axis, and F = 1 + rho, rho the truncation to p
    terms, for the axis's own sum."""
    e = lambda n: 1.0865 * math.exp(0.5 * n * math.log(2.0) + 0.5 * math.lgamma(n + 1))  # noqa: E731
    seen = 0
    for p in (1, 2, 3, 5, 7, 9, 12, 16):
        for r in np.arange(0.2, 1.31, 0.02):
            q = _order(6, p, 6, float(r))
            if q == 0:
                continue
            t = [(0.5 * r) ** m / math.factorial(m) for m in range(60)]
            R = sum(t[m] * t[a] * e(a + m) for m in range(q, 60) for a in range(p))
            rho = sum(t[n] * e(n) for n in range(p, 60))
            assert R * (2 * (1 + rho) + R) <= 2.0 ** -24 * (1 + rho), (p, r, q)
            seen += R * (2 * (1 + rho) + R) > 2.0 ** -25
    assert seen > 0  # 2^-25 is the bound of one axis
