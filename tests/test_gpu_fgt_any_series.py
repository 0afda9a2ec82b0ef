"""Evaluation of Hermite series that fgt_hermite_coeffs did not make, whose
entries don't fall off with the order, against the FP64 oracle, and the number
of terms chosen for them.

Tolerance, of the largest |G|: the direct FP32 sum rounds each of its
(2K+1)^2 p^2 terms and the recurrences of h_a, 1.0e-6 to 1.8e-6 here; the
polynomial's sums round less and its remainder is at most 2^-23: 2e-6, as in
the other tests of it."""
import math

import numpy as np
import pytest

from oracle import fgt as ofgt

TOL = 2e-6


def _sigma32(depth, r):
    """FP32 sigma with box width 2^-depth = r sqrt(2) sigma."""
    return float(np.float32(2.0 ** -depth / (r * math.sqrt(2.0))))


def _sizes(nt, depth, p, r, K):
    from paper_1009_3457_amd import _binding as B
    lib, s = B.load(), _sigma32(depth, r)
    return (int(lib.fgt2d_hermite_eval_workspace(nt, depth, p, s, K)),
            int(lib.fgt2d_hermite_eval_any_workspace(nt, depth, p, s, K)))


def test_series_of_any_origin_get_more_terms_or_the_direct_sum():
    nt = 100 * 4 ** 6
    coeffs, some = _sizes(nt, 6, 12, 0.5, 8)
    assert some > coeffs > 0        # 14 terms for 12
    coeffs, some = _sizes(nt, 6, 12, 1.0, 4)
    assert coeffs > 0 and some == 0  # 16 don't suffice
    coeffs, some = _sizes(nt, 6, 2, 0.5, 8)
    assert coeffs == some > 0       # nothing to fall off


def test_bad_arguments_are_rejected_on_host():
    import ctypes
    from paper_1009_3457_amd import _binding as B
    lib, fake = B.load(), ctypes.c_void_p(0x1000)
    nt, s = 100 * 4 ** 6, _sigma32(6, 0.5)
    need = _sizes(nt, 6, 12, 0.5, 8)[1]
    assert lib.fgt2d_hermite_eval_any(fake, nt, 6, 12, s, 8, fake, None, fake, fake, need - 1, None) == -5
    assert lib.fgt2d_hermite_eval_any(fake, nt, 6, 12, s, 8, None, None, fake, fake, need, None) == -1
    assert lib.fgt2d_hermite_eval_any(fake, nt, 6, 12, s, 8, fake, None, fake, ctypes.c_void_p(0x1008), need, None) == -1
    assert lib.fgt2d_hermite_eval_any(fake, nt, 6, 17, s, 8, fake, None, fake, fake, need, None) == -2
    assert lib.fgt2d_hermite_eval_any(None, 0, 6, 12, s, 8, fake, None, None, None, 0, None) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["one", "high", "random"])
@pytest.mark.parametrize("p,K,r", [(12, 4, 1.0), (12, 5, 0.8), (12, 7, 0.6), (9, 8, 0.5), (13, 16, 0.25)])
def test_series_of_any_origin_match_oracle(p, K, r, kind):
    """One random series in every box, one of the highest order alone in each,
    a random one in each."""
    import torch
    import paper_1009_3457_amd as P
    print(f"fgt any series p={p} K={K} r={r} {kind}", flush=True)
    depth, nt = 5, 40000
    g = np.random.Generator(np.random.PCG64(11))
    A = g.standard_normal((4 ** depth, p, p)).astype(np.float32)
    if kind == "one":
        A[:] = A[0]
    if kind == "high":
        A[:, :p - 1, :] = 0
        A[:, :, :p - 1] = 0
    t = g.random((nt, 2)).astype(np.float32)
    sigma = _sigma32(depth, r)
    G = P.fgt_hermite_eval(torch.from_numpy(t).cuda(), depth, p, sigma, K, torch.from_numpy(A).cuda()).cpu().numpy()
    at = np.arange(0, nt, 8)
    ref = ofgt.hermite_eval(t[at].astype(np.float64), depth, p, sigma, K, A.astype(np.float64))
    assert np.abs(G[at] - ref).max() < TOL * np.abs(ref).max()


@pytest.mark.gpu
def test_coefficients_take_fewer_terms_when_told_so():
    """from_coeffs=True against the default and the exact transform; the cutoff
    leaves exp(-16) a source."""
    import torch
    import paper_1009_3457_amd as P
    depth, p, K, n = 5, 12, 8, 60000
    sigma = _sigma32(depth, 0.5)
    g = np.random.Generator(np.random.PCG64(12))
    xy, q, t = g.random((n, 2)).astype(np.float32), g.random(n).astype(np.float32), g.random((n, 2)).astype(np.float32)
    _, ls, _, xs, qs = P._binding.sort_points(torch.from_numpy(xy).cuda(), torch.from_numpy(q).cuda(), depth)
    A, T = P.fgt_hermite_coeffs(xs, qs, ls, depth, p, sigma), torch.from_numpy(t).cuda()
    ref = ofgt.direct(xy.astype(np.float64), q.astype(np.float64), t[:2000].astype(np.float64), sigma)
    for told in (True, False):
        G = P.fgt_hermite_eval(T, depth, p, sigma, K, A, from_coeffs=told)[:2000].cpu().numpy()
        assert np.abs(G - ref).max() < TOL * np.abs(ref).max()
    place = torch.randperm(n, generator=torch.Generator().manual_seed(1)).to(torch.int32).cuda()
    placed = P.fgt_hermite_eval(T, depth, p, sigma, K, A, place=place, from_coeffs=True)
    assert torch.equal(placed[place.long()], P.fgt_hermite_eval(T, depth, p, sigma, K, A, from_coeffs=True))
