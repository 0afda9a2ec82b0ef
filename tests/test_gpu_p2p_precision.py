"""How exact one pair of the near field is, against FP64: the reciprocal of
the squared distance (field, and the charge's and position's gradients)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _differences(n=20000):
    """FP32 points about the origin in the leaf [0, 1/4)^2 of depth 2, all
    directions of the quadrant."""
    g = np.random.Generator(np.random.PCG64(5))
    th, rad = 0.5 * np.pi * g.random(n), np.exp2(-10.0 + 7.9 * g.random(n))
    return (rad[:, None] * np.stack([np.cos(th), np.sin(th)], 1)).astype(np.float32)


def _around_origin(d):
    """Device arrays: the points with their leaf starts, and one at the origin
    with its leaf starts."""
    import torch
    from paper_1009_3457_amd import _binding as B
    pts, one = torch.from_numpy(d).cuda(), torch.zeros(1, 2, device="cuda")
    perm, lsn = B.build_tree(pts, 2)
    assert np.array_equal(perm.cpu().numpy(), np.arange(len(d)))  # one leaf: the order is kept
    return pts, lsn, one, B.build_tree(one, 2)[1]


def _rms(got, ref):
    return float(np.sqrt(np.mean(np.abs(got - ref) ** 2 / np.abs(ref) ** 2)))


# 1/r of one pair.  r^2 has two roundings of at most 2^-24, the hardware
# reciprocal is good to 1 ulp (2^-23), each component is rounded once more:
# 4.1e-8 rms measured for 1/r^2 and 2.6e-8 (2^-24 / sqrt 3 over the mean
# mantissa) for the last rounding, together 4.8e-8.  The square of a 1-ulp
# reciprocal root has 6.8e-8 in the place of 4.1e-8: 7.3e-8 in all.
RMS = 5.5e-8


def test_field_has_the_reciprocals_precision():
    import torch
    from paper_1009_3457_amd import _binding as B
    d = _differences()
    n = len(d)
    pts, lsn, one, ls1 = _around_origin(d)
    q = torch.ones(1, device="cuda")
    ref = 1 / (d.astype(np.float64) @ [1, 1j])
    _, both = B.p2p(one, q, ls1, pts, lsn, 2)
    alone = torch.zeros(n, dtype=torch.complex64, device="cuda")
    B._check(B.load().fmm2d_p2p(B._p(one), B._p(q), B._p(ls1), B._p(pts), B._p(lsn), n, 2, None, B._p(alone), B._stream()))
    for f in (both, alone):
        assert _rms(f.cpu().numpy().astype(np.complex128), ref) < RMS


@pytest.mark.parametrize("c", [1.0, 1j], ids=["real", "imaginary"])
def test_gradients_have_the_reciprocals_precision(c):
    """G = -c / r of sources about one target (its cotangent c of phi, where an
    imaginary part needs the angle)."""
    import torch
    from paper_1009_3457_amd import _binding as B
    d = _differences()
    n = len(d)
    pts, lsn, one, ls1 = _around_origin(d)
    q = torch.ones(n, device="cuda")
    cphi = torch.full((1,), c, dtype=torch.complex64, device="cuda")
    gq, G = torch.zeros(n, device="cuda"), torch.zeros(n, dtype=torch.complex64, device="cuda")
    B.p2p_backward(pts, q, lsn, one, ls1, 2, cphi, None, gq, G)
    ref = -c / (-d.astype(np.float64) @ [1, 1j])
    assert _rms(G.cpu().numpy().astype(np.complex128), ref) < RMS
