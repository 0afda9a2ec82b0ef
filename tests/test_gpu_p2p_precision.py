"""How exact one pair of the near field is, against FP64: the reciprocal of
the squared distance (field, and the charge's and position's gradients), and
the angle (Im phi, and the charge's gradient of a loss on it)."""
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


def _angles(offsets):
    """(Im phi of a unit source at (1/8, 1/8) at the points around it, its exact
    value for the FP32 differences; the same with the points as sources and the
    charge's gradient of Im phi)."""
    import torch
    from paper_1009_3457_amd import _binding as B
    centre = np.full((1, 2), 0.125, np.float32)
    t = (centre + offsets).astype(np.float32)
    n = len(t)
    perm, lsn = B.build_tree(torch.from_numpy(t).cuda(), 2)
    assert np.array_equal(perm.cpu().numpy(), np.arange(n))  # one leaf
    pts, one = torch.from_numpy(t).cuda(), torch.from_numpy(centre).cuda()
    ls1 = B.build_tree(one, 2)[1]
    phi, _ = B.p2p(one, torch.ones(1, device="cuda"), ls1, pts, lsn, 2)
    d = (t - centre).astype(np.float64)  # FP32 differences, as the kernel's
    gq, G = torch.zeros(n, device="cuda"), torch.zeros(n, dtype=torch.complex64, device="cuda")
    c = torch.full((1,), -1j, dtype=torch.complex64, device="cuda")  # Re(c log r) = arg r
    B.p2p_backward(pts, torch.ones(n, device="cuda"), lsn, one, ls1, 2, c, None, gq, G)
    return ((phi.imag.cpu().numpy().astype(np.float64), np.arctan2(d[:, 1], d[:, 0])),
            (gq.cpu().numpy().astype(np.float64), np.arctan2(-d[:, 1], -d[:, 0])))


def test_angle_of_all_directions_is_no_worse_than_an_arctangents():
    """0.67e-7 rms over all directions; the arc tangent of the legs' ratio, with
    one reciprocal good to 1 ulp and the quadrant's angles subtracted after it,
    has 0.79e-7, the arc sine from the diagonal alone 0.85e-7."""
    g = np.random.Generator(np.random.PCG64(6))
    th, rad = 2 * np.pi * g.random(200000), np.exp2(-9.0 + 5.9 * g.random(200000))
    for got, ref in _angles(rad[:, None] * np.stack([np.cos(th), np.sin(th)], 1)):
        assert np.sqrt(np.mean((got - ref) ** 2)) < 7.3e-8


def test_small_angles_are_relatively_exact():
    """Relative bound: the reciprocal root's 1.2e-7, half of r^2's two roundings
    of 0.6e-7, and one rounding each of the product, the polynomial's last step
    and the sum: 3.6e-7."""
    g = np.random.Generator(np.random.PCG64(7))
    small = np.exp2(-17.0 + 10.0 * g.random(20000)) * np.where(g.random(20000) < 0.5, -1, 1)
    right, left = (np.stack([s * np.full(20000, 0.0625), 0.0625 * small], 1) for s in (1, -1))
    (got, ref), _ = _angles(right)
    assert np.all(np.abs(got - ref) <= 3.7e-7 * np.abs(ref))
    _, (got, ref) = _angles(left)  # towards the centre from its left: angles near 0
    assert np.all(np.abs(got - ref) <= 3.7e-7 * np.abs(ref))


def test_angle_on_the_axes_is_exact():
    k = np.arange(1, 60) / 512.0
    z = np.zeros_like(k)
    pi, half = np.float32(np.pi), np.float32(np.pi / 2)
    for off, want, back in ((np.stack([k, z], 1), 0.0, pi), (np.stack([-k, z], 1), pi, 0.0),
                            (np.stack([z, k], 1), half, -half), (np.stack([z, -k], 1), -half, half)):
        (got, _), (gq, _) = _angles(off)
        assert np.all(got == want) and np.all(gq == back)


def test_charges_in_a_row_add_no_angle():
    """Equal charges to the left of a target on its own horizontal line: Im phi
    is a sum of zeros, however many they are."""
    import torch
    from paper_1009_3457_amd import _binding as B
    x = np.linspace(0.26, 0.7, 5000).astype(np.float32)
    src = torch.from_numpy(np.stack([x, np.full_like(x, 0.3)], 1)).cuda()
    t = torch.tensor([[0.74, 0.3]], dtype=torch.float32, device="cuda")
    perm, ls = B.build_tree(src, 2)
    phi, _ = B.p2p(B.gather(src, perm), torch.ones(len(x), device="cuda"), ls, t, B.build_tree(t, 2)[1], 2)
    assert phi.imag.item() == 0.0


def test_rows_outside_the_square_see_their_columns_alone():
    """The near field takes rows wherever they are: a target (and, in the
    transpose, a source) at (4, 4) filed under a leaf of crowded neighbours
    interacts with the columns there and nothing else.  Tolerance as in the
    other near-field tests, 1e-5 of the largest value."""
    import torch
    from paper_1009_3457_amd import _binding as B
    g = np.random.Generator(np.random.PCG64(8))
    cols = ((np.array([1, 2]) + g.random((41, 2))) / 4).astype(np.float32)  # one other leaf, not whole phases
    rows = np.array([[4, 4], [4, 4], [0.3, 0.3]], np.float32)
    leaf, own = 9, 3  # Morton indices of (1, 2) and (1, 1)
    ls = np.where(np.arange(17) <= leaf, 0, len(cols)).astype(np.int32)
    rls = np.where(np.arange(17) <= own, 0, len(rows)).astype(np.int32)
    C, R, L, RL = (torch.from_numpy(a).cuda() for a in (cols, rows, ls, rls))
    qc = g.random(len(cols)).astype(np.float32)
    phi, f = B.p2p(C, torch.from_numpy(qc).cuda(), L, R, RL, 2)
    r = rows.astype(np.float64) @ [1, 1j]
    r = r[:, None] - (cols.astype(np.float64) @ [1, 1j])[None, :]
    pr, fr = np.log(r) @ qc.astype(np.float64), (1 / r) @ qc.astype(np.float64)
    assert np.abs(phi.cpu().numpy() - pr).max() < 1e-5 * np.abs(pr).max()
    assert np.abs(f.cpu().numpy() - fr).max() < 1e-5 * np.abs(fr).max()
    cphi = (g.standard_normal(len(cols)) + 1j * g.standard_normal(len(cols))).astype(np.complex64)
    for c in (cphi, cphi.real.astype(np.complex64)):
        gq, G = torch.zeros(3, device="cuda"), torch.zeros(3, dtype=torch.complex64, device="cuda")
        B.p2p_backward(R, torch.ones(3, device="cuda"), RL, C, L, 2, torch.from_numpy(c).cuda(), None, gq, G)
        gqr, Gr = (np.log(-r) @ c.astype(np.complex128)).real, (1 / r) @ c.astype(np.complex128)
        assert np.abs(gq.cpu().numpy() - gqr).max() < 1e-5 * np.abs(gqr).max()
        assert np.abs(G.cpu().numpy() - Gr).max() < 1e-5 * np.abs(Gr).max()
