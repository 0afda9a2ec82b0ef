"""The largest point sets the entry points take, 2^31 - 1 points: index
arithmetic at the end of the range.  Only the points that a test's results
depend on are written; the arrays are left as allocated otherwise (nothing
that is checked reads them)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 2 ** 31 - 1


def _last_leaves(counts):
    """Points of the leaves (6, 6), (7, 6), (6, 7), (7, 7) of depth 3, the last
    ones in Morton order, and the leaf starts of N points that end with them:
    all others in leaf 0."""
    g = np.random.Generator(np.random.PCG64(3))
    corner = [(6, 6), (7, 6), (6, 7), (7, 7)]
    pts = np.concatenate([(np.array(c) + 0.02 + 0.96 * g.random((k, 2))) / 8 for c, k in zip(corner, counts)])
    ends = np.full(65, N - sum(counts), np.int64)
    ends[0] = 0
    ends[61:65] = N - sum(counts) + np.cumsum(counts)
    return pts.astype(np.float32), ends.astype(np.int32)


def _last_rows(values):
    """A device array of N rows that ends with the given ones."""
    import torch
    v = torch.from_numpy(np.ascontiguousarray(values))
    a = torch.empty((N,) + tuple(v.shape[1:]), dtype=v.dtype, device="cuda")
    a[N - len(v):] = v.cuda()
    return a


@pytest.mark.parametrize("counts", [(20, 9, 17, 30), (130, 40, 5, 90)], ids=["staged whole", "lists"])
def test_near_field_columns_at_the_end_of_the_range(counts):
    """A few rows in the last leaf, whose columns end with the last of 2^31 - 1.
    Tolerance as in the other near-field tests."""
    import torch
    from paper_1009_3457_amd import _binding as B
    print(f"near field, columns end at 2^31 - 1, {counts}", flush=True)
    cols, ls = _last_leaves(counts)
    g = np.random.Generator(np.random.PCG64(4))
    rows = ((np.array([7, 7]) + g.random((5, 2))) / 8).astype(np.float32)
    rls = np.where(np.arange(65) <= 63, 0, 5).astype(np.int32)
    q = g.standard_normal(len(cols)).astype(np.float32)
    X, L, R, RL = _last_rows(cols), torch.from_numpy(ls).cuda(), torch.from_numpy(rows).cuda(), torch.from_numpy(rls).cuda()
    r = (rows.astype(np.float64) @ [1, 1j])[:, None] - (cols.astype(np.float64) @ [1, 1j])[None, :]
    phi, f = B.p2p(X, _last_rows(q), L, R, RL, 3)
    pr, fr = np.log(r) @ q.astype(np.float64), (1 / r) @ q.astype(np.float64)
    assert np.abs(phi.cpu().numpy() - pr).max() < 1e-5 * np.abs(pr).max()
    assert np.abs(f.cpu().numpy() - fr).max() < 1e-5 * np.abs(fr).max()
    c = (g.standard_normal(len(cols)) + 1j * g.standard_normal(len(cols))).astype(np.complex64)
    gq, G = torch.zeros(5, device="cuda"), torch.zeros(5, dtype=torch.complex64, device="cuda")
    B.p2p_backward(R, torch.ones(5, device="cuda"), RL, X, L, 3, _last_rows(c), None, gq, G)
    gqr, Gr = (np.log(-r) @ c.astype(np.complex128)).real, (1 / r) @ c.astype(np.complex128)
    assert np.abs(gq.cpu().numpy() - gqr).max() < 1e-5 * np.abs(gqr).max()
    assert np.abs(G.cpu().numpy() - Gr).max() < 1e-5 * np.abs(Gr).max()


DEPTH = 12  # 128 points a leaf, one less in the last


def _even_leaves():
    import torch
    return (torch.arange(4 ** DEPTH + 1, dtype=torch.int64, device="cuda") * 128).clamp_(max=N).to(torch.int32)


def _last_leaf_points():
    g = np.random.Generator(np.random.PCG64(6))
    off = g.random((127, 2)) - 0.5  # from the leaf's centre, in leaf widths
    xy = ((2 ** DEPTH - 0.5 + off) / 2 ** DEPTH).astype(np.float32)
    return xy, (xy.astype(np.float64) * 2 ** DEPTH - (2 ** DEPTH - 0.5)) @ [1, 1j]


def test_leaf_sums_at_the_end_of_the_range():
    """P2M and L2P^T of the last leaf.  FP32 and FP64 sums of 127 terms of at
    most 1 against FP64: 1e-5 of the largest coefficient."""
    import torch
    from paper_1009_3457_amd import _binding as B
    print("leaf sums, points end at 2^31 - 1", flush=True)
    p = 8
    xy, w = _last_leaf_points()
    g = np.random.Generator(np.random.PCG64(7))
    q, c = g.standard_normal(127).astype(np.float32), g.standard_normal(127).astype(np.complex64)
    X, L = _last_rows(xy), _even_leaves()
    M = B.p2m(X, _last_rows(q), L, DEPTH, p)[-1].cpu().numpy()
    ref = np.array([np.sum(q * w ** k) for k in range(p)])
    assert np.abs(M - ref).max() < 1e-5 * np.abs(ref).max()
    gL, gb = B.l2p_backward(X, L, _last_rows(c), None, DEPTH, p)
    ref = np.array([np.sum(c * w ** (k + 1)) / (k + 1) for k in range(p)])
    assert np.abs(gL[-1].cpu().numpy() - ref).max() < 1e-5 * np.abs(ref).max()
    assert abs(gb[-1].item() - c.sum()) < 1e-5 * np.abs(c).sum()


def test_gauss_coefficients_at_the_end_of_the_range():
    """Hermite coefficients of the last box (FP64 sums rounded once)."""
    import torch
    from paper_1009_3457_amd import _binding as B
    print("Gauss transform coefficients, sources end at 2^31 - 1", flush=True)
    p, r = 3, 0.5  # box width over sqrt(2) sigma
    sigma = float(np.float32(2.0 ** -DEPTH / (r * np.sqrt(2.0))))
    xy, w = _last_leaf_points()
    q = np.random.Generator(np.random.PCG64(8)).standard_normal(127).astype(np.float32)
    A = B.fgt_hermite_coeffs(_last_rows(xy), _last_rows(q), _even_leaves(), DEPTH, p, sigma)[-1].cpu().numpy()
    s = w * (2.0 ** -DEPTH / (np.sqrt(2.0) * sigma))
    f = np.array([1.0, 1.0, 2.0])
    ref = np.array([[np.sum(q * s.real ** a * s.imag ** b) / (f[a] * f[b]) for b in range(p)] for a in range(p)])
    assert np.abs(A - ref).max() < 2.5e-7 * np.abs(ref).max()


@pytest.mark.parametrize("rows", [N, N - 62, N - 63], ids=["all", "first past the line", "last before it"])
def test_near_field_rows_to_the_end_of_the_range(rows):
    """2^31 - 1 targets, and as many sources in the transpose, about three
    columns; the last rows are checked.  The line is the number of work-items of
    a launch."""
    import torch
    from paper_1009_3457_amd import _binding as B
    print(f"near field, {rows} rows", flush=True)
    cols = np.array([[0.9, 0.91], [0.95, 0.97], [0.99, 0.89]], np.float32)
    cls = np.where(np.arange(65) <= 63, 0, 3).astype(np.int32)
    rls = np.where(np.arange(65) <= 63, 0, rows).astype(np.int32)  # all in the last leaf
    q = np.array([0.3, -0.7, 1.1], np.float32)
    g = np.random.Generator(np.random.PCG64(9))
    last = ((np.array([7, 7]) + g.random((100, 2))) / 8).astype(np.float32)
    R = torch.full((rows, 2), 0.9375, device="cuda")
    R[rows - 100:] = torch.from_numpy(last).cuda()
    C, CL, RL = (torch.from_numpy(a).cuda() for a in (cols, cls, rls))
    r = (last.astype(np.float64) @ [1, 1j])[:, None] - (cols.astype(np.float64) @ [1, 1j])[None, :]
    phi = torch.zeros(rows, dtype=torch.complex64, device="cuda")
    Q = torch.from_numpy(q).cuda()
    B._check(B.load().fmm2d_p2p(B._p(C), B._p(Q), B._p(CL), B._p(R), B._p(RL), rows, 3, B._p(phi), None, B._stream()))
    ref = np.log(r) @ q.astype(np.float64)
    assert np.abs(phi[rows - 100:].cpu().numpy() - ref).max() < 1e-5 * np.abs(ref).max()
    first = np.log(complex(0.9375, 0.9375) - cols.astype(np.float64) @ [1, 1j]) @ q.astype(np.float64)
    assert bool((torch.view_as_real(phi[:rows - 100]).amax(dim=0) == torch.view_as_real(phi[:1])[0]).all())
    assert bool((torch.view_as_real(phi[:rows - 100]).amin(dim=0) == torch.view_as_real(phi[:1])[0]).all())
    assert abs(phi[0].item() - first) < 1e-5 * abs(first)
    del phi
    c = (g.standard_normal(3) + 1j * g.standard_normal(3)).astype(np.complex64)
    gq, G = torch.zeros(rows, device="cuda"), torch.zeros(rows, dtype=torch.complex64, device="cuda")
    w = torch.ones(rows, device="cuda")
    B.p2p_backward(R, w, RL, C, CL, 3, torch.from_numpy(c).cuda(), None, gq, G)
    gqr, Gr = (np.log(-r) @ c.astype(np.complex128)).real, (1 / r) @ c.astype(np.complex128)
    assert np.abs(gq[rows - 100:].cpu().numpy() - gqr).max() < 1e-5 * np.abs(gqr).max()
    assert np.abs(G[rows - 100:].cpu().numpy() - Gr).max() < 1e-5 * np.abs(Gr).max()
