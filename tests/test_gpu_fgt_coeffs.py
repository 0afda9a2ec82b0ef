"""Hermite coefficients where the choice between matrix products and a thread
per row changes: blocks of 64 boxes at and past the line, single boxes at and
past twice it, empty blocks, on grids whose waves take 4, 16 and 64
boxes.  FP64 sums rounded once on both sides: 2^-24 relative, 2.5e-7 allowed,
as in the other coefficient tests."""
import numpy as np
import pytest

from oracle import fgt as ofgt

pytestmark = pytest.mark.gpu


def _counts(nbox, meet):
    """Sources of every box."""
    g = np.random.Generator(np.random.PCG64(2))
    c = np.zeros(nbox, np.int64)
    blocks = c.reshape(-1, 64)
    blocks[0] = meet             # the mean at the line
    blocks[1] = meet
    blocks[1, 17] += 1           # and past it
    blocks[2, 5], blocks[2, 40] = 2 * meet, 2 * meet + 1
    blocks[4] = g.integers(0, 3, 64)
    blocks[5] = g.integers(0, 2 * meet + 3, 64)
    blocks[7, 63] = 70 * meet + 33
    blocks[8, ::9] = 9 * meet
    blocks[9, ::8] = 2 * meet
    blocks[-2] = g.integers(0, 2, 64)
    blocks[-1, 60:] = (1, 0, 4 * meet + 3, 2)
    return c


@pytest.mark.parametrize("depth,p,meet", [
    (7, 12, 13),                                           # products alone
    (8, 12, 13), (8, 16, 7), (8, 5, 76), (8, 1, 128),
    (9, 9, 23), (10, 4, 118), (11, 2, 128),
])
def test_coefficients_at_the_line_between_products_and_threads(depth, p, meet):
    import torch
    from paper_1009_3457_amd import _binding as B
    print(f"fgt coeffs depth={depth} p={p}", flush=True)
    nbox = 4 ** depth
    count = _counts(nbox, meet)
    ls = np.concatenate([[0], np.cumsum(count)])
    n = int(ls[-1])
    m = np.repeat(np.arange(nbox), count)
    ix, iy = (sum(((m >> (2 * b + s)) & 1) << b for b in range(depth)) for s in (0, 1))
    g = np.random.Generator(np.random.PCG64(3))
    xy = ((np.stack([ix, iy], 1) + 0.01 + 0.98 * g.random((n, 2))) / 2 ** depth).astype(np.float32)
    q = (g.random(n) + 0.5).astype(np.float32)
    sigma = float(np.float32(np.sqrt(2.0) * 2.0 ** -depth))
    A = B.fgt_hermite_coeffs(torch.from_numpy(xy).cuda(), torch.from_numpy(q).cuda(),
                             torch.from_numpy(ls.astype(np.int32)).cuda(), depth, p, sigma).cpu().numpy()
    ref = ofgt.hermite_coeffs(xy.astype(np.float64), q.astype(np.float64), ls.astype(np.int32), depth, p, sigma)
    assert not A[count == 0].any()
    # relative to the box's sum of magnitudes, which the FP64 sums are exact to
    mag = np.zeros(nbox)
    np.add.at(mag, m, q.astype(np.float64))
    assert np.all(np.abs(A - ref) <= 2.5e-7 * np.abs(ref) + 1e-15 * mag[:, None, None])
