"""The near field with many rows and few columns, where waves take windows of
64 rows: leaves of few columns in pieces of 64, others of 32, against the FP64 oracle.
Tolerance as for the other windows: 1e-5 of the norm."""
import numpy as np
import pytest

import oracle
import synthetic as sy
from tests._inputs import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,depth,kind", [
    (524296, 65537, 7, "mixed"),     # an eighth: windows of 64, pieces of 32 and 64
    (524296, 65538, 7, "mixed"),     # one column more: windows of 32
    (524288, 500, 7, "uniform"),     # 32 rows a leaf
    (524287, 500, 6, "uniform"),     # one row less: windows of 32
    (600003, 20, 3, "uniform"),      # leaves of thousands of rows
    (600000, 1, 5, "mixed"),
    (270000, 3000, 7, "mixed"),
    (262143, 500, 6, "uniform"),     # windows of 16
])
def test_many_rows_and_few_columns_match_oracle(rows, cols, depth, kind):
    import torch
    from paper_1009_3457_amd import _binding as B
    print(f"p2p rows={rows} cols={cols} depth={depth} {kind}", flush=True)
    make = sy.uniform if kind == "uniform" else sy.mixed
    r, c = make(rows, 1), make(cols, 2)
    k = min(cols // 3, 50)
    r[:k] = c[:k]  # coincident pairs
    rp, rls = oracle.build_tree(r.astype(np.float64), depth)
    cp, cls = oracle.build_tree(c.astype(np.float64), depth)
    r, c = r[rp], c[cp]
    q, w = sy.charges(cols, 3), sy.charges(rows, 4)
    R, C, RL, CL, Q, W = (torch.from_numpy(np.ascontiguousarray(a)).cuda()
                          for a in (r, c, rls.astype(np.int32), cls.astype(np.int32), q, w))
    phi, f = B.p2p(C, Q, CL, R, RL, depth)
    pr, fr = oracle.p2p(c.astype(np.float64), q.astype(np.float64), cls, r.astype(np.float64), rls, depth)
    assert rel(phi.cpu().numpy(), pr) < 1e-5 and rel(f.cpu().numpy(), fr) < 1e-5
    g = (sy.charges(cols, 5) + 1j * sy.charges(cols, 6)).astype(np.complex64)
    e = (sy.charges(cols, 7) + 1j * sy.charges(cols, 8)).astype(np.complex64)
    for cp, ce in ((g, e), (g.real.astype(np.complex64), None)):
        gq, G = torch.zeros(rows, device="cuda"), torch.zeros(rows, dtype=torch.complex64, device="cuda")
        dev = lambda a: None if a is None else torch.from_numpy(a).cuda()  # noqa: E731
        B.p2p_backward(R, W, RL, C, CL, depth, dev(cp), dev(ce), gq, G)
        wide = lambda a: None if a is None else a.astype(np.complex128)  # noqa: E731
        gqr, Gr = oracle.p2p_transpose(r.astype(np.float64), w.astype(np.float64), rls, c.astype(np.float64), cls, depth,
                                       wide(cp), wide(ce))
        assert rel(gq.cpu().numpy(), gqr) < 1e-5 and rel(G.cpu().numpy(), Gr) < 1e-5
