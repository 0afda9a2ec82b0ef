"""Fast Gauss transform through its Hermite stage (arXiv:1009.3457, Sec. 2.2
and Sec. 4.2) on the library's kernels (include/fgt2d.h).

    G(y) = sum_i q_i exp(-|x_i - y|^2 / (2 sigma^2))

Sources are grouped into the 4^depth boxes of the uniform grid over [0,1]^2;
each box's Hermite series (p x p terms) is evaluated at the targets whose box
lies within K boxes of it in both directions.
"""
from __future__ import annotations

import torch

from . import _binding as B


def gauss_transform(xy: torch.Tensor, q: torch.Tensor, targets: torch.Tensor, depth: int, p: int,
                    sigma: float, K: int) -> torch.Tensor:
    """G at the targets (float32 [nt], original order).  xy [n, 2], q [n] and
    targets [nt, 2] float32 on the GPU, points in [0,1]^2."""
    xy, q, targets = xy.contiguous(), q.contiguous(), targets.contiguous()
    _, ls, flag, xs, qs = B.sort_points(xy, q, depth, want_perm=False)
    A = B.fgt_hermite_coeffs(xs, qs, ls, depth, p, sigma)
    tperm, _, tflag, ts, _ = B.sort_points(targets, None, depth)  # box order keeps each wave within a few boxes
    G = B.fgt_hermite_eval(ts, depth, p, sigma, K, A, place=tperm, from_coeffs=True)
    B.check_domain(flag, tflag)  # read after everything has been enqueued
    return G
