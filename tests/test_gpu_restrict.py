"""The restriction against the prolongation it is the transpose of, <P x, r> =
<x, P^T r>, at the sizes where its blocks can go wrong: meshes that are no
multiple of a block (odd cell counts, one cell a side), blocks at the box edge
that own the last node layer, and levels with few active blocks."""
import numpy as np
import pytest

import workloads as W

try:  # import at collection time: the first import on a fresh machine is slow
    import torch  # noqa: F401
except ImportError:  # pragma: no cover
    torch = None

pytestmark = pytest.mark.gpu


def _w(dim, k, coarse, n_levels, radius):
    return W.Workload(f"edge-d{dim}-Q{k}-c{coarse}-r{radius}", dim, k, n_levels, coarse_cells=coarse,
                      centers=((0.03, -0.02, 0.01)[:dim],), semi=((radius,) * dim,))


# radius 1.3 covers the box except its corners (edge blocks own active nodes)
CASES = [_w(d, k, c, n, r) for d in (2, 3) for k in (1, 2, 3)
         for c, n, r in ((1, 3, 0.8), (3, 2, 1.3), (5, 2, 0.6))]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_restriction_is_the_transpose(w):
    import torch
    from paper_2508_11608_amd import Problem

    P = Problem(w)
    try:
        for level in range(1, w.n_levels):
            nf, nc = P.ndofs(level), P.ndofs(level - 1)
            x = torch.from_numpy(W.random_vector(nc, seed=11)).cuda()
            r = torch.from_numpy(W.random_vector(nf, seed=12)).cuda()
            for fp32 in (False, True):
                print(f"\n[case] {w.name} level {level} fp32={fp32}", flush=True)
                P.set_precision(fp32)
                px, rr = P.prolongate(level, x), P.restrict(level, r)
                # P is a tensor product of 1-D weights of at most 1.7 (Q3) in absolute value, so each side is a sum
                # of at most nf (k+1)^d terms below 1.7^d |x| |r|: eps times the sum of the absolute products
                eps = np.finfo(np.float32 if fp32 else np.float64).eps
                size = float((px.abs() * r.abs()).sum() + (x.abs() * rr.abs()).sum())
                diff = abs(float((px * r).sum() - (x * rr).sum()))
                tol = eps * 8 * (4 * w.k) ** w.dim * max(size, 1.0)
                print(f"  difference {diff:.2e}, tolerance {tol:.2e}", flush=True)
                assert diff <= tol
            P.set_precision(False)
    finally:
        P.close()
        torch.cuda.synchronize()
