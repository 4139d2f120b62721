"""The restriction entry by entry, in both precisions, against the transpose of
the oracle's prolongation matrix: at the block edges and box edges of small and
odd meshes every single node counts."""
import numpy as np
import pytest

import workloads as W

try:  # import at collection time: the first import on a fresh machine is slow
    import torch  # noqa: F401
except ImportError:  # pragma: no cover
    torch = None

pytestmark = pytest.mark.gpu

# coarse cells, levels, radius: one cell a side, the box but its corners, a few active blocks
CASES = [W.Workload(f"entries-d{d}-Q{k}-c{c}", d, k, n, coarse_cells=c, centers=((0.03, -0.02, 0.01)[:d],),
                    semi=((r,) * d,))
         for d in (2, 3) for k in (1, 2, 3) for c, n, r in ((1, 3, 0.8), (3, 2, 1.3), (5, 2, 0.6))]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_restriction_entries(w):
    from oracle import problem as OP
    from oracle.geometry import build_levels
    from oracle.transfer import prolongation
    from paper_2508_11608_amd import Problem

    levels = build_levels(OP.shapes_of(w), w.dim, w.k, w.n_levels, w.coarse_cells, w.lo, w.hi)
    P = Problem(w)
    try:
        for l in range(1, w.n_levels):
            pt = prolongation(levels[l - 1], levels[l]).T.tocsr()
            r = W.random_vector(levels[l].n_dofs, seed=31)
            want, size = pt @ r, abs(pt) @ abs(r)
            for fp32 in (False, True):
                print(f"\n[case] {w.name} level {l} fp32={fp32}", flush=True)
                P.set_precision(fp32)
                got = P.restrict(l, torch.from_numpy(r).cuda()).cpu().numpy()
                # d passes, each a sum of at most 4k - 1 products with rounded weights, of rounded entries: at most
                # d (4k + 1) + 1 roundings a term, half an eps each; as much again for the matrix product
                eps = np.finfo(np.float32 if fp32 else np.float64).eps
                bad = np.abs(got - want) > eps * (w.dim * (4 * w.k + 1) + 1) * size
                assert not bad.any(), (l, fp32, np.flatnonzero(bad)[:10])
    finally:
        P.close()
        torch.cuda.synchronize()
