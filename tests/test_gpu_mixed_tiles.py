"""The operator on tiles that hold special or inactive cells, at the edges of its
3-D matrix-core form: meshes that are no multiple of a tile (1, 3, 5 and 6 cells a
direction), tiles with no, few and more than 16 regular cells, one and several
columns' worth of tiles per block, both precisions, against the oracle's assembled
matrix."""
import numpy as np
import pytest

import oracle_cache
import workloads as W

try:  # import at collection time: the first import on a fresh machine is slow
    import torch  # noqa: F401
except ImportError:  # pragma: no cover
    torch = None

pytestmark = pytest.mark.gpu


def _w(k, coarse, n_levels, radius):
    return W.Workload(f"mixed-Q{k}-c{coarse}-r{radius}", 3, k, n_levels, coarse_cells=coarse,
                      centers=((0.03, -0.02, 0.01),), semi=((radius,) * 3,))


CASES = [_w(2, 3, 2, 0.7), _w(2, 5, 1, 1.3), _w(2, 1, 3, 0.9), _w(3, 3, 1, 1.3), _w(3, 3, 2, 0.6)]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_operator_matches_oracle(w):
    import torch
    from paper_2508_11608_amd import Problem

    levels, mats, *_ = oracle_cache.build(w)
    P = Problem(w)
    try:
        for level in range(w.n_levels):
            x = W.random_vector(levels[level].n_dofs, seed=31 + level)
            want = mats[level] @ x
            # FP32 rounding of x and the matrix entries, sums of at most a row's entries
            size = abs(mats[level]) @ np.abs(x)
            for fp32 in (False, True):
                P.set_precision(fp32)
                for blocks in (2048, 1):
                    print(f"\n[case] {w.name} level {level} fp32={fp32} max_blocks={blocks}", flush=True)
                    P.set_launch(max_blocks=blocks)
                    y = P.apply(level, torch.from_numpy(x).cuda()).cpu().numpy()
                    if fp32:
                        row = np.diff(mats[level].tocsr().indptr).max()
                        assert (np.abs(y - want) <= row * np.finfo(np.float32).eps * size.max()).all()
                    else:
                        assert np.abs(y - want).max() < 1e-12 * np.abs(want).max()
            P.set_launch()
            P.set_precision(False)
    finally:
        P.close()
        torch.cuda.synchronize()
