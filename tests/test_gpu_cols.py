"""The multi-column cut step (cell rows and local solves on the matrix cores,
ghost rows by sum factorisation) at the shapes where its tiling can go wrong:
every degree and dimension (cell rows of 1 to 27 of a tile's 16 rows, matrices
of 4 to 64 columns, local systems of 1 to 125 unknowns), first and last column
counts, narrow and wide blocks.  FP64 against the oracle's V-cycle, both
precisions bitwise between block widths."""
import numpy as np
import pytest

import oracle_cache
import workloads as W

try:  # import at collection time: the first import on a fresh machine is slow
    import torch  # noqa: F401
except ImportError:  # pragma: no cover
    torch = None

pytestmark = pytest.mark.gpu

CASES = [W.offcentre_disc(1, 3), W.offcentre_disc(3, 3), W.disc_union(2, 3), W.offcentre_ball(1, 3),
         W.ball_union(2, 2), W.offcentre_ball(3, 2)]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_columns_and_block_widths(w):
    import torch
    from paper_2508_11608_amd import Problem

    levels, mats, prols, H = oracle_cache.build(w)
    P = Problem(w)
    try:
        n = levels[-1].n_dofs
        rn = W.random_vector(n, seed=77, nrhs=8)
        r = torch.from_numpy(rn).cuda()
        for fp32 in (False, True):
            P.set_precision(fp32)
            for nrhs in (1, 5, 8):
                z = {}
                for small in (0, 1536, 1 << 30):
                    print(f"\n[case] {w.name} fp32={fp32} nrhs={nrhs} small_cut_launch={small}", flush=True)
                    P.set_launch(small_cut_launch=small)
                    z[small] = P.vcycle_multi(r[:nrhs].contiguous()).cpu().numpy()
                assert np.array_equal(z[0], z[1536]) and np.array_equal(z[0], z[1 << 30])
                if not fp32:
                    for c in range(nrhs):
                        zo = H.vcycle(rn[c])
                        assert np.abs(z[0][c] - zo).max() < 1e-10 * np.abs(zo).max(), c
    finally:
        P.close()
        torch.cuda.synchronize()
