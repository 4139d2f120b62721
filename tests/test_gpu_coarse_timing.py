"""Kernel timing of the coarse solve: one launch on level 0 per V-cycle, whether
the V-cycle ends there or in the dense matrix of several levels, replayed or
launched kernel by kernel."""
import pytest

import workloads as W

try:  # import at collection time: the first import on a fresh machine is slow
    import torch  # noqa: F401
except ImportError:  # pragma: no cover
    torch = None

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w", [W.disc_q2(), W.offcentre_ball(3, 2)], ids=["matrix-on-level-2", "no-matrix"])
def test_coarse_solves_count_on_level_0(w):
    from paper_2508_11608_amd import Problem

    P = Problem(w)
    try:
        r = torch.from_numpy(W.random_vector(P.ndofs(), seed=21)).cuda()
        for graphs in (True, False):
            P.set_graphs(graphs)
            for level in (0, None):
                P.timing(["coarse"], level=level)
                for _ in range(3):
                    P.vcycle(r)
                assert [P.timing_read("coarse", l)[0] for l in range(w.n_levels)] == [3] + [0] * (w.n_levels - 1)
        P.timing([])
    finally:
        P.close()
