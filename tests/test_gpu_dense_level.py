"""V-cycles whose smallest levels are applied as one dense matrix (the finest
level below the top with at most 2048 DoFs): against the oracle's level by level
V-cycle for every dimension and degree, with the matrix on level 1 and on higher
levels, one and several columns, both precisions, and with the patch-local ghost
coupling, which runs every level, switched on and off in between."""
import numpy as np
import pytest

import oracle_cache
import workloads as W

try:  # import at collection time: the first import on a fresh machine is slow
    import torch  # noqa: F401
except ImportError:  # pragma: no cover
    torch = None

pytestmark = pytest.mark.gpu

# (domain, the level of its matrix): 1,637 (made in several batches), 1,217, 1,669, 479, 153 and no DoFs
CASES = [(W.offcentre_ball(2, 3), 1), (W.offcentre_ball(1, 4), 2), (W.offcentre_disc(2, 5), 3),
         (W.offcentre_disc(3, 4), 2), (W.disc_q2().with_levels(3), 1), (W.offcentre_ball(3, 2), 0)]


def _rel(a, b):
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


@pytest.mark.parametrize("w,level", CASES, ids=lambda v: getattr(v, "name", str(v)))
def test_dense_levels_match_oracle(w, level):
    import torch
    from paper_2508_11608_amd import Problem

    levels, mats, prols, H = oracle_cache.build(w)
    assert level == max([l for l in range(1, w.n_levels - 1) if levels[l].n_dofs <= 2048], default=0)
    H32 = oracle_cache.hierarchy32(w)
    P = Problem(w)
    try:
        rn = W.random_vector(levels[-1].n_dofs, seed=91, nrhs=3)
        r = torch.from_numpy(rn).cuda()
        for fp32 in (False, True):
            print(f"\n[case] {w.name} matrix on level {level} fp32={fp32}", flush=True)
            P.set_precision(fp32)
            one = P.vcycle(r[0].contiguous())
            many = P.vcycle_multi(r)
            P.set_ghost_coupling(True)
            P.vcycle(r[0].contiguous())
            P.set_ghost_coupling(False)
            assert torch.equal(P.vcycle(r[0].contiguous()), one)
            for c in range(3):
                zo = H.vcycle(rn[c])
                # FP32 bound of the parity tests: 10x the oracle's own float32 deviation + 1e-6
                tol = 10.0 * _rel(H32.vcycle(rn[c]).astype(np.float64), zo) + 1e-6 if fp32 else 1e-10
                for z in [many[c]] + ([one] if c == 0 else []):
                    assert _rel(z.cpu().numpy(), zo) < tol, (fp32, c)
    finally:
        P.close()
        torch.cuda.synchronize()
