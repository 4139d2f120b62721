"""Groups whose members apply different numbers of levels as one dense matrix:
the finest level below the top with at most 2048 DoFs, which differs between
domains of one lattice shape.  Every member's grouped V-cycle and grouped PCG
equal, bit for bit, what the member gives alone."""
import numpy as np
import pytest

import workloads as W

try:  # import at collection time: the first import on a fresh machine is slow
    import torch  # noqa: F401
except ImportError:  # pragma: no cover
    torch = None

pytestmark = pytest.mark.gpu


def _balls(dim, n_levels, *radii):
    return [W.Workload(f"ball-d{dim}-r{r}", dim, 2, n_levels, centers=((0.02 * i,) + (0.0,) * (dim - 1),),
                       semi=((r,) * dim,)) for i, r in enumerate(radii)]


# domains of one lattice shape, the level of each one's matrix (0: none)
GROUPS = {
    "2d-Q2": (_balls(2, 5, 0.80, 0.70, 0.74), (2, 3, 2)),
    "2d-Q3": ([W.Workload("ellipses-a", 2, 3, 5, centers=((0.0226, 0.2991), (0.2343, 0.1754)),
                          semi=((0.4720, 0.4841), (0.4972, 0.4316))),
               W.Workload("ellipses-b", 2, 3, 5, centers=((-0.2821, 0.1769), (-0.0881, 0.2198)),
                          semi=((0.4050, 0.4926), (0.3533, 0.3591)))], (2, 3)),
    "3d-Q2": (_balls(3, 4, 0.70, 0.75), (1, 0)),
}


@pytest.mark.parametrize("fp32", [False, True], ids=["fp64", "fp32"])
@pytest.mark.parametrize("name", list(GROUPS))
def test_members_on_both_sides_of_the_limit(name, fp32):
    from paper_2508_11608_amd import Group, Problem

    ws, want = GROUPS[name]
    print(f"\n[case] {name} fp32={fp32}", flush=True)
    ps = [Problem(w, fp32=fp32) for w in ws]
    try:
        level = tuple(max([l for l in range(1, w.n_levels - 1) if p.ndofs(l) <= 2048], default=0)
                      for w, p in zip(ws, ps))
        assert level == want
        g = Group(ps)
        try:
            # the first grouped V-cycle captures the graph, the others replay it
            for rep in range(3):
                rs = [torch.from_numpy(W.random_vector(p.ndofs(), seed=700 + 10 * rep + i)).cuda()
                      for i, p in enumerate(ps)]
                for p, r, z in zip(ps, rs, g.vcycle(rs)):
                    assert torch.equal(z, p.vcycle_multi(r[None, :])[0]), rep
            bs = [torch.from_numpy(np.ascontiguousarray(p.rhs_manufactured())).cuda() for p in ps]
            xs, infos = g.solve(bs, rtol=1e-8, maxit=200)
            for p, b, x, info in zip(ps, bs, xs, infos):
                x1, i1 = p.solve_multi(b[None, :], rtol=1e-8, maxit=200)
                assert info["status"] == 0 and info["iterations"] == i1[0]["iterations"]
                assert torch.equal(x, x1[0])
        finally:
            g.close()
    finally:
        for p in ps:
            p.close()
        torch.cuda.synchronize()
