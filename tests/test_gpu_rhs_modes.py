"""The device load vector's rule for Fourier data, against the library's host
assembly of the same quadrature: wavenumbers that take every way through the
powers of e^{i pi t} (negative, repeated, consecutive, far apart), point counts
with and without a kernel of their own, and domains whose kinked cells hold
more quadrature columns than one block takes."""
import numpy as np
import pytest

import workloads as W

try:  # import at collection time: the first import on a fresh machine is slow
    import torch  # noqa: F401
except ImportError:  # pragma: no cover
    torch = None

pytestmark = pytest.mark.gpu


def _kappa(dim, kind):
    if kind == "run":  # every wavenumber of a run, more of them than products are taken in a row
        return np.array([[q % 13] + [(5 * q) % 7] * (dim - 1) for q in range(20)], dtype=np.int32)
    if kind == "mixed":
        return np.array([[-7, 3, -2][:dim], [0, 0, 1][:dim], [40, -1, 5][:dim], [-7, 9, 9][:dim], [9, 8, 0][:dim],
                         [10, -40, 17][:dim]], dtype=np.int32)
    return np.zeros((1 if kind == "constant" else 0, dim), dtype=np.int32)


@pytest.mark.parametrize("quad_n", [5, 14, 16])
@pytest.mark.parametrize("w", [W.disc_union(1, 3), W.ball_union(2, 2), W.offcentre_ball(3, 2)], ids=lambda w: w.name)
def test_modes_match_host_assembly(w, quad_n):
    import torch
    from paper_2508_11608_amd import Problem

    P = Problem(w, quad_n=quad_n)
    try:
        for kind in ("run", "mixed", "constant", "none"):
            print(f"\n[case] {w.name} quad_n={quad_n} modes {kind}", flush=True)
            kappa = _kappa(w.dim, kind)
            n = len(kappa)
            rng = np.random.default_rng(n)
            amp, phase = rng.standard_normal(n), rng.uniform(0.0, 2.0 * np.pi, n)
            bd = P.rhs_fourier_device(kappa, amp, phase).cpu().numpy()
            bh = P.rhs_fourier(kappa, amp, phase)
            # a mode's phase carries a few roundings of its own size on either side, and its integral against a
            # basis function is at most the volume of the function's support; |psi| <= 1
            eps = np.finfo(np.float64).eps
            size = 2.0 * np.pi + np.pi * np.abs(kappa).sum(axis=1)
            h = (w.hi - w.lo) / w.fine_cells
            tol = 8.0 * eps * float(np.sum(np.abs(amp) * (8.0 + size))) * (2.0 * h) ** w.dim
            d = np.abs(bd - bh).max()
            print(f"  difference {d:.2e}, tolerance {tol:.2e}", flush=True)
            assert d <= tol
    finally:
        P.close()
        torch.cuda.synchronize()
