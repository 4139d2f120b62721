"""The device load vector at phases of many periods: the same as at the phases
reduced to one period beforehand (in extended precision)."""
import numpy as np
import pytest

import workloads as W

try:  # import at collection time: the first import on a fresh machine is slow
    import torch  # noqa: F401
except ImportError:  # pragma: no cover
    torch = None

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("periods", [1, 16, 10000])
@pytest.mark.parametrize("w", [W.offcentre_disc(3, 3), W.offcentre_ball(2, 2)], ids=lambda w: w.name)
def test_phases_of_many_periods(w, periods):
    from paper_2508_11608_amd import Problem

    pi = np.longdouble("3.14159265358979323846264338327950288")
    kappa, amp, _ = W.fourier_modes(w.dim, seed=41)
    phase = np.random.default_rng(42).uniform(-2 * np.pi * periods, 2 * np.pi * periods, len(amp))
    turns = phase.astype(np.longdouble) / (2 * pi)
    reduced = (2 * pi * (turns - np.floor(turns))).astype(np.float64)
    P = Problem(w)
    try:
        one = P.rhs_fourier_device(np.zeros((1, w.dim), np.int32), np.ones(1), np.zeros(1))  # integrals of the basis
        b, b0 = P.rhs_fourier_device(kappa, amp, phase), P.rhs_fourier_device(kappa, amp, reduced)
        # the reduced phase is rounded at up to 2 pi (8 eps / 2 is its ulp), then both are divided by pi and rounded
        tol = 16 * np.finfo(float).eps * np.abs(amp).sum() * float(one.abs().max())
        print(f"\n  {w.name} {periods}: {float((b - b0).abs().max()):.2e}, tolerance {tol:.2e}", flush=True)
        assert float((b - b0).abs().max()) <= tol
    finally:
        P.close()
        torch.cuda.synchronize()
