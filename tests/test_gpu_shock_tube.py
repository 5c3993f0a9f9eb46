"""Long runs with characteristic variables: the viscous shock tube (Sec. 5.8,
500 x 250, Re 200, Pr 0.73, CFL 0.2).  The run amplifies rounding across its
shock, so single runs tell little; how many of a set of runs that differ by
1e-13 of the Courant number survive tells whether the kernels' rounding of the
Gauss-point values still suits it."""
import math

import numpy as np
import pytest

from gpu_common import GpuProblem, problem
from paper_2309_10534_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def shock_tube(fallback):
    W0, dx = I.viscous_shock_tube(500, 250)
    return W0, problem([500, 250], [dx, dx], bc=[("noslip", "noslip"), ("noslip", "reflective")], tau="viscous",
                       mu=1.0 / 200.0, prandtl=0.73, recon=1, fallback=fallback)


@pytest.mark.parametrize("fallback", [0, 1])
def test_characteristic_shock_tube_reaches_t1(torch_dev, fallback):
    """To t = 1 with no failure and no fallback taken, mass and energy kept to
    rounding (closed box), positive density and pressure."""
    W0, pr = shock_tube(fallback)
    gp = GpuProblem(pr)
    try:
        print(f"[shock tube] characteristic to t = 1, fallback={fallback}", flush=True)
        W, td, bad = gp.run(W0, 11000, cfl=0.2, t_end=1.0, t0=0.0)
        nfb = gp.t.tgks_fallback_count(gp.ctx)
    finally:
        gp.close()
    assert bad == 0 and nfb == 0 and abs(td[0] - 1.0) <= 1e-14
    rho, _, p = I.primitive(W)
    assert np.all(np.isfinite(W)) and rho.min() > 0.0 and p.min() > 0.0
    for c in (0, 3):
        assert abs(W[c].sum() - W0[c].sum()) <= 1e-12 * W0[c].sum()


def test_characteristic_shock_tube_survives_rounding(torch_dev):
    """Of ten runs to t = 0.25 (past the shock's reflection, where the losses
    lie) with Courant numbers 0.2 (1 + 1e-13 k) at least eight survive.  The
    rounding that the kernels keep lets 97 of 100 through (three misses in ten:
    chance 0.003); the one that lost the run lets a third through (eight of
    ten: chance 0.003)."""
    W0, pr = shock_tube(0)
    ok = []
    for k in range(10):
        gp = GpuProblem(pr)
        try:
            W, td, bad = gp.run(W0, 6000, cfl=0.2 * (1.0 + 1e-13 * k), t_end=0.25, t0=0.0)
        finally:
            gp.close()
        ok.append(bad == 0 and math.isfinite(td[1]) and abs(td[0] - 0.25) <= 1e-14)
        print(f"[shock tube] run {k}: t={td[0]:.4f} failures={bad}", flush=True)
    assert sum(ok) >= 8, ok
