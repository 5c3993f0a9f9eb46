"""The 1-D kernel's options at the sizes where its wavefronts (58 cells) and
blocks (one wavefront, four above 14,848 cells) begin and end: characteristic
variables, prescribed sides at both ends, the first-order fallback with the cell
that needs it beside a wavefront's first and last faces, Navier-Stokes, the
comparison schemes.  One step with flags against the oracle, and three CFL steps
of tgks_run against single steps."""
import math

import numpy as np
import pytest

from gpu_common import GpuProblem, assert_close, orc_params, problem
from paper_2309_10534_amd import inputs as I

pytestmark = pytest.mark.gpu

SIZES = [3, 4, 57, 58, 59, 61, 62, 115, 116, 117, 232, 233, 14848, 14849, 59392, 59393]
NS = dict(tau="viscous", mu=1e-3, prandtl=0.72)


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def field(n):
    rng = np.random.default_rng(n)
    x = (np.arange(n) + 0.5) / n
    rho = 1.0 + 0.2 * np.sin(2 * np.pi * x) + 0.5 * (x > 0.6) + 1e-3 * rng.normal(size=n)
    return I.conservative(rho, [0.3 * np.cos(2 * np.pi * x)], 1.0 + 0.4 * (x < 0.3) + 0.0 * x)


def prescribed():
    """Both ends given, the left one switching between two states in time."""
    A = I.conservative(np.array([1.3]), [np.array([0.2])], np.array([1.1])).reshape(-1)
    B = I.conservative(np.array([0.9]), [np.array([-0.1])], np.array([0.8])).reshape(-1)
    return dict(bc=[("prescribed", "prescribed")], states=(A.tolist(), B.tolist()),
                lines={(0, 0): (-1e-9, 0.0, 1.0), (0, 1): (math.inf, 0.0, 0.0)}, far={(0, 0): "state_b"})


OPTIONS = {
    "char": dict(recon=1, bc=[("periodic", "periodic")]),
    "char ns walls": dict(recon=1, bc=[("noslip", "reflective")], **NS),
    "prescribed": prescribed(),
    "prescribed char ns": dict(recon=1, **prescribed(), **NS),
    "ns": dict(bc=[("transmissive", "noslip")], **NS),
    "weno_ao": dict(scheme="weno_ao", bc=[("reflective", "transmissive")]),
    "teno5 ns": dict(scheme="teno5", bc=[("periodic", "periodic")], **NS),
    "weno_z": dict(scheme="weno_z", bc=[("transmissive", "transmissive")]),
}


@pytest.mark.parametrize("option", list(OPTIONS))
def test_line_kernel_options(orc, torch_dev, option):
    for n in SIZES:
        W = field(n)
        pr = problem([n], [1.0 / n], **OPTIONS[option])
        P = orc_params(orc, pr)
        dt = orc.cfl_dt(P, W, 0.5)
        Wo, fo, Wso, bado = orc.step(P, W, dt, want_flags=True, want_wstar=True)
        print(f"[line] {option} n={n}", flush=True)
        gp = GpuProblem(pr)
        try:
            Wg, Wsg, fg, badg = gp.step(W, dt, t0=0.0)
            Wr, td, badr = gp.run(W, 3, cfl=0.5, t0=0.0)
            Wc, t = W, 0.0
            for _ in range(3):
                d = gp.cfl_dt(Wc, 0.5)
                Wc = gp.step(Wc, d, flags=False, t0=t)[0]
                t += d
        finally:
            gp.close()
        assert badg == bado == 0 and badr == 0
        assert np.array_equal(fg, fo), (option, n, np.count_nonzero(fg != fo))
        assert_close(Wsg, Wso, 1e-10, f"W* {option} n={n}")
        assert_close(Wg, Wo, 1e-10, f"{option} n={n}")
        assert np.array_equal(Wr, Wc) and td[0] == t


@pytest.mark.parametrize("recon", [0, 1])
@pytest.mark.parametrize("n,at", [(125, 57), (125, 58), (125, 61), (125, 124), (58, 57), (59, 58), (62, 0), (63, 62)])
def test_line_kernel_fallback_counts(orc, torch_dev, recon, n, at):
    """Side states that the fallback replaces at faces which two wavefronts
    evaluate are counted once, and the replacements are the oracle's."""
    # a cold cell between two hot ones that recede from it into a cold gas
    i = np.arange(n)
    p = np.where(abs(i - at) == 1, 1.0, 1e-5)
    W = I.conservative(field(n)[0], [np.where(i < at, -0.1, np.where(i > at, 0.2, 0.0))], p)
    pr = problem([n], [1.0 / n], bc=[("transmissive", "reflective")], recon=recon, fallback=1)
    P = orc_params(orc, pr)
    nfb = [0]
    Wo, fo, _, bado = orc.step(P, W, 1e-6, want_flags=True, fallbacks=nfb)
    print(f"[line] fallback recon={recon} n={n} at={at}: {nfb[0]} replaced", flush=True)
    gp = GpuProblem(pr)
    try:
        Wg, _, fg, badg = gp.step(W, 1e-6)
    finally:
        gp.close()
    assert gp.fallbacks == nfb[0] > 0 and badg == bado
    assert np.array_equal(fg, fo)
    assert_close(Wg, Wo, 1e-10, f"fallback recon={recon} n={n} at={at}")
