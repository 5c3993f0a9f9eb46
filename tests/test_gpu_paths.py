"""The routes a step can take through the kernels, at the sizes and on the
data where each begins and ends: 1-D grids around the cells that one wavefront
(58) and one block (232 above 59,392 cells) own, the steps that take their
clock from the step before (up to 256 partial minima), the time step of small
grids in one block (up to 4,096 cells), and the smooth / general forms of the
tangential selections, which must agree to the bit; the two tile shapes of the
3-D face kernel."""
import numpy as np
import pytest

from gpu_common import GpuProblem, assert_close, orc_params, problem
from paper_2309_10534_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


BC1 = [("periodic", "periodic"), ("transmissive", "reflective"), ("noslip", "transmissive")]


def field_1d(n, seed):
    rng = np.random.default_rng(seed)
    x = (np.arange(n) + 0.5) / n
    rho = 1.0 + 0.2 * np.sin(2 * np.pi * x) + 0.5 * (x > 0.6) + 1e-3 * rng.normal(size=n)
    return I.conservative(rho, [0.3 * np.cos(2 * np.pi * x)], 1.0 + 0.4 * (x < 0.3) + 0.0 * x)


@pytest.mark.parametrize("n", [3, 4, 57, 58, 59, 60, 61, 62, 63, 64, 115, 116, 117, 123, 124, 125, 174, 175, 186, 187,
                               4096, 4097, 14848, 14849, 59392, 59393, 63488, 63489])
def test_line_kernel_sizes(orc, torch_dev, n):
    """One step with flags and three CFL steps of tgks_run against the
    oracle, every boundary pair, and the failure counter of a state that is
    non-physical at the last face a wavefront owns."""
    for k, bc in enumerate(BC1 if n < 1000 else BC1[1:2]):
        pr = problem([n], [1.0 / n], bc=[bc])
        W = field_1d(n, 7 * n + k)
        P = orc_params(orc, pr)
        dt = orc.cfl_dt(P, W, 0.5)
        Wo, fo, Wso, bado = orc.step(P, W, dt, want_flags=True, want_wstar=True)
        print(f"[paths] 1-D n={n} bc={bc}", flush=True)
        gp = GpuProblem(pr)
        try:
            Wg, Wsg, fg, badg = gp.step(W, dt)
            Wr, td, badr = gp.run(W, 3, cfl=0.5)
            Wc = W
            for _ in range(3):
                Wc = gp.step(Wc, gp.cfl_dt(Wc, 0.5), flags=False)[0]
        finally:
            gp.close()
        assert badg == bado and badr == 0
        assert np.array_equal(fg, fo), (n, bc)
        assert_close(Wsg, Wso, 1e-10, f"W* n={n} {bc}")
        assert_close(Wg, Wo, 1e-10, f"n={n} {bc}")
        assert np.array_equal(Wr, Wc) and td[0] > 0


@pytest.mark.parametrize("t_end", [0.0, 0.02])
@pytest.mark.parametrize("sizes", [[57, 231, 232, 233, 465], [40, 59392], [40, 59393]])
def test_batch_clocks_between_steps(torch_dev, sizes, t_end):
    """Batches of grids around a block's 232 cells and the 256 partial minima
    up to which a step takes its clock from the step before: states, times,
    time steps and step counts of single runs, to the bit, eager and captured,
    with instances that stop at t_end after different numbers of steps."""
    from paper_2309_10534_amd import tgks
    from gpu_common import gpu_params
    torch, steps = torch_dev, 7
    probs = [(field_1d(n, n), problem([n], [1.0 / min(n, 500)], bc=[BC1[k % 3]])) for k, n in enumerate(sizes)]
    ref = []
    for W, pr in probs:
        gp = GpuProblem(pr)
        try:
            ref.append(gp.run(W, steps, cfl=0.5, t_end=t_end))
        finally:
            gp.close()
    b = tgks.tgks_batch_create([gpu_params(pr) for _, pr in probs])
    try:
        off = tgks.tgks_batch_offsets(b)
        W0 = torch.from_numpy(tgks.pack([W for W, _ in probs])).cuda()
        td = torch.zeros(2 * len(sizes), dtype=torch.float64, device="cuda")
        for graph in (False, True, True):
            W = W0.clone()
            tgks.tgks_batch_run(b, W, steps, 0.5, t_end, td, graph)
            torch.cuda.synchronize()
            out = tgks.unpack(W.cpu().numpy(), off, [w.shape for w, _ in probs])
            clock = td.cpu().numpy().reshape(-1, 2)
            count = tgks.tgks_batch_steps(b)
            for k, (Wr, tr, bad) in enumerate(ref):
                assert bad == 0 and np.array_equal(out[k], Wr), (sizes[k], graph)
                assert np.array_equal(clock[k], tr), (sizes[k], graph)
                assert count[k] == (steps if tr[1] > 0.0 else count[k]) <= steps
                assert t_end == 0.0 or tr[1] > 0.0 or abs(clock[k][0] - t_end) < 1e-13
    finally:
        tgks.tgks_batch_destroy(b)


@pytest.mark.parametrize("n,at", [(125, 57), (125, 58), (125, 61), (125, 62), (125, 124), (58, 57), (59, 58),
                                  (62, 61), (63, 62)])
def test_line_kernel_counts_each_failure_once(orc, torch_dev, n, at):
    """A cell of negative pressure beside a wavefront's first and last faces:
    the faces on both sides of a boundary between wavefronts are evaluated
    by both and counted by one."""
    W = field_1d(n, n)
    W[2, at] = 0.01
    W[1, at] = 1.0
    pr = problem([n], [1.0 / n])
    P = orc_params(orc, pr)
    Wo, fo, _, bado = orc.step(P, W, 1e-6, want_flags=True)
    print(f"[paths] 1-D n={n} negative pressure at {at}", flush=True)
    gp = GpuProblem(pr)
    try:
        _, _, fg, badg = gp.step(W, 1e-6)
    finally:
        gp.close()
    assert badg == bado > 0
    assert np.array_equal(fg, fo)


def mixed(shape, level, seed):
    """A field whose third differences reach `level` of its first ones: 0
    constant, small values smooth, 0.1 the edge of what counts as smooth."""
    rng = np.random.default_rng(seed)
    D = len(shape)
    x = np.meshgrid(*[(np.arange(n) + 0.5) / n for n in shape[::-1]], indexing="ij")
    s = sum(np.sin(2 * np.pi * (c + 0.1 * k)) for k, c in enumerate(x)) / D
    f = lambda a: a * (s + level * rng.normal(size=s.shape) / 30.0) if level is not None else 0.0 * s
    rho = 1.0 + f(0.2)
    if level is not None:
        rho = rho + (0.7 if level > 0.5 else 0.0) * (x[-1] > 0.5)
    return I.conservative(rho, [0.2 + f(0.1) for _ in range(D)], 1.0 + f(0.3))


@pytest.mark.parametrize("level", [None, 0.0, 1e-6, 0.03, 0.1, 0.3, 1.0])
@pytest.mark.parametrize("shape", [(41, 37), (64, 16), (11, 9, 13)])
def test_smooth_and_general_selections_agree(torch_dev, shape, level):
    """The step that records its flags takes the general form of every
    tangential selection, the plain step the smooth one where a wavefront
    allows it: the same bits on constant, smooth, rough and mixed data."""
    D = len(shape)
    W = mixed(shape, level, 5)
    kw = dict(tau="viscous", mu=1e-3, prandtl=0.72) if level == 0.03 else {}
    bc = [("periodic", "periodic"), ("reflective", "transmissive"), ("noslip", "periodic")][:D]
    bc = [b if "periodic" not in b or b == ("periodic", "periodic") else ("noslip", "noslip") for b in bc]
    pr = problem(list(shape), [1.0 / max(shape)] * D, bc=bc, **kw)
    print(f"[paths] selections {shape} level={level}", flush=True)
    gp = GpuProblem(pr)
    try:
        dt = gp.cfl_dt(W, 0.4)
        a, sa, _, ba = gp.step(W, dt, flags=True)
        b, sb, _, bb = gp.step(W, dt, flags=False)
    finally:
        gp.close()
    assert ba == bb == 0
    assert np.array_equal(sa, sb) and np.array_equal(a, b)


@pytest.mark.parametrize("shape", [(1500,), (70, 45)])
@pytest.mark.parametrize("ct,q,eps", [(1e-7, 6, 1e-40), (1e-5, 6, 1e-12), (1e-3, 2, 1e-40), (0.1, 1, 1e-6),
                                      (0.3, 6, 1e-40), (0.34, 5, 1e-40), (0.6, 6, 1e-8), (1e-5, 16, 0.0)])
def test_teno5_cutoffs_with_spread_indicators(orc, torch_dev, shape, ct, q, eps):
    """TENO5 cut-off flags of one step equal to the oracle's, bit for bit, on
    data whose differences span fifteen decades from cell to cell (with
    constant stretches), for cut-offs that keep everything, split the stencils
    or keep none, and powers that overflow; the states agree too."""
    rng = np.random.default_rng(int(1e6 * ct) + q)
    n = int(np.prod(shape))
    amp = np.repeat(10.0 ** rng.uniform(-16, -1, size=n // 5 + 1), 5)[:n]
    amp *= rng.random(n) < 0.9
    field = lambda: (1.0 + amp * rng.uniform(-1, 1, size=n)).reshape(shape[::-1])
    W = I.conservative(field(), [0.2 * field() for _ in shape], field())
    pr = problem(list(shape), [1.0 / m for m in shape], bc="periodic", scheme="teno5", ct1=ct, q=q, eps=eps)
    P = orc_params(orc, pr)
    dt = orc.cfl_dt(P, W, 0.3)
    Wo, fo, _, bado = orc.step(P, W, dt, want_flags=True)
    print(f"[paths] teno5 {shape} ct={ct} q={q}", flush=True)
    gp = GpuProblem(pr)
    try:
        Wg, _, fg, badg = gp.step(W, dt)
    finally:
        gp.close()
    assert np.array_equal(fg, fo), np.count_nonzero(fg != fo)
    assert badg == bado
    if bado == 0:
        assert_close(Wg, Wo, 1e-10, f"teno5 {shape} ct={ct} q={q}")


@pytest.mark.parametrize("ns", [False, True])
@pytest.mark.parametrize("shape", [(32, 32, 32), (29, 35, 22), (7, 17, 9), (18, 4, 24), (3, 3, 3), (5, 33, 40)])
def test_tile_shapes_3d(orc, torch_dev, shape, ns):
    """3-D grids whose directions take either tile shape (planes that fill
    2 x 16 or 4 x 8 faces, remainders of both): one step with flags against the
    oracle, and two steps of tgks_run equal to stepping without flags."""
    rng = np.random.default_rng(sum(shape))
    field = lambda: 1.0 + 0.1 * rng.uniform(-1, 1, size=shape[::-1])
    W = I.conservative(field(), [0.2 * field() for _ in range(3)], field())
    kw = dict(tau="viscous", mu=1e-3, prandtl=0.72) if ns else {}
    pr = problem(list(shape), [1.0 / n for n in shape],
                 bc=[("periodic", "periodic"), ("reflective", "transmissive"), ("noslip", "reflective")], **kw)
    P = orc_params(orc, pr)
    dt = orc.cfl_dt(P, W, 0.3)
    Wo, fo, Wso, bado = orc.step(P, W, dt, want_flags=True, want_wstar=True)
    print(f"[paths] 3-D tiles {shape} ns={ns}", flush=True)
    gp = GpuProblem(pr)
    try:
        Wg, Wsg, fg, badg = gp.step(W, dt)
        Wr, _, badr = gp.run(W, 2, fixed_dt=dt)
        W1 = gp.step(W, dt, flags=False)[0]
        W2 = gp.step(W1, dt, flags=False)[0]
    finally:
        gp.close()
    assert badg == bado == 0 and badr == 0
    assert np.array_equal(fg, fo)
    assert_close(Wsg, Wso, 1e-10, f"W* {shape}")
    assert_close(Wg, Wo, 1e-10, f"{shape}")
    assert np.array_equal(W1, Wg) and np.array_equal(Wr, W2)
