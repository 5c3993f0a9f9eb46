"""The time step and the clock of tgks_run and of batches where their routes
change: 2-D grids at 256 and 257 partial minima (256 x 256 and 257 x 256 cells:
up to there a step takes its clock from the step before, beyond a kernel of its
own does), the one-block reduction at 4,096 and 4,097 cells in 2-D and 3-D, steps
after the end time, and the step counts of batch instances that stop."""
import numpy as np
import pytest

from gpu_common import GpuProblem, gpu_params, problem
from paper_2309_10534_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def field(shape, hot):
    """A smooth flow with a few cells of jumps; the cell `hot` (flat index) has
    the smallest time step by far."""
    D = len(shape)
    rng = np.random.default_rng(sum(shape))
    x = np.meshgrid(*[(np.arange(n) + 0.5) / n for n in shape[::-1]], indexing="ij")
    s = sum(np.sin(2 * np.pi * (c + 0.1 * k)) for k, c in enumerate(x)) / D
    p = 1.0 + 0.2 * s + 0.05 * rng.random(s.shape)
    p.reshape(-1)[hot] *= 4.0
    return I.conservative(1.0 + 0.2 * s, [0.1 + 0.2 * s for _ in range(D)], p)


def stepped(gp, W, steps, cfl, t_end):
    """cfl_dt + step, one at a time: states, clock, steps taken."""
    t, dt, taken = 0.0, gp.cfl_dt(W, cfl, 0.0, t_end), 0
    for _ in range(steps):
        if not dt > 0.0:
            break
        W = gp.step(W, dt, flags=False)[0]
        t += dt
        taken += 1
        dt = gp.cfl_dt(W, cfl, t, t_end)
    return W, np.array([t, dt]), taken


@pytest.mark.parametrize("clip", [False, True])
@pytest.mark.parametrize("shape", [(256, 256), (257, 256), (64, 64), (241, 17), (16, 16, 16), (17, 241, 3), (41, 41, 41)])
def test_run_equals_steps(torch_dev, shape, clip):
    """Seven CFL steps of tgks_run, eager and captured (replayed), with the
    limiting cell in the first and in the last partial minimum, with and
    without an end time that clips the fourth step: the bits of separate
    cfl_dt and step calls, and their clock."""
    D, n = len(shape), int(np.prod(shape))
    pr = problem(list(shape), [1.0 / max(shape)] * D, bc="periodic")
    for hot in (0, n - 1):
        W0 = field(shape, hot)
        gp = GpuProblem(pr)
        try:
            print(f"[clock] {shape} hot={hot} clip={clip}", flush=True)
            t_end = 3.4 * gp.cfl_dt(W0, 0.4) if clip else 0.0
            Ws, clock, taken = stepped(gp, W0, 7, 0.4, t_end)
            assert taken < 7 if clip else taken == 7
            for graph in (False, True, True):
                Wr, td, bad = gp.run(W0, 7, cfl=0.4, t_end=t_end, use_graph=graph)
                assert bad == 0
                assert np.array_equal(Wr, Ws), (hot, graph)
                assert np.array_equal(td, clock), (hot, graph, td, clock)
        finally:
            gp.close()


@pytest.mark.parametrize("sizes", [[(57,), (231,), (232,), (465,)], [(40,), (59393,)], [(19, 23), (40, 31), (64, 9)]])
def test_batch_steps_at_the_end_time(torch_dev, sizes):
    """Instances that reach t_end after different numbers of steps: states,
    clocks and step counts of separate cfl_dt and step calls, eager and
    captured."""
    from paper_2309_10534_amd import tgks
    torch, steps, t_end = torch_dev, 9, 0.01
    ref, probs = [], []
    for k, shape in enumerate(sizes):
        D = len(shape)
        W = field(shape, int(np.prod(shape)) // 2)
        pr = problem(list(shape), [1.0 / (30 * (k + 2) if D == 1 else 20 * (k + 2))] * D, bc="transmissive")
        probs.append((W, pr))
        gp = GpuProblem(pr)
        try:
            ref.append(stepped(gp, W, steps, 0.5, t_end))
        finally:
            gp.close()
    assert min(r[2] for r in ref) < steps and len({r[2] for r in ref}) > 1, [r[2] for r in ref]
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
            assert list(tgks.tgks_batch_steps(b)) == [r[2] for r in ref], graph
            for k, (Ws, ck, _) in enumerate(ref):
                assert np.array_equal(out[k], Ws) and np.array_equal(clock[k], ck), (sizes[k], graph)
    finally:
        tgks.tgks_batch_destroy(b)
