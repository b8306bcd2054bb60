"""Captured steps and what the host keeps between calls: a step may use what the
step before it left on the device only where that step has run, in the same
order, whenever it runs itself.  Every run is compared bit for bit with the same
steps launched eagerly."""
import numpy as np
import pytest

from paper_2507_04192_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("x", "v", "C", "stress")
DIMS = pytest.mark.parametrize("dim", [2, 3])


def _problem(dim):
    cells = (59, 44, 1) if dim == 2 else (33, 21, 14)
    g = (0.0, -9.81, 0.0) if dim == 2 else (0.0, 0.0, -9.81)
    cfg = W.SimConfig(dim=dim, n=cells, dx=0.01, dt=2e-4, material=W.FLUID, ppc=4, gravity=g, bulk=1e4, gamma=1.0)
    rng = np.random.default_rng(dim)
    n = 6000
    x = rng.uniform(0.0, 1.0, size=(dim, n)) * np.array([[c * 0.01] for c in cells[:dim]])
    return cfg, x, rng.normal(0.0, 2.0, size=(dim, n))   # 4 per cent of a cell per step


def _pair(cfg, n, stream, **kw):
    from paper_2507_04192_amd.native import Solver
    return [Solver(cfg, "f32", capacity=n, stream=stream, **kw) for _ in range(2)]


def _capture(s, stream, steps=2):
    import torch
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        s.mpm_step(steps)
    return g


def _same(a, b, stream, what):
    import torch
    stream.synchronize()
    read = [[s.mpm_read_state(f) for f in FIELDS + ("pid",)] + [s.read_keys()] for s in (a, b)]
    for p, q in zip(*read):
        assert torch.equal(p, q), what


@DIMS
def test_steps_after_a_capture_that_has_not_run(dim):
    """Steps that are only captured leave nothing for the eager ones after them."""
    import torch
    cfg, x, v = _problem(dim)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        a, b = _pair(cfg, x.shape[1], st)
        for s in (a, b):
            s.mpm_init_particles(x, v)
    g = _capture(a, st)
    with torch.cuda.stream(st):
        for s in (a, b):
            s.mpm_step(2)
        _same(a, b, st, "eager after the capture")
        g.replay()
        b.mpm_step(2)
        _same(a, b, st, "replay")
        for s in (a, b):
            s.mpm_step(4)
        _same(a, b, st, "eager after the replay")
        g2 = _capture(a, st, 4)      # captured, dropped
        del g2
        for s in (a, b):
            s.mpm_step(1)
        _same(a, b, st, "eager after a dropped capture")
    for s in (a, b):
        assert s.mpm_sync_status()[0] == 0
        s.close()


@DIMS
def test_replay_after_new_particles(dim):
    """New particles start in the buffers of the first ones, after any number of
    eager steps."""
    import torch
    cfg, x, v = _problem(dim)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        a, b = _pair(cfg, x.shape[1], st)
        a.mpm_init_particles(x, v)
        a.mpm_step(2)
    g = _capture(a, st)
    with torch.cuda.stream(st):
        for k, steps in enumerate((1, 2, 3)):
            a.mpm_step(steps)
            y = np.ascontiguousarray(x[:, ::-1])
            for s in (a, b):
                s.mpm_init_particles(y, v)
            g.replay()
            g.replay()
            b.mpm_step(4)
            _same(a, b, st, steps)
            for s in (a, b):        # and the eager steps go on from the replays
                s.mpm_step(2)
            _same(a, b, st, steps)
    for s in (a, b):
        assert s.mpm_sync_status()[0] == 0
        s.close()


# rollouts whose steps off the tape, and whose segments before the taped ones,
# are even and odd in number; with and without the reverse sweep after them
@DIMS
@pytest.mark.parametrize("steps,every,reverse", [(4, 2, False), (5, 2, False), (5, 2, True), (6, 3, False), (8, 4, False)])
def test_replay_after_a_rollout(dim, steps, every, reverse):
    import torch
    cfg, x, v = _problem(dim)
    n = x.shape[1]
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        a, b = _pair(cfg, n, st, tape_steps=steps, ckpt_every=every)
        for s in (a, b):
            s.mpm_init_particles(x, v)
            s.mpm_step(2)
    g = _capture(a, st)
    with torch.cuda.stream(st):
        a.mpm_set_observations([steps], tracer_pid=np.arange(8), lag_field="x", lag_target=np.zeros((1, dim, 8)))
        off_tape = (steps - 1) // every * every
        a.mpm_forward_loss(steps)
        b.mpm_step(steps)
        if reverse:
            a.mpm_backward()
        if off_tape % 2:            # the state is in the other buffer, as after as many steps
            for s in (a, b):
                s.mpm_step(1)
        g.replay()
        b.mpm_step(2)
        _same(a, b, st, "replay")
        for s in (a, b):
            s.mpm_step(3)
        _same(a, b, st, "eager")
    for s in (a, b):
        assert s.mpm_sync_status()[0] == 0
        s.close()
