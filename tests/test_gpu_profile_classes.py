"""Spans per kernel class in the reverse sweep."""
import numpy as np
import pytest

from paper_2507_04192_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,scans", [(2, 4), (3, 6)])
def test_recomputed_segments_count_in_their_classes(dim, scans):
    """Six steps in segments of two, the last on the tape: the sweep recomputes
    two segments.  Each begins with a key pass (SCAN) and scans in its first step,
    in 3-D in every step."""
    from paper_2507_04192_amd.native import Solver
    cells = (20, 16, 1) if dim == 2 else (20, 16, 12)
    cfg = W.SimConfig(dim=dim, n=cells, dx=0.01, dt=1e-4, material=W.FLUID, ppc=4, gravity=(0.0,) * 3, bulk=1e4, gamma=1.0)
    rng = np.random.default_rng(1)
    x = rng.uniform(0.02, 0.1, size=(dim, 500))
    s = Solver(cfg, "f64", capacity=500, tape_steps=6, ckpt_every=2)
    s.mpm_init_particles(x, np.zeros_like(x))
    s.mpm_set_observations([6], tracer_pid=np.arange(9), lag_field="x", lag_target=np.zeros((1, dim, 9)))
    s.mpm_forward_loss(6)
    s.mpm_profile_enable(True)
    s.mpm_profile_read()
    s.mpm_backward()
    n = {k: c for k, (_, c) in s.mpm_profile_read().items()}
    s.close()
    assert n["scan"] == scans and n["p2g"] == 4 and n["g2p_adj"] == 6 and n["p2g_adj"] == 6
