"""Vectors of 3-D particles read in particle order, below, at and past the sizes
(40 MB, in binary32 100, and 200 MB) between which the read gathers."""
import numpy as np
import pytest

from paper_2507_04192_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,n", [("f64", 1666666), ("f64", 1666667), ("f32", 8333335), ("f64", 8333334)])
def test_vectors_by_pid(precision, n):
    import torch
    from paper_2507_04192_amd.native import Solver
    print(f"[case] read vectors {precision} {n}", flush=True)
    cfg = W.SimConfig(dim=3, n=(128, 96, 96), dx=0.01, dt=1e-5, material=W.FLUID, ppc=8, gravity=(0.0, 0.0, -9.81), bulk=1e4, gamma=1.0)
    g = torch.Generator(device="cuda").manual_seed(n)
    dt = torch.float32 if precision == "f32" else torch.float64
    x = torch.rand((3, n), generator=g, device="cuda", dtype=dt) * 0.95
    v = torch.randn((3, n), generator=g, device="cuda", dtype=dt)
    s = Solver(cfg, precision, capacity=n + 3)
    s.mpm_init_particles(x, v)
    s.mpm_step(2)
    pid = s.mpm_read_state("pid")[0].long()
    for f in ("x", "v"):
        mem, by = s.mpm_read_state(f), s.mpm_read_state(f, "pid")
        assert bool((by[:, pid] == mem).all()), f
    s.close()
    assert bool((torch.sort(pid)[0] == torch.arange(n, device="cuda")).all())
