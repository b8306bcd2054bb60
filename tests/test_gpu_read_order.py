"""Fields read in particle order against the same fields in memory order,
below and above the size from which the read gathers."""
import numpy as np
import pytest

from paper_2507_04192_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,material,precision,n", [(3, W.SAND, "f32", 277777), (3, W.SAND, "f64", 277778),
                                                      (2, W.FLUID, "f32", 625001), (2, W.DP_JAUMANN, "f64", 630016)])
def test_particle_order_is_memory_order_by_pid(dim, material, precision, n):
    from paper_2507_04192_amd.native import Solver
    print(f"[case] read order {dim}-D {material} {precision} {n}", flush=True)
    cells = (64, 48, 32) if dim == 3 else (512, 384)
    cfg = W.SimConfig(dim=dim, n=cells, dx=0.01, dt=1e-5, material=material, ppc=4, gravity=(0.0, -9.81, 0.0),
                      phi_deg=30.0)
    x, v, _, _ = W.random_state(cfg, n, seed=n)
    s = Solver(cfg, precision, capacity=n + 5)
    s.mpm_init_particles(x, v)
    s.mpm_step(3)
    pid = s.mpm_read_state("pid")[0].long()
    for f in ("x", "v", "C", "stress", "F", "FmI") if material == W.SAND else ("x", "v", "C", "stress", "J", "Jm1"):
        mem, by = s.mpm_read_state(f), s.mpm_read_state(f, "pid")
        assert bool((by[:, pid] == mem).all()), f
    s.close()
    assert np.array_equal(np.sort(pid.cpu().numpy()), np.arange(n))
