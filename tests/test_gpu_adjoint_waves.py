"""The reverse G2P in 3-D binary64 is built for one wave per SIMD and for two,
taken by the number of particles and tiles: the same body, small and in a grid
past the line, gives the same gradient."""
import numpy as np
import pytest

from paper_2507_04192_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("material,transfer,viscosity", [
    (W.FLUID, W.APIC, 0.0), (W.FLUID, W.FLIP, 0.0), (W.FLUID, W.FLIP, 2.0), (W.DP_JAUMANN, W.FLIP, 0.0),
    (W.DP_JAUMANN, W.TPIC, 0.0)])
def test_gradient_on_both_sides_of_the_line(material, transfer, viscosity):
    from paper_2507_04192_amd.native import Solver
    from tests.helpers import rel_l2
    print(f"[case] reverse G2P {material} {transfer} {viscosity}", flush=True)
    n, steps = 132000, 3        # past 131,072: the grid of 8^3 tiles decides
    rng = np.random.default_rng(7)
    x = rng.uniform(0.03, 0.2, size=(3, n))
    v = rng.normal(0.0, 0.5, size=(3, n))
    tr = np.arange(0, n, 997)
    tgt = x[:, tr][None] + 1e-3
    out = []
    for cells in ((24, 24, 24), (28, 28, 28)):      # 8^3 and 9^3 tiles
        cfg = W.SimConfig(dim=3, n=cells, dx=0.01, dt=1e-4, material=material, ppc=27, gravity=(0.0, 0.0, -9.81), bulk=1e4,
                          gamma=1.0, youngs=1e5, transfer=transfer, flip_alpha=0.9, viscosity=viscosity)
        s = Solver(cfg, "f64", capacity=n, tape_steps=steps, ckpt_every=steps)
        s.mpm_init_particles(x, v)
        s.mpm_set_observations([steps], tracer_pid=tr, lag_field="x", lag_target=tgt)
        loss = s.mpm_forward_loss(steps)
        out.append((loss, s.mpm_backward(want_mu=False)[0].cpu().numpy()))
        s.close()
    (la, ga), (lb, gb) = out
    # binary64; the node adjoints' atomics add in any order
    assert abs(la - lb) <= 1e-12 * abs(la)
    assert np.isfinite(ga).all() and np.linalg.norm(ga) > 0.0 and rel_l2(gb, ga) <= 1e-10
