"""Nodes in empty tiles beside a body's, and past the last tiles of the grid:
every node that a particle reaches is summed once, whoever its tile is."""
import numpy as np
import pytest

from paper_2507_04192_amd import workloads as W

pytestmark = pytest.mark.gpu


# tiles end at, one, two and three nodes past the grid's last node, alone and mixed
@pytest.mark.parametrize("cells", [(9, 9, 9), (10, 11, 12), (8, 6, 33), (41, 30, 7)])
@pytest.mark.parametrize("precision,transfer", [("f64", W.APIC), ("f64", W.FLIP), ("f32", W.APIC)])
def test_every_node_of_scattered_particles(cells, precision, transfer):
    """Few particles, most tiles empty, some particles past the upper walls:
    nodal masses against a sum over the particles (8 terms and rounding of the
    weights: 64 eps of the largest), and a uniform velocity along x, which slip
    walls leave alone, comes back (27 products of weights that sum to one, two
    steps: 256 eps)."""
    from paper_2507_04192_amd.native import Solver
    print(f"[case] halo {cells} {precision} {transfer}", flush=True)
    cfg = W.SimConfig(dim=3, n=cells, dx=0.5, dt=1e-3, material=W.FLUID, ppc=8, gravity=(0.0, 0.0, 0.0), bulk=1.0,
                      gamma=1.0, transfer=transfer, flip_alpha=0.5, wall_mode=(W.SLIP,) * 6)
    G, nd, n = cfg.ghost, cfg.node_dims(), 24
    rng = np.random.default_rng(sum(cells))
    x = np.empty((3, n))
    x[0] = rng.uniform(3.0, cells[0] - 3.0, n)
    for a in (1, 2):
        x[a] = rng.uniform(0.0, cells[a], n)
        x[a, :6] = cells[a] + rng.uniform(-0.5, G - 0.5, 6)   # in cells; past the wall
    dtype = np.float64 if precision == "f64" else np.float32
    x = (0.5 * x).astype(dtype).astype(np.float64)   # dx is a power of two: cells exactly
    v = np.zeros((3, n))
    v[0] = 1.0
    s = Solver(cfg, precision, capacity=n, keep_grid=True)
    s.mpm_init_particles(x, v)
    s.mpm_step(1)
    got = s.mpm_read_grid("mass").cpu().numpy()[0].astype(np.float64)
    ref = np.zeros((nd[2], nd[1], nd[0]))
    xi = x / 0.5
    base = np.floor(xi - 0.5).astype(int)
    fx = xi - base
    w = np.stack([0.5 * (1.5 - fx) ** 2, 0.75 - (fx - 1.0) ** 2, 0.5 * (fx - 0.5) ** 2])
    for p in range(n):
        for k in range(27):
            i, j, l = k % 3, (k // 3) % 3, k // 9
            I = base[0, p] + i + G, base[1, p] + j + G, base[2, p] + l + G
            if all(0 <= I[a] < nd[a] for a in range(3)):
                ref[I[2], I[1], I[0]] += w[i, 0, p] * w[j, 1, p] * w[l, 2, p]
    mass = got.sum() / ref.sum()
    eps = np.finfo(dtype).eps
    assert mass > 0 and np.array_equal(got != 0, ref.ravel() != 0)
    assert np.abs(got / mass - ref.ravel()).max() <= 64 * eps * ref.max()
    s.mpm_step(1)
    assert np.abs(s.mpm_read_state("v").cpu().numpy()[0] - 1.0).max() <= 256 * eps
    s.close()
