"""The two ways in which a 2-D step finds a tile's particles: from the previous
step's layout, or (keys written anew) by the scan and the scatter.  Both give
the same order, so a run and a run whose positions are written back before
every step agree bit for bit."""
import numpy as np
import pytest

from paper_2507_04192_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("x", "v", "C", "stress")


def _config(cells, material=W.FLUID, transfer=W.APIC, dt=2e-4):
    return W.SimConfig(dim=2, n=cells, dx=0.01, dt=dt, material=material, ppc=4, gravity=(0.0, -9.81, 0.0),
                       bulk=1e4, gamma=1.0, youngs=1e4, transfer=transfer, flip_alpha=0.9)


def _state(s):
    out = [s.mpm_read_state(f) for f in FIELDS] + [s.mpm_read_state("pid")]
    return out + list(s.mpm_read_sort())


# one tile; ragged grids about a tile's edge; the last grid whose tiles a
# workgroup counts itself (45 x 45 = 2025 of 2048) and the first past it
# (46 x 45); rows of more than 256 and tiles of more than 1024 particles
@pytest.mark.parametrize("cells,n,spot,material,transfer,precision", [
    ((3, 3, 1), 40, None, W.FLUID, W.APIC, "f32"), ((13, 3, 1), 300, None, W.SAND, W.APIC, "f64"),
    ((59, 44, 1), 9000, None, W.FLUID, W.FLIP, "f32"), ((60, 45, 1), 9001, None, W.DP_JAUMANN, W.TPIC, "f64"),
    ((355, 355, 1), 20000, None, W.FLUID, W.APIC, "f64"), ((363, 355, 1), 20000, None, W.FLUID, W.APIC, "f32"),
    ((40, 30, 1), 3000, 0.03, W.FLUID, W.APIC, "f32"), ((40, 30, 1), 9000, 0.03, W.FLUID, W.FLIP, "f64")])
def test_layout_and_keys_find_the_same(cells, n, spot, material, transfer, precision):
    import torch
    from paper_2507_04192_amd.native import Solver
    print(f"[case] 2-D step {cells} {n} {material} {transfer} {precision}", flush=True)
    cfg = _config(cells, material, transfer)
    rng = np.random.default_rng(n)
    ext = np.array([[cells[0] * 0.01], [cells[1] * 0.01]])
    x = rng.uniform(0.0, 1.0, size=(2, n)) * ext
    if spot:
        # half of them within a few cells: a crowded tile, and a crowded neighbour
        x[:, : n // 2] = 0.5 * ext + rng.uniform(-spot, spot, size=(2, n // 2))
    v = rng.normal(0.0, 2.0, size=(2, n))    # 4 per cent of a cell per step: hundreds change their tile
    a, b = (Solver(cfg, precision, capacity=n) for _ in range(2))
    for s in (a, b):
        s.mpm_init_particles(x, v)
    for k in range(6):
        a.mpm_step(1)
        b.mpm_write_state("x", b.mpm_read_state("x"))
        b.mpm_step(1)
        for p, q in zip(_state(a), _state(b)):
            assert torch.equal(p, q), k
    assert a.mpm_sync_status()[0] == b.mpm_sync_status()[0] == 0
    a.close()
    b.close()


def test_particles_past_the_neighbouring_tiles_are_found():
    """Steps beyond the CFL limit are reported, and lose no particle."""
    import torch
    from paper_2507_04192_amd.native import Solver
    cfg = _config((96, 64, 1))
    rng = np.random.default_rng(5)
    n = 3000
    x = rng.uniform(0.05, 0.6, size=(2, n))
    v = rng.normal(0.0, 0.5, size=(2, n))
    v[0] += 1500.0       # 30 cells per step
    a, b = (Solver(cfg, "f64", capacity=n) for _ in range(2))
    for s in (a, b):
        s.mpm_init_particles(x, v)
    for k in range(4):
        a.mpm_step(1)
        b.mpm_write_state("x", b.mpm_read_state("x"))
        b.mpm_step(1)
        for p, q in zip(_state(a), _state(b)):
            # a body thrown at the wall ends in NaN, alike on both sides
            assert torch.equal(p.isnan(), q.isnan()) and torch.equal(p.nan_to_num(), q.nan_to_num()), k
        assert np.array_equal(np.sort(a.mpm_read_state("pid")[0].cpu().numpy()), np.arange(n))
    sa, sb = a.mpm_sync_status(), b.mpm_sync_status()
    assert sa == sb and sa[0] in (-4, -5)
    a.close()
    b.close()


def test_captured_steps_replay():
    """Two captured steps replayed, with eager steps and new positions between
    the replays, against the same steps taken eagerly."""
    import torch
    from paper_2507_04192_amd.native import Solver
    cfg = _config((59, 44, 1))
    rng = np.random.default_rng(9)
    n = 5000
    x = rng.uniform(0.0, 0.44, size=(2, n))
    v = rng.normal(0.0, 2.0, size=(2, n))
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        a, b = (Solver(cfg, "f32", capacity=n, stream=st) for _ in range(2))
        for s in (a, b):
            s.mpm_init_particles(x, v)
            s.mpm_step(2)
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        a.mpm_step(2)
    with torch.cuda.stream(st):
        for k in range(5):
            g.replay()
            b.mpm_step(2)
            st.synchronize()
            for p, q in zip(_state(a), _state(b)):
                assert torch.equal(p, q), k
            if k == 1:      # an even number of eager steps
                a.mpm_step(2)
                b.mpm_step(2)
            if k == 2:      # positions that owe nothing to the last sort
                y = torch.flip(a.mpm_read_state("x"), dims=(1,)).contiguous()
                a.mpm_write_state("x", y)
                b.mpm_write_state("x", y)
    st.synchronize()
    a.close()
    b.close()


# one tile, ragged tiles, particles of many tiles in the corner nodes, and a grid
# past the tiles that a workgroup counts itself; with floor friction
@pytest.mark.parametrize("cells,n,transfer", [((3, 3, 1), 30, W.APIC), ((13, 9, 1), 400, W.FLIP), ((59, 44, 1), 4000, W.APIC),
                                              ((363, 355, 1), 3000, W.APIC)])
def test_gradient_over_tiles_matches_oracle(orc, cells, n, transfer):
    from paper_2507_04192_amd.native import Solver
    from tests.helpers import rel_l2
    cfg = _config(cells, W.FLUID, transfer, dt=5e-5).replace(wall_mode=(W.SLIP, W.SLIP, W.COULOMB, W.SLIP, W.SLIP, W.SLIP))
    print(f"[case] 2-D gradient {cells} {n} {transfer}", flush=True)
    rng = np.random.default_rng(n)
    x = rng.uniform(0.0, 1.0, size=(2, n)) * np.array([[cells[0] * 0.01], [min(cells[1], 20) * 0.01]])
    v = rng.normal(0.0, 1.0, size=(2, n)) - np.array([[0.0], [0.5]])
    mu = rng.uniform(0.1, 0.5, size=cfg.floor_nodes())
    frames, tr = [3, 6, 8], W.pick_tracers(n, 20, 3)
    tgt = x[:, tr][None] + rng.normal(0.0, 1e-3, size=(3, 2, 20))
    loss_o, gv_o, gmu_o = orc.rollout_grad(cfg, x, v, 8, cfg.dt, mu, orc.Observations(frames, tr, "x", tgt))
    s = Solver(cfg, "f64", capacity=n, tape_steps=8, ckpt_every=3)
    s.mpm_init_particles(x, v)
    s.mpm_set_floor_mu(mu)
    s.mpm_set_observations(frames, tracer_pid=tr, lag_field="x", lag_target=tgt)
    loss = s.mpm_forward_loss(8)
    gv, gmu = (t.cpu().numpy() for t in s.mpm_backward())
    s.close()
    # binary64 to the bounds of the other gradient tests
    assert abs(loss - loss_o) <= 1e-10 * loss_o
    assert rel_l2(gv, gv_o) <= 1e-8 and rel_l2(gmu, gmu_o) <= 1e-8
