"""The two ways in which a 3-D step finds a tile's particles: from the previous
step's layout and the marks of the particles that changed their tile, or (keys
written anew) by the scatter.  Both give the same order, so a run and a run
whose positions are written back before every step agree bit for bit."""
import numpy as np
import pytest

from paper_2507_04192_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("x", "v", "C", "stress")


def _config(cells, material=W.FLUID, transfer=W.APIC):
    return W.SimConfig(dim=3, n=cells, dx=0.01, dt=2e-4, material=material, ppc=8, gravity=(0.0, 0.0, -9.81),
                       bulk=1e4, gamma=1.0, youngs=1e4, transfer=transfer, flip_alpha=0.9)


def _state(s):
    out = [s.mpm_read_state(f) for f in FIELDS] + [s.mpm_read_state("pid")]
    return out + list(s.mpm_read_sort())


def _alike(a, b, k):
    import torch
    for p, q in zip(_state(a), _state(b)):
        # a body thrown at a wall may end in NaN, alike on both sides
        assert torch.equal(p.isnan(), q.isnan()) and torch.equal(p.nan_to_num(), q.nan_to_num()), k


def _particles(cells, n, spot, speed, seed):
    rng = np.random.default_rng(seed)
    ext = np.array([[c * 0.01] for c in cells])
    x = rng.uniform(0.0, 1.0, size=(3, n)) * ext
    if spot:
        x[:, : n // 2] = 0.5 * ext + rng.uniform(-spot, spot, size=(3, n // 2))
    return x, rng.normal(0.0, speed, size=(3, n))


# one tile; ragged grids; several scan chunks; tiles whose own range is past the
# 512 particles held in registers, and crowded ones past 1024
@pytest.mark.parametrize("cells,n,spot,material,transfer,precision", [
    ((1, 1, 1), 20, None, W.FLUID, W.APIC, "f32"), ((9, 3, 6), 700, None, W.SAND, W.APIC, "f64"),
    ((33, 21, 14), 40000, None, W.FLUID, W.FLIP, "f32"), ((70, 66, 60), 60000, None, W.DP_JAUMANN, W.TPIC, "f64"),
    ((12, 12, 12), 9000, 0.02, W.FLUID, W.APIC, "f64"), ((12, 12, 12), 14000, 0.02, W.SAND, W.FLIP, "f32")])
def test_layout_and_keys_find_the_same(cells, n, spot, material, transfer, precision):
    from paper_2507_04192_amd.native import Solver
    print(f"[case] 3-D step {cells} {n} {material} {transfer} {precision}", flush=True)
    cfg = _config(cells, material, transfer)
    x, v = _particles(cells, n, spot, 2.0, n)   # 4 per cent of a cell per step
    a, b = (Solver(cfg, precision, capacity=n) for _ in range(2))
    for s in (a, b):
        s.mpm_init_particles(x, v)
    for k in range(6):
        a.mpm_step(1)
        b.mpm_write_state("x", b.mpm_read_state("x"))
        b.mpm_step(1)
        _alike(a, b, k)
    assert a.mpm_sync_status() == b.mpm_sync_status()
    a.close()
    b.close()


def test_particles_past_the_neighbouring_tiles_are_found():
    """Steps beyond the CFL limit are reported, and lose no particle."""
    from paper_2507_04192_amd.native import Solver
    cfg = _config((64, 20, 20))
    n = 5000
    x, v = _particles((20, 20, 20), n, None, 0.5, 5)
    v[0] += 700.0       # 14 cells per step
    a, b = (Solver(cfg, "f64", capacity=n) for _ in range(2))
    for s in (a, b):
        s.mpm_init_particles(x, v)
    for k in range(4):
        a.mpm_step(1)
        b.mpm_write_state("x", b.mpm_read_state("x"))
        b.mpm_step(1)
        _alike(a, b, k)
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
    cfg = _config((33, 21, 14))
    n = 20000
    x, v = _particles((33, 21, 14), n, None, 2.0, 9)
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
            _alike(a, b, k)
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


def test_scan_in_one_and_two_launches():
    """The same body in grids that grow only away from it: one chunk of tiles,
    many, and more than the one-launch scan takes.  The tiles' order is the
    same, so sort and state are, bit for bit."""
    from paper_2507_04192_amd.native import Solver
    n = 4000
    rng = np.random.default_rng(3)
    x = rng.uniform(0.01, 0.15, size=(3, n))
    v = rng.normal(0.0, 0.5, size=(3, n))
    ref = None
    for cells in ((32, 24, 16), (500, 400, 16), (1000, 800, 16)):
        print(f"[case] scan {cells}", flush=True)
        s = Solver(_config(cells), "f32", capacity=n)
        s.mpm_init_particles(x, v)
        s.mpm_step(3)
        assert s.mpm_sync_status()[0] == 0
        out = [t.cpu().numpy() for t in _state(s)[:-1]]
        s.close()
        for a, b in zip(ref or out, out):
            assert np.array_equal(a, b)
        ref = ref or out
