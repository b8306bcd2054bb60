"""The order that a step's sort gives, against the keys before it: by tile, then
by the particle's rank among those of its cell (in their slots' order), then by
cell."""
import numpy as np
import pytest

from paper_2507_04192_amd import workloads as W

pytestmark = pytest.mark.gpu


def expected_perm(key):
    """The slots in the sorted order of int32 keys (tile * 64 + cell)."""
    key = np.asarray(key, dtype=np.int64)
    by_key = np.argsort(key, kind="stable")
    k = key[by_key]
    first = np.r_[True, k[1:] != k[:-1]]
    start = np.maximum.accumulate(np.where(first, np.arange(k.size), 0))
    rank = np.empty(k.size, dtype=np.int64)
    rank[by_key] = np.arange(k.size) - start
    return np.lexsort((key & 63, rank, key >> 6))


def _config(dim, cells, dt=2e-4):
    g = (0.0, -9.81, 0.0) if dim == 2 else (0.0, 0.0, -9.81)
    return W.SimConfig(dim=dim, n=cells, dx=0.01, dt=dt, material=W.FLUID, ppc=4, gravity=g, bulk=1e3, gamma=1.0)


# particles of one cell in every lane of a batch, of two and of three cells in
# turn, and of all; tiles past the 512 particles held in registers
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n,width", [(64, 0.005), (500, 0.005), (700, 0.015), (2500, 0.025), (4000, 0.12)])
def test_crowded_cells_keep_their_order(dim, n, width):
    from paper_2507_04192_amd.native import Solver
    rng = np.random.default_rng(n)
    x = 0.056 + rng.uniform(0.0, width, size=(dim, n))
    s = Solver(_config(dim, (20, 20, 20) if dim == 3 else (20, 20, 1)), "f64", capacity=n)
    s.mpm_init_particles(x, rng.normal(0.0, 0.3, size=(dim, n)))
    for k in range(5):
        key = s.read_keys().cpu().numpy()
        s.mpm_step(1)
        perm = s.mpm_read_sort()[0].cpu().numpy()
        assert np.array_equal(perm, expected_perm(key)), k
    s.close()
