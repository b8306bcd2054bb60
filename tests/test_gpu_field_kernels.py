"""The tabulated field's gradient and the network's backward pass at the sizes
where their kernels change their split: against plain binary64 sums."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# (components, nx, ny, points): one workgroup and the first size past it, tables
# that are repeated in LDS, that just fit (8192 entries), that fit one component
# at a time, and one too large for LDS
@pytest.mark.parametrize("nc,nx,ny,n", [(1, 1, 1, 1), (2, 16, 8, 2048), (2, 16, 8, 2049), (1, 4, 1, 100003),
                                        (2, 64, 64, 5000), (3, 64, 64, 5001), (2, 128, 65, 6000), (2, 16, 8, 600000)])
def test_cell_scatter(nc, nx, ny, n):
    import torch
    from paper_2507_04192_amd.native import CellField
    print(f"[case] cell scatter {nc} x {nx} x {ny}, {n} points", flush=True)
    rng = np.random.default_rng(n)
    x = rng.uniform(-0.05, 1.05, size=(2, n)).astype(np.float32)
    d = rng.normal(size=(nc, n)).astype(np.float32)
    f = CellField(nc, nx, ny, (0.0, 0.0), (1.0, 1.0))
    got = f.scatter(torch.tensor(x, device="cuda"), torch.tensor(d, device="cuda")).cpu().numpy().reshape(nc, nx * ny)
    c = [np.clip(np.floor(x[a] * np.float32(m)).astype(np.int64), 0, m - 1) for a, m in ((0, nx), (1, ny))]
    cell = c[1] * nx + c[0]
    for k in range(nc):
        ref = np.bincount(cell, weights=d[k].astype(np.float64), minlength=nx * ny)
        mag = np.bincount(cell, weights=np.abs(d[k]).astype(np.float64), minlength=nx * ny)
        hits = np.bincount(cell, minlength=nx * ny)
        # binary32 additions into an entry: one per workgroup (at most 256), or
        # one per point where the table does not fit LDS; each rounds a partial
        # sum of at most mag
        adds = hits if nx * ny > 8192 else np.minimum(hits, 256)
        assert np.all(np.abs(got[k] - ref) <= (adds + 2) * 2.0 ** -24 * mag)
