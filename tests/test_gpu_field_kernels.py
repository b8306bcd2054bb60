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


# (widths, output, hidden, samples): each bound of the widths (32, 64, 128) at
# and past its edge, sample counts about the workgroup's 64, the first split
# into several workgroups, and more samples than the workgroups take in one turn
@pytest.mark.parametrize("widths,out,hidden,n", [
    ([1, 30, 30, 30, 1], "none", "relu", 1), ([2, 32, 32, 2], "none", "tanh", 63), ([3, 33, 64, 2], "none", "tanh", 64),
    ([2, 64, 64, 2], "none", "tanh", 65), ([2, 65, 17, 1], "sigmoid", "tanh", 129), ([2, 128, 128, 1], "sigmoid", "tanh", 200),
    ([4, 128, 128, 128, 128], "none", "tanh", 131), ([2, 64, 64, 2], "none", "relu", 33001),
    ([2, 128, 128, 1], "sigmoid", "tanh", 16500), ([2], "none", "tanh", 100)])
def test_mlp_gradient(widths, out, hidden, n):
    import torch
    from paper_2507_04192_amd.native import MLP
    if len(widths) == 1:
        widths = widths + [2]        # a single layer
    print(f"[case] mlp gradient {widths} {hidden}/{out} n={n}", flush=True)
    g = torch.Generator().manual_seed(n)
    net = MLP(widths, out, in_scale=[2.0] * widths[0], in_shift=[-1.0] * widths[0], math="f32", hidden_act=hidden)
    theta = torch.cat([(torch.rand(o * (i + 1), generator=g) * 2 - 1) / i ** 0.5 for i, o in zip(widths[:-1], widths[1:])])
    x = torch.rand((widths[0], n), generator=g)
    dy = torch.randn((widths[-1], n), generator=g)
    y, cache = net.forward(theta.cuda(), x.cuda())
    dp = net.backward(theta.cuda(), x.cuda(), cache, dy.cuda())
    again = net.backward(theta.cuda(), x.cuda(), cache, dy.cuda())
    assert torch.equal(dp, again), "the gradient is summed in a fixed order"
    t = theta.double().requires_grad_(True)
    h, at, mag = x.double() * 2 - 1, 0, []
    for l, (i, o) in enumerate(zip(widths[:-1], widths[1:])):
        h = t[at:at + o * i].reshape(o, i) @ h + t[at + o * i:at + o * (i + 1), None]
        at += o * (i + 1)
        if l < len(widths) - 2:
            h = torch.relu(h) if hidden == "relu" else torch.tanh(h)
    ref = torch.sigmoid(h) if out == "sigmoid" else h
    (ref * dy.double()).sum().backward()
    # binary32 rounding of sums of up to 129 products per layer, four layers, and
    # of n terms of random sign: sqrt-growth, with a factor of ten to spare
    eps = 2.0 ** -24
    assert torch.linalg.norm(y.cpu().double() - ref.detach()) <= 10 * eps * 129 ** 0.5 * len(widths) * torch.linalg.norm(ref.detach())
    tol = 10 * eps * 129 ** 0.5 * len(widths)
    assert torch.linalg.norm(dp.cpu().double() - t.grad) <= tol * torch.linalg.norm(t.grad)
