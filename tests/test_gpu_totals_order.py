"""The order of the totals' sums: blocks of 256 cells as a binary tree over the
cells (128 apart, 64, .., 1), then 256 chains over the blocks and a tree over the
chains.  Summed on the host in that order from the density that the read-out
gives, on a mesh of unit cells, the total mass is the same to the bit, in
either precision; a state's totals so stay what they are whatever the kernels."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu


def tree(a):
    """binary tree over the last axis (256 values)"""
    while a.shape[-1] > 1:
        h = a.shape[-1] // 2
        a = a[..., :h] + a[..., h:]
    return a[..., 0]


def total(rho):
    n = rho.size
    blocks = -(-n // 256)
    rounds = -(-blocks // 256)
    a = np.zeros(rounds * 256 * 256)
    a[:n] = rho.ravel()
    part = tree(a.reshape(rounds * 256, 256)).reshape(rounds, 256)
    chains = np.zeros(256)
    for p in part:
        chains = chains + p
    return tree(chains)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [(7, 5), (256, 1), (511, 129), (700, 500), (2048, 1025)])
def test_mass_in_its_order(n, dtype):
    print(f"[totals order] {n} {dtype}", flush=True)
    cfg = dict(lattice=9, dtype=dtype, n=n + (1,), L=(float(n[0]), float(n[1]), 1.0), rho0=1.0, RT=1 / 3, tau=0.4, dt=0.2,
               bc=(0,) * 6)
    T = M.torch_dtype(cfg)
    x = torch.arange(n[0] * n[1], dtype=torch.float64, device="cuda").reshape(1, n[1], n[0])
    f = torch.empty((9, 1, n[1], n[0]), dtype=T, device="cuda")
    ctx = M.dugks_init(cfg, f, (1 + 0.1 * torch.sin(0.37 * x)).to(T))
    try:
        rho = torch.empty((1, n[1], n[0]), dtype=T, device="cuda")
        t = M.dugks_moments(ctx, f, None, 0.0, rho, None, None, True)
        assert t[0] == total(rho.cpu().numpy().astype(np.float64))
        out = torch.empty(6, dtype=torch.float64, device="cuda")
        M.dugks_totals_async(ctx, f, out)
        assert out.tolist() == t
    finally:
        M.dugks_destroy(ctx)
