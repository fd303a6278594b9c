"""Totals and velocity change over cell counts around the edges of their
reduction (256 cells a workgroup; the last stage takes 160 workgroups a
round and 32 rounds at a time) against sums in torch.

Tolerance: sums of n terms of one sign in trees and chains of at most about
200 adds, each with a relative error of 1.1e-16: 1e-13 with a factor of four
to spare; the momentum is compared to the sum of magnitudes."""
import pytest

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu

BLOCKS = [1, 2, 159, 160, 161, 320, 5119, 5120, 5121, 5280]


@pytest.mark.parametrize("short", [0, 1, 255])
@pytest.mark.parametrize("blocks", BLOCKS)
def test_totals_of_ragged_cell_counts(blocks, short):
    n = blocks * 256 - short
    print(f"[totals] {n} cells", flush=True)
    cfg = dict(lattice=9, dtype="f64", n=(n, 1, 1), L=(float(n), 1.0, 1.0), mesh=(0, 0, 0), k_stretch=1.0, rho0=1.0,
               RT=1 / 3, tau=0.45, dt=0.25, bc=(0,) * 6, G=(0, 0, 0))
    x = torch.arange(n, dtype=torch.float64, device="cuda").reshape(1, 1, n)
    rho = 1 + 0.1 * torch.sin(0.37 * x)
    u = torch.stack((0.05 * torch.cos(0.11 * x), 0.03 * torch.sin(0.23 * x)))
    f = torch.empty((9, 1, 1, n), dtype=torch.float64, device="cuda")
    ctx = M.dugks_init(cfg, f, rho, u)
    try:
        g = f * (1 + 1e-3 * torch.cos(0.05 * x))
        r, v = torch.empty_like(rho), torch.empty_like(u)
        t = M.dugks_moments(ctx, g, None, 0.0, r, v, None, True)
        want = r.sum().item()
        assert abs(t[0] - want) <= 1e-13 * want
        for a in range(2):
            # cell momentum = rho0 u without acceleration
            assert abs(t[1 + a] - v[a].sum().item()) <= 1e-12 * v[a].abs().sum().item()
        want = 0.5 * (v ** 2).sum().item()
        assert abs(t[4] - want) <= 1e-13 * want
        assert t[5] == 0
        ua = torch.empty_like(u)
        M.dugks_moments(ctx, f, None, 0.0, None, ua, None, False)
        d, b = M.dugks_velocity_change(ctx, f, g, None, 0.0, 0.0)
        assert abs(d - ((v - ua) ** 2).sum().sqrt().item()) <= 1e-12 * d
        assert abs(b - (v ** 2).sum().sqrt().item()) <= 1e-13 * b
        # one value that is not finite is found wherever it is
        for c in (0, n // 2, n - 1):
            h = f.clone()
            h[3, 0, 0, c] = float("inf")
            with pytest.raises(M.DugksError) as e:
                M.dugks_moments(ctx, h)
            assert e.value.code == M.ENONFINITE
    finally:
        M.dugks_destroy(ctx)
