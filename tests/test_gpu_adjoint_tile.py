"""The one-launch D2Q9 FP64 adjoint (tiles of 28 x 4 cells on small meshes and of
28 x 12 on others, here the last two sizes; wall rules folded into the pairs
of cells next to them) against the general reverse pass, at the
edges of its tiles and of its axes.

Tolerance: both evaluate the same sums of some thousand products in another
order, each with a relative error of 1.1e-16 against the largest term; 1e-12
of the largest result leaves a factor of about ten, as in the oracle's tests,
and 1e-11 for the force gradient, whose terms cancel."""
import numpy as np
import pytest

from synthetic import field

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu

SIDES = {"box": (0,) * 6, "lid": (1, 1, 1, 1, 0, 0), "noslip": (3, 3, 3, 3, 0, 0), "inlet": (2, 2, 3, 1, 0, 0),
         "channel_x": (0, 0, 3, 1, 0, 0), "channel_y": (2, 3, 0, 0, 0, 0)}
UW = [[0, 0.02, 0], [0, -0.01, 0], [0.03, 0, 0], [0.05, 0, 0], [0, 0, 0], [0, 0, 0]]
SIZES = [(28, 12), (29, 13), (27, 11), (30, 14), (56, 25), (57, 24), (26, 10), (1, 1), (1, 30), (33, 1), (2, 2), (2, 40),
         (64, 2), (3, 3), (31, 3), (150, 61), (28, 4), (29, 5), (57, 8), (250, 253), (253, 252)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("sides", SIDES)
@pytest.mark.parametrize("n", SIZES, ids=lambda n: f"{n[0]}x{n[1]}")
def test_tile_adjoint_matches_general(sides, n, monkeypatch):
    bc = SIDES[sides]
    if any(bc[2 * a] != 0 and n[a] < 2 for a in range(2)):
        pytest.skip("wall-bounded axes have at least two cells")
    print(f"[adjoint tile] {sides} n={n}", flush=True)
    for mesh, force in ((0, False), (1, True)):
        cfg = dict(lattice=9, dtype="f64", n=(n[0], n[1], 1), L=(float(n[0]), float(n[1]), 1.0), mesh=(mesh, mesh, 0),
                   k_stretch=1.5, rho0=1.0, RT=1 / 3, tau=0.45, dt=0.25, bc=bc, G=(1e-3, -5e-4, 0.0), omega=0.7,
                   phase=0.3, uw=UW, pw=[3e-3, -2e-3, 0, 0, 0, 0], pw_osc=[1e-3, 0, 0, 0, 0, 0])
        Q, D, shp = M.shape_of(cfg)
        f = torch.empty((Q,) + shp, dtype=torch.float64, device="cuda")
        G = dev(field(51, (D,) + shp, 2e-3)) if force else None
        ctx = M.dugks_init(cfg, f, dev(1 + field(52, shp, 0.02)), dev(field(53, (D,) + shp, 0.05)), G)
        try:
            f += dev(field(54, f.shape, 1e-3))
            lam = dev(field(55, f.shape, 1.0))
            out, grad = [], []
            for general in ("1", "0"):
                monkeypatch.setenv("DUGKS_ADJOINT_GENERAL", general)
                o = torch.full_like(f, float("nan"))
                g = dev(field(56, (D,) + shp, 1e-3))  # the gradient is added to what is there
                M.dugks_step_adjoint(ctx, f, lam, o, G, 0.4, g)
                out.append(o)
                grad.append(g)
            assert (out[0] - out[1]).abs().max() < 1e-12 * out[0].abs().max()
            assert (grad[0] - grad[1]).abs().max() < 1e-11 * grad[0].abs().max()
            # no gradient asked for; the static entry point
            for call in (M.dugks_step_adjoint, M.dugks_step_adjoint_static):
                o = torch.full_like(f, float("nan"))
                call(ctx, f, lam, o, G, 0.4, None)
                assert torch.equal(o, out[1])
        finally:
            M.dugks_destroy(ctx)
