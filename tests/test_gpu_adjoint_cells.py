"""The D3Q19 FP64 adjoint in three launches over the cells against the general
reverse pass: row ends inside and at the ends of waves (64 cells) and
workgroups, every wall rule on every axis, axes of the fewest cells it takes
(four between walls, one periodic) and of fewer, which stay on the general pass.

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

SIDES = {"box": (0,) * 6, "lid": (1,) * 6, "noslip": (3,) * 6, "mixed": (2, 3, 1, 2, 3, 1), "channel_x": (0, 0, 3, 1, 0, 0),
         "channel_z": (2, 1, 0, 0, 0, 0), "duct": (0, 0, 2, 1, 1, 3)}
UW = [[0, 0.02, 0], [0, -0.01, 0], [0.03, 0, 0], [0.05, 0, 0.01], [0, 0, 0.01], [0.02, 0, 0]]
SIZES = [(64, 4, 4), (16, 4, 4), (63, 5, 4), (65, 4, 5), (4, 4, 4), (7, 9, 5), (33, 8, 4), (1, 5, 6), (5, 1, 4), (4, 6, 1),
         (1, 1, 1), (3, 4, 5), (4, 2, 6)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("sides", SIDES)
@pytest.mark.parametrize("n", SIZES, ids=lambda n: "x".join(map(str, n)))
def test_cells_adjoint_matches_general(sides, n, monkeypatch):
    bc = SIDES[sides]
    if any(bc[2 * a] != 0 and n[a] < 2 for a in range(3)):
        pytest.skip("wall-bounded axes have at least two cells")
    print(f"[adjoint cells] {sides} n={n}", flush=True)
    for mesh, force in ((0, False), (1, True)):
        cfg = dict(lattice=19, dtype="f64", n=n, L=tuple(float(v) for v in n), mesh=(mesh,) * 3, k_stretch=1.5, rho0=1.0,
                   RT=1 / 3, tau=0.45, dt=0.25, bc=bc, G=(1e-3, -5e-4, 2e-4), omega=0.7, phase=0.3, uw=UW,
                   pw=[3e-3, -2e-3, 0, 1e-3, 0, 0], pw_osc=[1e-3, 0, 0, 0, 0, 0])
        Q, D, shp = M.shape_of(cfg)
        f = torch.empty((Q,) + shp, dtype=torch.float64, device="cuda")
        G = dev(field(61, (D,) + shp, 2e-3)) if force else None
        ctx = M.dugks_init(cfg, f, dev(1 + field(62, shp, 0.02)), dev(field(63, (D,) + shp, 0.05)), G)
        try:
            f += dev(field(64, f.shape, 1e-3))
            lam = dev(field(65, f.shape, 1.0))
            out, grad = [], []
            for general in ("1", "0"):
                monkeypatch.setenv("DUGKS_ADJOINT_GENERAL", general)
                o = torch.full_like(f, float("nan"))
                g = dev(field(66, (D,) + shp, 1e-3))  # the gradient is added to what is there
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
