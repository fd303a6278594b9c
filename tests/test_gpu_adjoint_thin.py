"""The FP64 D2Q9 adjoint on meshes of few columns or rows, some of which take the
passes over the ghost-extended grid (or the periodic ones) and their neighbours
the one launch on tiles: both against the general reverse pass (tolerances as for
the tiles: the same sums of some thousand products in another order), and the
default no slower than the general pass, which thin meshes used to be."""
import pytest

from synthetic import field
from tests.test_gpu_adjoint_tile import SIDES, UW, dev

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu


def cfg_of(n, bc, mesh):
    return dict(lattice=9, dtype="f64", n=(n[0], n[1], 1), L=(float(n[0]), float(n[1]), 1.0), mesh=(mesh, mesh, 0),
                k_stretch=1.5, rho0=1.0, RT=1 / 3, tau=0.45, dt=0.25, bc=bc, G=(1e-3, -5e-4, 0.0), omega=0.7, phase=0.3, uw=UW,
                pw=[3e-3, -2e-3, 0, 0, 0, 0], pw_osc=[1e-3, 0, 0, 0, 0, 0])


@pytest.mark.parametrize("sides", SIDES)
@pytest.mark.parametrize("n", [(1, 20000), (2, 16384), (3, 20011), (6, 30000), (8, 30000), (40000, 5), (40001, 6), (40000, 8)],
                         ids=lambda n: f"{n[0]}x{n[1]}")
def test_thin_adjoint_matches_general(sides, n, monkeypatch):
    bc = SIDES[sides]
    if any(bc[2 * a] != 0 and n[a] < 2 for a in range(2)):
        pytest.skip("wall-bounded axes have at least two cells")
    print(f"[adjoint thin] {sides} n={n}", flush=True)
    cfg = cfg_of(n, bc, 0)
    Q, D, shp = M.shape_of(cfg)
    f = torch.empty((Q,) + shp, dtype=torch.float64, device="cuda")
    G = dev(field(51, (D,) + shp, 2e-3))
    ctx = M.dugks_init(cfg, f, dev(1 + field(52, shp, 0.02)), dev(field(53, (D,) + shp, 0.05)), G)
    try:
        f += dev(field(54, f.shape, 1e-3))
        lam = dev(field(55, f.shape, 1.0))
        out, grad = [], []
        for general in ("1", "0"):
            monkeypatch.setenv("DUGKS_ADJOINT_GENERAL", general)
            o = torch.full_like(f, float("nan"))
            g = dev(field(56, (D,) + shp, 1e-3))
            M.dugks_step_adjoint(ctx, f, lam, o, G, 0.4, g)
            out.append(o)
            grad.append(g)
        assert (out[0] - out[1]).abs().max() < 1e-12 * out[0].abs().max()
        assert (grad[0] - grad[1]).abs().max() < 1e-11 * grad[0].abs().max()
    finally:
        M.dugks_destroy(ctx)


@pytest.mark.parametrize("sides,n", [("channel_x", (1, 65536)), ("channel_x", (3, 65536)), ("lid", (2, 65536)), ("lid", (4, 16384)),
                                     ("box", (65536, 5)), ("lid", (256, 256)), ("box", (4, 65536))],
                         ids=lambda v: v if isinstance(v, str) else f"{v[0]}x{v[1]}")
def test_default_no_slower_than_general(sides, n, monkeypatch):
    cfg = cfg_of(n, SIDES[sides], 0)
    Q, D, shp = M.shape_of(cfg)
    f = torch.empty((Q,) + shp, dtype=torch.float64, device="cuda")
    ctx = M.dugks_init(cfg, f)
    us = {}
    try:
        lam = dev(field(55, f.shape, 1.0))
        out = torch.empty_like(f)
        for general in ("0", "1"):
            monkeypatch.setenv("DUGKS_ADJOINT_GENERAL", general)
            best = 1e9
            for _ in range(5):
                t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                t[0].record()
                for _ in range(10):
                    M.dugks_step_adjoint(ctx, f, lam, out)
                t[1].record()
                torch.cuda.synchronize()
                best = min(best, t[0].elapsed_time(t[1]) * 100)
            us[general] = best
    finally:
        M.dugks_destroy(ctx)
    print(f"[adjoint thin] {sides} {n}: {us['0']:.1f} us, general pass {us['1']:.1f}", flush=True)
    assert us["0"] < 1.25 * us["1"]


def test_first_call_in_a_capture():
    # a thin mesh's scratch is not allocated inside a capture: the tiles take it
    cfg = cfg_of((1, 20000), SIDES["channel_x"], 0)
    f = torch.empty((9, 1, 20000, 1), dtype=torch.float64, device="cuda")
    ctx = M.dugks_init(cfg, f)
    try:
        lam = dev(field(55, f.shape, 1.0))
        out = torch.full_like(f, float("nan"))
        torch.cuda.synchronize()
        s = torch.cuda.Stream()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            M.dugks_step_adjoint(ctx, f, lam, out)
        ref = torch.empty_like(f)
        M.dugks_step_adjoint(ctx, f, lam, ref)
        for _ in range(3):
            out.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert (out - ref).abs().max() < 1e-12 * ref.abs().max()
    finally:
        M.dugks_destroy(ctx)
