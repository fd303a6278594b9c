"""The FP64 3-D row kernel on meshes around the edges of its tiles (14 x 6 columns
of its own): against the oracle, and the same to the bit for every march chunk
(which decides the workgroups that run the wall body or the wall-free one)."""
import os

import pytest

import oracle as O
from synthetic import field
from tests.test_gpu_parity import LID3, custom_faces, rel_linf, start_state, to_dev

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu

SIZES = [(2, 2, 2), (13, 5, 3), (14, 6, 4), (15, 7, 2), (16, 8, 5), (17, 13, 9), (29, 12, 7), (31, 20, 11)]
KINDS = {
    "lid": dict(bc=(1,) * 6, uw=LID3),
    "box": dict(bc=(0,) * 6, G=(1e-4, 0, -2e-4), omega=0.1, phase=0.3),
    "noslip-field": dict(bc=(3,) * 6, uw=LID3, mesh=(1, 1, 1), k_stretch=1.5, dt=0.2, force_field=True),
    "pressure": dict(bc=(2, 2, 3, 1, 0, 0), uw=LID3, pw=[1e-3, 0, 0, 0, 0, 0], pw_osc=[-2e-3, 1e-3, 0, 0, 0, 0],
                     omega=0.05, phase=0.4),
    "duct-field": dict(bc=(0, 0, 3, 1, 2, 3), uw=LID3, pw=[0, 0, 0, 0, 1e-3, 0], force_field=True, omega=0.1),
    "original-field": dict(bc=(0, 0, 1, 2, 3, 3), uw=LID3, model=1, force_field=True, G=(1e-4, 0, 0)),
}


def run(cfg, f0, force, chunk, n=3, t0=0.4):
    a = to_dev(f0, cfg)
    b = torch.empty_like(a)
    old = os.environ.get("DUGKS_CHUNK")
    os.environ["DUGKS_CHUNK"] = str(chunk)
    try:
        ctx = M.dugks_init(cfg, b)
    finally:
        if old is None:
            del os.environ["DUGKS_CHUNK"]
        else:
            os.environ["DUGKS_CHUNK"] = old
    try:
        which = M.dugks_run(ctx, a, b, n, force, t0)
        torch.cuda.synchronize()
        return b if which else a
    finally:
        M.dugks_destroy(ctx)


@pytest.mark.parametrize("lattice", [19, 27])
@pytest.mark.parametrize("kind", list(KINDS))
def test_tile_edges(kind, lattice):
    for n in SIZES:
        cfg = dict(lattice=lattice, dtype="f64", n=n, L=tuple(float(v) for v in n), rho0=1.0, RT=1 / 3, tau=0.3, dt=0.5)
        cfg.update(KINDS[kind])
        print(f"[row] D3Q{lattice} {kind} {n}", flush=True)
        force = field(5, (3,) + n[::-1], 1e-4) if cfg.get("force_field") else None
        f0 = start_state(cfg, 11, force)
        dev = None if force is None else to_dev(force, cfg)
        got = run(cfg, f0, dev, 0)
        assert rel_linf(got.cpu().numpy(), O.run(cfg, f0, 3, force, 0.4)) < 3e-12  # 1e-12 a step
        for chunk in (1, 2, 3, 16):
            assert torch.equal(run(cfg, f0, dev, chunk), got), (n, chunk)


def test_custom_faces_and_degenerate_periodic_axes():
    for n, bc in (((1, 6, 5), (0, 0, 3, 3, 1, 1)), ((9, 1, 4), (1, 3, 0, 0, 2, 1)), ((16, 9, 1), (1, 1, 1, 1, 0, 0)),
                  ((3, 2, 2), (0,) * 6)):
        cfg = dict(lattice=19, dtype="f64", n=n, L=tuple(float(v) for v in n), rho0=1.0, RT=1 / 3, tau=0.3, dt=0.2,
                   bc=bc, uw=LID3, pw=[0, 0, 0, 0, 1e-3, 0], mesh=(2, 2, 2), G=(1e-4, 0, 2e-4),
                   faces=tuple(custom_faces(3 + a, n[a], float(n[a])) for a in range(3)))
        print(f"[row] custom faces {n} {bc}", flush=True)
        f0 = start_state(cfg, 11, None)
        got = run(cfg, f0, None, 0)
        assert rel_linf(got.cpu().numpy(), O.run(cfg, f0, 3, None, 0.4)) < 3e-12
        assert torch.equal(run(cfg, f0, None, 2), got)
