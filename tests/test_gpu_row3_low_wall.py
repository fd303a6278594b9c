"""The low z wall of the FP64 3-D row kernel, whose face is formed before the
march: every wall kind there, with the fewest planes and march chunks that begin
and end at it, against the oracle (1e-12 a step, as for the others); and what z
walls may cost: on meshes of few planes they took 1.7 times the periodic step."""
import pytest

import oracle as O
from synthetic import field
from tests.test_gpu_parity import LID3, rel_linf, start_state, to_dev
from tests.test_gpu_row3 import run

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lattice", [19, 27])
@pytest.mark.parametrize("force", [False, True])
@pytest.mark.parametrize("low,high", [(1, 1), (1, 3), (2, 1), (2, 2), (3, 2), (3, 3)])
def test_low_wall(lattice, force, low, high):
    for n, mesh, xy in (((15, 7, 2), 0, (0, 0, 0, 0)), ((9, 8, 3), 1, (1, 3, 0, 0)), ((17, 6, 4), 1, (0, 0, 3, 1)),
                        ((2, 3, 5), 0, (1, 1, 1, 1)), ((1, 1, 9), 1, (0, 0, 0, 0)), ((30, 13, 18), 0, (2, 3, 1, 1))):
        cfg = dict(lattice=lattice, dtype="f64", n=n, L=tuple(float(v) for v in n), rho0=1.0, RT=1 / 3, tau=0.3, dt=0.2,
                   bc=xy + (low, high), uw=LID3, pw=[1e-3, 0, 0, 0, 2e-3, -1e-3], pw_osc=[0, 0, 0, 0, 1e-3, 5e-4],
                   mesh=tuple(mesh if v > 1 else 0 for v in n), k_stretch=1.5, omega=0.3, phase=0.2,
                   G=(1e-4, 0, -2e-4) if n[2] % 2 else (0, 0, 0), model=1 if n[2] == 4 else 0)
        print(f"[low wall] D3Q{lattice} {cfg['bc']} {n} force {force}", flush=True)
        G = field(5, (3,) + n[::-1], 1e-4) if force else None
        f0 = start_state(cfg, 11, G)
        dev = None if G is None else to_dev(G, cfg)
        got = run(cfg, f0, dev, 0)
        assert rel_linf(got.cpu().numpy(), O.run(cfg, f0, 3, G, 0.4)) < 3e-12
        for chunk in (1, 2, 7):
            assert torch.equal(run(cfg, f0, dev, chunk), got), (n, chunk)


@pytest.mark.parametrize("mesh", [0, 1], ids=["uniform", "tanh"])
def test_time_of_z_walls(mesh):
    def us(n, bc):
        cfg = dict(lattice=19, dtype="f64", n=n, L=tuple(float(v) for v in n), rho0=1.0, RT=1 / 3, tau=0.3, dt=0.2, bc=bc,
                   uw=LID3, mesh=(mesh,) * 3, k_stretch=1.0)
        f = torch.empty((19,) + n[::-1], dtype=torch.float64, device="cuda")
        g = torch.empty_like(f)
        ctx = M.dugks_init(cfg, f)
        best = 1e9
        try:
            for _ in range(6):
                t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                t[0].record()
                M.dugks_run(ctx, f, g, 20)
                t[1].record()
                torch.cuda.synchronize()
                best = min(best, t[0].elapsed_time(t[1]) * 50)
        finally:
            M.dugks_destroy(ctx)
        return best

    for n in ((512, 512, 2), (512, 256, 6)):
        walls, box = us(n, (0, 0, 0, 0, 1, 1)), us(n, (0,) * 6)
        print(f"[low wall] {n}: z walls {walls:.1f} us a step, periodic {box:.1f}", flush=True)
        assert walls < 1.5 * box
