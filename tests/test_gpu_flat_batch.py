"""Batches on flat tiles (most of their cells in few rows, or most tiles at
walls): per instance to the bit what the instance gives alone, eager and in
replayed graphs, tuned or not; and no more time per cell than twice that of
square instances (on 32 x 16 tiles four times)."""
import pytest

from synthetic import field
from tests.test_gpu_batch import single_run

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu

LID = [[0, 0.01, 0], [0, -0.02, 0], [0.02, 0, 0], [0.1, 0, 0], [0, 0, 0], [0, 0, 0]]


def instance(i, n, bc, stretch):
    return dict(lattice=9, dtype="f64", n=n + (1,), L=(float(n[0]), float(n[1]), 1.0), rho0=1.0, RT=1 / 3, tau=0.3 + 0.01 * i,
                mesh=tuple(1 if stretch and bc[2 * a] and n[a] > 2 else 0 for a in range(2)) + (0,), k_stretch=1.2, dt=0.1,
                bc=bc, uw=LID, G=(1e-4, -2e-5, 0.0), omega=0.02 * i, phase=0.1 * i)


# instances, each with a thick one between (64 x 4, 32 x 6 and 32 x 8 tiles)
SETS = {"two rows": [(2101 + 61 * i, 2) for i in range(40)], "four rows": [(2101 + 61 * i, 3 + i % 2) for i in range(40)],
        "small boxes": [(40 + i, 17 + i % 30) for i in range(60)]}


@pytest.mark.parametrize("force", [False, True])
@pytest.mark.parametrize("name", SETS)
def test_equals_single_instances(name, force):
    print(f"[flat batch] {name} force {force}", flush=True)
    sides = [(1, 1, 1, 1, 0, 0), (0, 0, 3, 1, 0, 0), (2, 2, 3, 3, 0, 0), (1, 3, 0, 0, 0, 0)]
    ns = SETS[name] + [(61, 45)]
    cfgs = [instance(i, n, sides[i % 3 if i % 9 else 3], i % 4 == 1) for i, n in enumerate(ns)]
    forces = [torch.from_numpy(field(50 + i, (2, 1, n[1], n[0]), 1e-5)).to("cuda") if force and i % 2 else None
              for i, n in enumerate(ns)]
    B = M.BatchSolver(cfgs, forces=forces if force else None)
    try:
        f0 = [B.state(i).clone() for i in range(len(ns))]
        B.run(3)
        B.run(4, use_graph=True)
        B.run(4, use_graph=True)
        B.tune(nsteps=2)
        B.run(4, use_graph=True)
        torch.cuda.synchronize()
        for i, c in enumerate(cfgs):
            assert torch.equal(B.state(i), single_run(c, f0[i], 15, forces[i])), f"instance {i}"
    finally:
        B.close()


def test_time_per_cell():
    def us(ns):
        B = M.BatchSolver([instance(0, n, (1, 1, 1, 1, 0, 0), False) for n in ns])
        best = 1e9
        try:
            for _ in range(6):
                t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                t[0].record()
                B.run(20)
                t[1].record()
                torch.cuda.synchronize()
                best = min(best, t[0].elapsed_time(t[1]) * 50)
        finally:
            B.close()
        return best

    square = us([(128, 128)] * 32)
    for n in ((4096, 2), (2048, 4), (512, 16)):
        t = us([n] * (32 * 128 * 128 // (n[0] * n[1])))
        print(f"[flat batch] {n}: {t:.1f} us a step, 128 x 128: {square:.1f}", flush=True)
        assert t < 2 * square
