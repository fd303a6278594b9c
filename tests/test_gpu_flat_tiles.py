"""The flat tiles of the D2Q9 kernel (32 x 8, 32 x 6 and 64 x 4 cells, one of them
halo on each side), which meshes of few rows, or of few columns between walls,
take: around the edges of the tiles, a run must give to the bit what single
steps give, and both agree with the oracle (1e-12 a step, as for the others).
And such meshes must not cost much more per cell than a square one: on tiles of
32 x 16 cells they took three to twelve times as long."""
import pytest

import oracle as O
from synthetic import field
from tests.test_gpu_parity import LID, c2, rel_linf, start_state, to_dev
from tests.test_gpu_tile import both_ways, config

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu

# 32 x 8: (7749, 1) to (7801, 18), (16, 20000), (31, 9001); 64 x 4: (20000, 2), (15873, 3);
# 32 x 6: the last three
SIZES = [(7749, 2), (7800, 5), (7801, 6), (7799, 13), (7801, 18), (16, 20000), (31, 9001), (20000, 2), (15873, 3), (24000, 4),
         (23999, 3), (24031, 7)]


@pytest.mark.parametrize("kind", ["lid", "noslip-field", "pressure", "original"])
@pytest.mark.parametrize("n", SIZES, ids=lambda n: f"{n[0]}x{n[1]}")
def test_run_equals_steps_and_oracle(kind, n):
    check(config(kind, *n, "f64"), n)


@pytest.mark.parametrize("bc", [(0, 0, 0, 0, 0, 0), (1, 3, 0, 0, 0, 0)], ids=["box", "x walls"])
@pytest.mark.parametrize("n", [(20000, 1), (20001, 2), (7800, 1), (24000, 3), (16000, 16), (9, 20011)],
                         ids=lambda n: f"{n[0]}x{n[1]}")
def test_periodic_across(bc, n):
    for force in (False, True):
        check(c2("flat", n, bc, uw=LID, force_field=force, G=(2e-4, -1e-4, 0), omega=0.05, phase=0.3), n)


def check(cfg, n):
    print(f"[flat tiles] {cfg['bc']} {n}", flush=True)
    force = field(5, (2, 1, n[1], n[0]), 1e-4) if cfg.get("force_field") else None
    f0 = start_state(cfg, 11, force)
    dev = None if force is None else to_dev(force, cfg)
    (a, b), (c, d) = both_ways(cfg, f0, dev, 5, 0.7)
    assert torch.equal(a, c) and torch.equal(b, d)
    assert rel_linf(a.cpu().numpy(), O.run(cfg, f0, 5, force, 0.7)) < 5e-12


def us_per_step(n, one):
    cfg = c2("time", n, (1, 1, 1, 1, 0, 0), uw=LID)
    f = torch.empty((9, 1, n[1], n[0]), dtype=torch.float64, device="cuda")
    g = torch.empty_like(f)
    ctx = M.dugks_init(cfg, f)
    best = 1e9
    try:
        for _ in range(6):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            for _ in range(20 if one else 1):
                M.dugks_run(ctx, f, g, 1 if one else 20)
            t[1].record()
            torch.cuda.synchronize()
            best = min(best, t[0].elapsed_time(t[1]) * 50)
    finally:
        M.dugks_destroy(ctx)
    return best


@pytest.mark.parametrize("one", [False, True], ids=["run", "steps"])
def test_time_per_cell(one):
    square = us_per_step((1024, 1024), one)
    for n in ((65536, 16), (524288, 2), (16384, 64)):
        t = us_per_step(n, one)
        print(f"[flat tiles] {n}: {t:.1f} us a step, 1024 x 1024: {square:.1f}", flush=True)
        assert t < 1.9 * square
