"""Steps per launch of the D2Q9 kernel on meshes with walls across one axis whose
32 x 16 tiles nearly fill the chip: a run gives to the bit what single steps give
and agrees with the oracle (1e-12 a step), on both sides of the rule's lines
(256 tiles of one step, 512 of several).  And a wall across x costs such a mesh
no more than half of its periodic step: with single steps where several a launch
are better it took 1.8 times as long."""
import pytest

import oracle as O
from synthetic import field
from tests.test_gpu_parity import LID, c2, rel_linf, start_state, to_dev
from tests.test_gpu_tile import both_ways

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bc", [((3654, 16), (1, 1, 0, 0, 0, 0)), ((3841, 15), (1, 3, 0, 0, 0, 0)), ((450, 200), (0, 0, 1, 1, 0, 0)),
                                  ((16, 3500), (0, 0, 3, 1, 0, 0)), ((481, 209), (1, 1, 0, 0, 0, 0))],
                         ids=lambda v: "x".join(map(str, v)))
def test_run_equals_steps_and_oracle(n, bc):
    cfg = c2("steps", n, bc, uw=LID, force_field=True, G=(2e-4, -1e-4, 0), omega=0.05, phase=0.3)
    force = field(5, (2, 1, n[1], n[0]), 1e-4)
    f0 = start_state(cfg, 11, force)
    (a, b), (c, d) = both_ways(cfg, f0, to_dev(force, cfg), 5, 0.7)
    assert torch.equal(a, c) and torch.equal(b, d)
    assert rel_linf(a.cpu().numpy(), O.run(cfg, f0, 5, force, 0.7)) < 5e-12


def us_per_step(bc):
    cfg = c2("time", (3654, 16), bc, uw=LID)
    f = torch.empty((9, 1, 16, 3654), dtype=torch.float64, device="cuda")
    g = torch.empty_like(f)
    ctx = M.dugks_init(cfg, f)
    best = 1e9
    try:
        for _ in range(8):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            M.dugks_run(ctx, f, g, 60)
            t[1].record()
            torch.cuda.synchronize()
            best = min(best, t[0].elapsed_time(t[1]) * 1e3 / 60)
    finally:
        M.dugks_destroy(ctx)
    return best


def test_time_of_a_wall():
    wall, box = us_per_step((1, 1, 0, 0, 0, 0)), us_per_step((0, 0, 0, 0, 0, 0))
    print(f"[tile steps] walls across x {wall:.2f} us a step, periodic {box:.2f}", flush=True)
    assert wall < 1.5 * box
