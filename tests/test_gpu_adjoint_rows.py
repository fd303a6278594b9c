"""Tile rows of the D2Q9 FP64 adjoint inside walls: with as many 16-row tiles, a
mesh of fewer rows must not take longer than one of more.  (Chosen with the share
of the tiles at walls, 5035 x 54 took 8-row tiles: 47.4 us where 16-row ones take
40.1 and 5035 x 60 44.5.)"""
import pytest

from tests.test_gpu_parity import LID, c2

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu


def us_per_step(n):
    cfg = c2("rows", n, (1, 1, 1, 1, 0, 0), uw=LID)
    f = torch.empty((9, 1, n[1], n[0]), dtype=torch.float64, device="cuda")
    ctx = M.dugks_init(cfg, f)
    lam, out = torch.ones_like(f), torch.empty_like(f)
    best = 1e9
    try:
        for _ in range(8):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            for _ in range(20):
                M.dugks_step_adjoint(ctx, f, lam, out, None, 0.0, None)
            t[1].record()
            torch.cuda.synchronize()
            best = min(best, t[0].elapsed_time(t[1]) * 50)
    finally:
        M.dugks_destroy(ctx)
    return best


def test_fewer_rows_take_no_longer():
    few, more = us_per_step((5035, 54)), us_per_step((5035, 60))
    print(f"[adjoint rows] 5035 x 54 {few:.1f} us, 5035 x 60 {more:.1f}", flush=True)
    assert few < more
