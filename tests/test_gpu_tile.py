"""The D2Q9 tile kernel: several steps per launch must give, to the bit, what
single steps give, on meshes around the edges of its tiles (32 x 16 cells with
an overlap of one cell per step on each side), for every wall kind, mesh kind,
forcing and model; and both agree with the oracle."""
import numpy as np
import pytest

import oracle as O
from synthetic import field
from tests.test_gpu_parity import LID, c2, custom_faces, rel_linf, start_state, to_dev

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_1411_6121_amd")

pytestmark = pytest.mark.gpu

SIZES = [(1, 2), (2, 3), (19, 4), (20, 5), (21, 9), (28, 12), (29, 13), (30, 14), (31, 15), (32, 16), (33, 17),
         (63, 31), (97, 40)]
KINDS = {
    "lid": dict(bc=(1, 1, 1, 1, 0, 0), uw=LID),
    "box": dict(bc=(0, 0, 0, 0, 0, 0), G=(2e-4, -1e-4, 0), omega=0.05, phase=0.3),
    "noslip-field": dict(bc=(3, 3, 3, 3, 0, 0), uw=LID, mesh=(1, 1, 0), k_stretch=1.5, dt=0.2, force_field=True),
    "pressure": dict(bc=(2, 2, 3, 1, 0, 0), uw=LID, pw=[1e-3, 0, 0, 0, 0, 0], pw_osc=[-3e-3, 1e-3, 0, 0, 0, 0],
                     omega=0.05, phase=0.4),
    "mixed-field": dict(bc=(1, 3, 0, 0, 0, 0), uw=[[0, 0.02, 0], [0, -0.01, 0]] + [[0, 0, 0]] * 4, force_field=True,
                        omega=0.1),
    "original": dict(bc=(0, 0, 1, 2, 0, 0), uw=LID, model=1, force_field=True, G=(1e-4, 0, 0)),
}


def config(kind, nx, ny, dtype):
    kw = dict(KINDS[kind])
    bc = list(kw.pop("bc"))
    if nx < 2:
        bc[0] = bc[1] = 0
    return c2(kind, (nx, ny), tuple(bc), dtype=dtype, **kw)


def both_ways(cfg, f0, force, n, t0):
    """(result, state before the last step) of dugks_run and of n dugks_step calls"""
    out = []
    for one in (False, True):
        a = to_dev(f0, cfg)
        b = torch.empty_like(a)
        ctx = M.dugks_init(cfg, b)
        try:
            if one:
                for k in range(n):
                    M.dugks_step(ctx, a, b, force, t0 + k * cfg["dt"])
                    a, b = b, a
            elif M.dugks_run(ctx, a, b, n, force, t0):
                a, b = b, a
            torch.cuda.synchronize()
            out.append((a, b))
        finally:
            M.dugks_destroy(ctx)
    return out


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("kind", list(KINDS))
def test_run_equals_steps_and_oracle(kind, dtype):
    for nx, ny in SIZES:
        cfg = config(kind, nx, ny, dtype)
        print(f"[tile] {kind} {dtype} {nx}x{ny}", flush=True)
        force = field(5, (2, 1, ny, nx), 1e-4) if cfg.get("force_field") else None
        f0 = start_state(cfg, 11, force)
        dev = None if force is None else to_dev(force, cfg)
        for n in (2, 13, 20):
            (a, b), (c, d) = both_ways(cfg, f0, dev, n, 0.7)
            assert torch.equal(a, c), (nx, ny, n)
            assert torch.equal(b, d), (nx, ny, n)
            if dtype == "f64" and n == 13:
                ref = O.run(cfg, f0, n, force, 0.7)
                assert rel_linf(a.cpu().numpy(), ref) < 1e-11  # 1e-12 a step


@pytest.mark.parametrize("kind", ["lid", "noslip-field"])
def test_many_tiles_against_oracle(kind):
    # more tiles than CUs, most of them clear of walls: the kernel's other body
    cfg = config(kind, 607, 401, "f64")
    print(f"[tile] {kind} 607x401", flush=True)
    force = field(5, (2, 1, 401, 607), 1e-4) if cfg.get("force_field") else None
    f0 = start_state(cfg, 11, force)
    dev = None if force is None else to_dev(force, cfg)
    (a, b), (c, d) = both_ways(cfg, f0, dev, 8, 0.0)
    assert torch.equal(a, c) and torch.equal(b, d)
    assert rel_linf(a.cpu().numpy(), O.run(cfg, f0, 8, force, 0.0)) < 1e-11


def test_custom_faces_periodic_and_wall():
    for bc in ((0, 0, 1, 3, 0, 0), (3, 2, 0, 0, 0, 0)):
        cfg = c2("faces", (45, 38), bc, uw=LID, pw=[0, 1e-3, 0, 0, 0, 0], mesh=(2, 2, 0), dt=0.2,
                 faces=(custom_faces(1, 45, 45.0), custom_faces(2, 38, 38.0), None), G=(1e-4, 2e-4, 0))
        print(f"[tile] custom faces {bc}", flush=True)
        f0 = start_state(cfg, 11, None)
        (a, b), (c, d) = both_ways(cfg, f0, None, 9, 0.3)
        assert torch.equal(a, c) and torch.equal(b, d)
        assert rel_linf(a.cpu().numpy(), O.run(cfg, f0, 9, None, 0.3)) < 1e-11


def test_run_edges():
    cfg = config("lid", 33, 17, "f64")
    print("[tile] zero and one step, replay in a captured graph", flush=True)
    f0 = start_state(cfg, 11, None)
    a = to_dev(f0, cfg)
    b = torch.empty_like(a)
    ctx = M.dugks_init(cfg, b)
    try:
        assert M.dugks_run(ctx, a, b, 0) == 0
        assert np.array_equal(a.cpu().numpy(), f0)
        assert M.dugks_run(ctx, a, b, 1) == 1
        with pytest.raises(M.DugksError):
            M.dugks_run(ctx, a, a, 5)
        # several steps per launch inside a captured graph, replayed between eager work
        a.copy_(to_dev(f0, cfg))
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            M.dugks_run(ctx, a, b, 14)
        ref = to_dev(f0, cfg)
        spare = torch.empty_like(ref)
        for rep in range(3):
            g.replay()
            torch.cuda.synchronize()
            M.dugks_run(ctx, ref, spare, 14)
            torch.cuda.synchronize()
            assert torch.equal(a, ref), rep
    finally:
        M.dugks_destroy(ctx)
