"""The host side where the runtime fails or a count is extreme, on a device that
runs nothing (fake_device.c, in a process of its own): no GPU is used."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
for n in ("fake_launches", "fake_uploads"): getattr(fake, n).argtypes = [ctypes.c_longlong]
for n in ("fake_launch_count", "fake_upload_count"): getattr(fake, n).restype = ctypes.c_longlong
for n in ("fake_upload_bytes", "fake_held_bytes"): getattr(fake, n).restype = ctypes.c_size_t
import paper_1411_6121_amd as M
lib = M.load()
VP = ctypes.c_void_p
def cfg(n, **kw):
    return dict(dict(lattice=9, dtype="f64", n=n, L=tuple(float(v) for v in n), rho0=1.0, RT=1/3, tau=0.4, dt=0.2,
                     bc=(0,) * 6), **kw)
def batch(cfgs):
    keep = [M.config(c) for c in cfgs]
    b = VP()
    rc = lib.dugks_batch_create((M.Config * len(keep))(*keep), len(keep), (ctypes.c_int64 * len(keep))(), None,
                                ctypes.byref(b))
    return rc, b
def context(c):
    h = VP()
    assert lib.dugks_init(ctypes.byref(M.config(c)), None, None, None, VP(4096), None, ctypes.byref(h)) == M.OK
    return h
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_device.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", "-o", so, os.path.join(HERE, "fake_device.c")], check=True)
    return so


def run(fake, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, fake], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])


def test_table_that_was_not_uploaded_is_not_used(fake):
    # the autotuner tries one step per launch more than the batch has tables
    # for; where that table's upload fails, the next call must not take it
    run(fake, """
rc, b = batch([cfg((300, 200, 1))] * 20)
assert rc == M.OK
t, c = ctypes.c_int(), ctypes.c_int()
args = (b, VP(4096), VP(8192), None, None, 2, None, ctypes.byref(t), ctypes.byref(c))
for _ in range(2):
    fake.fake_uploads(0)
    assert lib.dugks_batch_tune(*args) == M.EHIP
fake.fake_uploads(-1)
held = fake.fake_held_bytes()
assert lib.dugks_batch_tune(*args) == M.OK
assert fake.fake_upload_count() > 0 and fake.fake_held_bytes() > held
lib.dugks_batch_destroy(b)
assert fake.fake_held_bytes() == 0
""")


@pytest.mark.parametrize("lattice,dtype", [(9, "f64"), (9, "f32"), (19, "f64"), (19, "f32")])
@pytest.mark.parametrize("batched", [False, True])
def test_any_step_count_is_taken_launch_by_launch(fake, lattice, dtype, batched):
    # the largest step counts: nothing is held per step (2 GiB of address space
    # for the whole process), and the run goes on until a launch fails
    run(fake, f"""
c = cfg((40, 20, 1) if {lattice} == 9 else (8, 8, 8), lattice={lattice}, dtype="{dtype}")
if {batched}: rc, h = batch([c]); assert rc == M.OK
else: h = context(c)
import resource
resource.setrlimit(resource.RLIMIT_AS, (2 << 30, 2 << 30))
w = ctypes.c_int()
for n in (2**31 - 1, 2**31 - 2, 2**31 - 9):
    fake.fake_launches(50)
    if {batched}: rc = lib.dugks_batch_run(h, VP(4096), VP(8192), None, None, n, 0, None, ctypes.byref(w))
    else: rc = lib.dugks_run(h, VP(4096), VP(8192), None, 0.0, n, None, ctypes.byref(w))
    assert rc == M.EHIP and fake.fake_launch_count() == 50, (n, rc, fake.fake_launch_count())
""")


def test_tuning_steps_are_taken_launch_by_launch(fake):
    run(fake, """
rc, b = batch([cfg((300, 200, 1))] * 20)
import resource
resource.setrlimit(resource.RLIMIT_AS, (2 << 30, 2 << 30))
t, c = ctypes.c_int(), ctypes.c_int()
fake.fake_launches(50)
rc = lib.dugks_batch_tune(b, VP(4096), VP(8192), None, None, 2**31 - 1, None, ctypes.byref(t), ctypes.byref(c))
assert rc == M.EHIP and fake.fake_launch_count() == 50
""")


def test_batch_of_very_many_tiles_is_created(fake):
    # more than 2^26 tiles of 30 x 14 cells: their tables go to the device in
    # pieces (the host holds less than half a GiB at any time)
    run(fake, """
rc, b = batch([cfg((40, 20, 1))])  # (the runtime's own start)
lib.dugks_batch_destroy(b)
fake.fake_uploads(-1)
rc, b = batch([cfg((170000, 170000, 1))])
assert rc == M.OK, lib.dugks_batch_last_error(None)
peak = int([l for l in open("/proc/self/status") if l.startswith("VmHWM")][0].split()[1]) >> 10
assert peak < 512, peak  # MiB
tiles = -(-170000 // 30) * -(-170000 // 14)
assert tiles > 2**26 and fake.fake_upload_bytes() >= 16 * tiles
# and its launches (single steps: a run of one) hold less than 2^32 threads each
fake.fake_launches(-1)
assert lib.dugks_batch_run(b, VP(4096), VP(8192), None, None, 1, 0, None, None) == M.OK
assert fake.fake_launch_count() > tiles * 512 // 2**32 + 1
lib.dugks_batch_destroy(b)
assert fake.fake_held_bytes() == 0
""")
