"""The library's host code where something goes wrong or runs on a special stream, without a GPU: in a process
of its own against a stand-in for the HIP runtime (tests/fake_hip/fake_hip.c: device memory is host memory,
kernels do nothing), which can refuse a copy and count the launches of other threads."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIP = os.environ.get("ROCM_PATH", "/opt/rocm") + "/include"

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None or not os.path.isdir(HIP), reason="no gcc or HIP headers")

PRELUDE = """
import ctypes, sys
sys.modules["torch"] = None  # the stand-in is the only runtime here
sys.path.insert(0, {root!r})
fake = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
fake.fake_watch.argtypes = [ctypes.c_void_p]
import numpy as np
from paper_1902_09813_amd import btrt, btrt3
"""


@pytest.fixture(scope="module")
def fake_lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so")
    subprocess.run(["gcc", "-O1", "-std=c11", "-shared", "-fPIC", "-pthread", "-I", HIP,
                    os.path.join(HERE, "fake_hip", "fake_hip.c"), "-o", out], check=True, capture_output=True, text=True)
    return out


def run(fake_lib, body):
    res = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, lib=fake_lib) + body], capture_output=True,
                         text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.strip().endswith("done"), res.stdout + res.stderr


def test_reads_on_the_per_thread_stream_stay_on_the_calling_thread(fake_lib):
    # hipStreamPerThread (2) is another stream in each thread: a copy launched by a helper thread would not be
    # ordered behind the caller's work. Any other stream is shared out.
    run(fake_lib, """
seen = []
for stream in (0x1000, 2):
    p = btrt.Problem(700, 600, A0=(0.01, 0.0, 0.01))
    p.grid.stream = stream
    p3 = btrt3.Problem3(96, 80, 70, A0=(0.05, 0.01, 0.005, 0.04, -0.008, 0.03))
    p3.grid.stream = stream
    phi0, phi3 = np.zeros((600, 700)), np.zeros((70, 80, 96))
    with btrt.Solver(p, phi0) as s, btrt3.Solver3(p3, phi3) as s3, btrt.Batch([(p, phi0)], stream=stream) as b:
        for read in (s.field, s3.field, lambda: b.field(0)):
            fake.fake_watch(stream)
            read()
            seen.append((fake.fake_launches(), fake.fake_foreign_launches()))
assert all(t > 3 and f > 0 for t, f in seen[:3]), seen
assert all(t > 3 and f == 0 for t, f in seen[3:]), seen
print("done")
""")


def test_a_wall_schedule_whose_upload_fails_leaves_the_old_one_in_force(fake_lib):
    # 500 rows go up in three pieces behind the copy of the row in force; each of the four copies fails once.
    # The values in force at every later step (in the checkpoint's last bytes) stay those of the old schedule.
    run(fake_lib, """
n, rows = 40, 500
P = 4 * (n + n) + 4
rng = np.random.default_rng(1)
first, second, third = rng.random((3, rows, P))

def solver():
    return btrt.Solver(btrt.Problem(n, n, A0=(0.01, 0.0, 0.01), bc_type=(1,) * 4, bc_value=(0.1, 0.2, 0.3, 0.4)),
                       np.zeros((n, n)))

def entries(s, steps):
    out = []
    for _ in range(steps):
        out.append(s.step(1).checkpoint()[-8 * (P + 4):])
    return out

with solver() as s, solver() as ref:
    for x in (s, ref):
        x.set_walls(first).step(7)
    for round in range(2):
        for k in range(4):
            fake.fake_fail_copy(k)
            try:
                s.set_walls(second)
            except btrt.BtrtError as e:
                assert e.code == btrt.E_DEVICE, e
            else:
                raise AssertionError("no failure at copy %d" % k)
            fake.fake_fail_copy(-1)
        assert entries(s, 150) == entries(ref, 150), round
        want = first if round == 0 else third
        assert s.checkpoint()[-8 * (P + 4):][:8 * P] == want[(157 if round == 0 else 150) - 1].tobytes()
        for x in (s, ref):
            x.set_walls(third)
    for x in (s, ref):
        x.set_walls(first).step(rows)
        try:
            x.step(1)
        except btrt.BtrtError as e:
            assert e.code == btrt.E_INVAL
        else:
            raise AssertionError("stepped past the schedule")
print("done")
""")


def test_reported_sweeps_are_the_launches_made(fake_lib):
    # btrt_get_sweep against the launches a stream gets: k launches for k times its steps, one more for a step
    # more (or for what the general model's walkers make of the rest), for every form, storage and model.
    run(fake_lib, """
S = 0x1000
kinds = set()
for n in (16, 64, 200, 330, 500, 1100):
    for precision in (btrt.F64, btrt.F32, btrt.F16DEV):
        for kw in (dict(), dict(k2=1.1), dict(bc_type=(1,) * 4), dict(bc_type=(1,) * 4, k2=0.9), dict(beta=0.3),
                   dict(flux_c=(0.01, 0.0), flux_q=2.0), dict(flux_c=(0.01, 0.0), flux_q=2.0, k2=1.1)):
            if "flux_c" in kw and precision == btrt.F16DEV:
                continue
            p = btrt.Problem(n, n, A0=(0.01, 0.0, 0.01), precision=precision, **kw)
            p.grid.stream = S
            with btrt.Solver(p, np.zeros((n, n))) as s:
                s.step(1)
                for shape in ((0, 0, 0, 0), (1, 0, 0, 0), (2, 0, 0, 1), (4, 0, 0, 0), (4, 16, 4, 0), (6, 0, 0, 0), (7, 32, 1, 0)):
                    w = s.set_launch(*shape).sweep()
                    k = w["steps_per_launch"]
                    kinds.add((w["kernel"], w["moments"]))
                    fake.fake_watch(S)
                    s.step(5 * k)
                    assert fake.fake_launches() == 5, (n, precision, kw, shape, w, fake.fake_launches())
                    s.step(k + 1)
                    assert fake.fake_launches() == 7, (n, precision, kw, shape, w, fake.fake_launches())
                    assert w["automatic"] == (shape[0] == 0) and w["columns"] > 0 and w["rows"] > 0
                    assert w["moments"] == ("k2" not in kw)
                    if shape[0] == 1:
                        assert (w["kernel"], w["columns"], w["rows"], w["threads"]) == (btrt.SWEEP_STEP, 64, 4, 256)
                    if shape == (4, 16, 4, 0):
                        assert (w["kernel"], w["rows"], w["threads"]) == (btrt.SWEEP_STRIPS, 16, 256)
                    words = 3 if w["moments"] else 10
                    if precision != btrt.F16DEV:
                        assert w["bytes_per_node"] == 2 * words * (8 if precision == btrt.F64 else 4)
assert kinds == {(btrt.SWEEP_STEP, 0), (btrt.SWEEP_STEP, 1), (btrt.SWEEP_TILE, 0), (btrt.SWEEP_STRIPS, 0),
                 (btrt.SWEEP_STRIPS, 1), (btrt.SWEEP_BLOCKS, 0), (btrt.SWEEP_BLOCKS, 1), (btrt.SWEEP_REGIONS, 1)}, kinds
print("done")
""")


def test_a_tuned_shape_runs_on_another_handle_and_follows_the_model(fake_lib):
    # What btrt_tune keeps, set elsewhere as btrt_get_sweep says to, runs the same launches; and an automatic
    # choice is made again when a wall schedule changes the model.
    run(fake_lib, """
seen = set()
for n in (20, 64, 100, 330, 500, 1100):
    for kw, budget in ((dict(), 2000), (dict(), 30), (dict(k2=1.1), 2000), (dict(k2=1.1), 30)):
        make = lambda: btrt.Solver(btrt.Problem(n, n, A0=(0.01, 0.0, 0.01), bc_type=(1,) * 4, **kw), np.zeros((n, n)))
        walls = np.zeros((40, 8 * n + 4))
        with make() as a, make() as b:
            best, used = a.tune(budget)  # with few steps only the automatic shape and its like are timed
            assert used > 0 and best == a.launch()
            w = a.sweep()
            seen.add(w["automatic"])
            b.set_launch(*((0, 0, 0, 0) if w["automatic"] else best))
            assert b.sweep() == w, (n, kw, w, b.sweep())
            for s in (a, b):
                s.set_walls(walls)
            assert a.sweep() == b.sweep(), (n, kw, a.sweep(), b.sweep())
            if w["automatic"]:
                with make() as c:
                    assert c.set_walls(walls).sweep() == a.sweep(), (n, kw)
assert seen == {0, 1}, seen
print("done")
""")
