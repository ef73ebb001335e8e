"""Bookkeeping of the host code, against the HIP stand-in of
tests/hoststub (no GPU, no kernel runs), built with AddressSanitizer and
UndefinedBehaviorSanitizer: a call that is refused because the caller captures the
stream leaves nothing marked as done, a call that fails half way counts exactly the
steps that were enqueued, graphs captured late are dropped and captured again where
the launches change, and populations are exchanged where device memory is short."""
import ctypes as C
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
WRAPPED = ["hipMalloc", "hipFree", "hipStreamBeginCapture", "hipStreamEndCapture", "hipGraphInstantiate", "hipGraphLaunch",
           "_ZN5lbmib17launch_bead_statsERKNS_3DevEiP12ihipStream_t",
           "_ZN5lbmib21launch_interp_advanceERKNS_3DevEP12ihipStream_t"]

def _asan_runtime():
    return subprocess.run([CLANG, "-print-file-name=libclang_rt.asan-x86_64.so"], capture_output=True,
                          text=True).stdout.strip()


pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm clang++")


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("stub") / "libhoststep.so")
    csrc = os.path.join(ROOT, "paper_2202_12147_amd", "csrc")
    here = os.path.join(ROOT, "tests", "hoststub")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-D__HIP_MEMORY_SCOPE_SYSTEM=5",
                    "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-g", "-O1", "-fPIC", "-shared",
                    "-D_GLIBCXX_ASSERTIONS", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    os.path.join(csrc, "runtime.cpp"), os.path.join(csrc, "adjoint.cpp"),
                    os.path.join(here, "hip_stub.cpp"), os.path.join(here, "step_control.cpp"), "-o", lib]
                   + ["-Wl,--wrap=" + w for w in WRAPPED], check=True)
    return lib


def _run(stub, body):
    """`body` in a process of its own (the stand-in's state is global), with
    `lat` a 32^3 swimmer handle, control() and records() in scope."""
    prelude = f"""
import ctypes as C, sys
sys.path.insert(0, {ROOT!r})
from paper_2202_12147_amd import lbmib, workloads as wl
lib = C.CDLL({stub!r})
lbmib._lib = lbmib.bind(lib)
def control(capturing=0, fail_instantiate=0, fail_launch=-1):
    lib.control(capturing, fail_instantiate, fail_launch)
def records():
    out = (C.c_long * 4)()
    lib.records(out)
    return list(out)
lib.limit_malloc.argtypes = [C.c_size_t]
def allocations():
    out = (C.c_long * 2)()
    lib.allocations(out)
    return list(out)
def refused(f, *a):
    try:
        f(*a)
    except lbmib.LbmError as e:
        assert e.code == -3, e
    else:
        raise AssertionError("the call was not refused")
case = wl.small_case()
def handle(**kw):
    return lbmib.from_workload(case, **kw)
"""
    env = dict(os.environ, LD_PRELOAD=_asan_runtime(), ASAN_OPTIONS="detect_leaks=0:abort_on_error=1")
    r = subprocess.run([sys.executable, "-c", prelude + body], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("storage", [0, 1])  # the fused and the two-stream schedule
def test_refused_under_capture_leaves_the_marks_to_be_made(stub, storage):
    _run(stub, f"""
lat = handle(storage={storage})
control(capturing=1)
refused(lat.step, 3)
assert records()[0] == 0 and lat.time == 0
lat.set_populations([0.0] * (19 * 32 ** 3))    # nothing was stepped
control()
lat.step(3)
assert records()[0] == 1 and lat.time == 3
""")


def test_recorded_marks_are_made_again(stub):
    # a handle without graphs may be recorded by the caller; its marks are then
    # made by the caller's graph only, so the next direct call makes its own
    _run(stub, """
lat = handle(use_graphs=False)
lat.step(0)
assert records()[0] == 1
lat.set_stream_collide_launch(512, False, 0)   # marks to be made anew
control(capturing=1)
lat.step(2)
assert records()[0] == 2
control()
lat.step(2)
assert records()[0] == 3
lat.step(2)
assert records()[0] == 3
""")


def test_failed_capture_counts_the_steps_enqueued(stub):
    _run(stub, """
lat = handle()
control(fail_instantiate=1)
refused(lat.step, 700)
done = records()[1]
assert 0 < done < 700 and lat.time == done
control()
lat.step(700)
r = records()
assert lat.time == done + 700 == r[1] + r[2] and r[3] > 0
""")


def test_failed_replay_counts_the_steps_enqueued(stub):
    _run(stub, """
lat = handle()
lat.step(640)
control(fail_launch=2)
refused(lat.step, 320)
r = records()
assert lat.time == r[1] + r[2] < 960
""")


@pytest.mark.parametrize("swimmers", [True, False])
def test_graphs_across_changes_of_the_launches(stub, swimmers):
    _run(stub, f"""
if not {swimmers}:
    case = dict(case, swimmers=[])
lat = handle()
def run(first, calls):
    before = records()[3]
    for n in calls[:first]:
        lat.step(n)
    assert records()[3] == before       # launched directly
    for n in calls[first:]:
        lat.step(n)
    assert records()[3] > before        # replayed
calls = [1, 300, 211, 640, 33, 7]
run(3, calls)
lat.average_begin(3)
run(3, calls)
lat.set_stream_collide_launch(128, True, -1)
run(3, calls)
lat.average_begin(0)
lat.set_kernel_timing(True)
lat.step(40)
lat.set_kernel_timing(False)
run(3, calls)
lat.adjoint(1, checkpoint=1) if {swimmers} else None
lat.step(64)
assert lat.time == 4 * sum(calls) + 104 + ({swimmers} is True)
lat.close()
""")


@pytest.mark.parametrize("storage,scale", [(0, 1.0), (1, 2.0 ** 20), (2, 1.0), (3, 1.0)])
def test_populations_without_device_memory(stub, storage, scale):
    # the host converts: what is set comes back as the storage rounds it
    _run(stub, f"""
import numpy as np
lat = lbmib.Lattice((33, 24, 35), 0.9, storage={storage}, fp16_scale={scale})
g = 1e-3 * np.random.default_rng(0).standard_normal((19, 35, 24, 33))
lib.limit_malloc(1 << 10)
lat.set_populations(g)
got = lat.populations()
assert np.abs(got - g).max() < {2e-6 if storage == 1 else 1e-7} and got.any()
""")


def test_exchange_keeps_its_buffer(stub):
    # a free waits for the whole device: none, and no allocation, after the first call
    _run(stub, """
import numpy as np
lat = lbmib.Lattice((64, 40, 32), 0.9)
g = np.zeros((19, 32, 40, 64))
lat.set_populations(g)
before = allocations()
for _ in range(3):
    lat.set_populations(g)
    lat.populations()
assert allocations() == before
n = before[0] - before[1]
lat.close()
assert allocations()[1] - before[1] == n   # destroyed with the handle
""")


def test_two_stream_box(stub, tmp_path):
    # an FP32 box of more beads than the fused step takes: its buffers, graphs, launch
    # shapes, checkpoints and the adjoint's recompute on two streams
    _run(stub, f"""
sw = [wl.swimmer((16 + 33 * (i % 3), 2 + 12 * (i // 3), 3), 10.0, level=0, T=500.0) for i in range(13)]
case = dict(case, shape=(99, 63, 29), swimmers=sw)
for graphs in (True, False):
    lat = handle(use_graphs=graphs)
    lat.step(7)
    lat.step(70)
    for shape in ((128, True, 3), (512, False, 1), (256, False, -1), (256, True, 0)):
        lat.set_stream_collide_launch(*shape)
        lat.step(40)
    lat.average_begin(2)
    lat.step(33)
    lat.average_begin(0)
    for steps, checkpoint in ((1, 4), (40, 16), (90, 20)):
        lat.adjoint(steps, checkpoint=checkpoint, swimmer=12, rewind=steps == 40)
    lat.save({str(tmp_path / "ck.bin")!r})
    lat.step(3)
    lat.load({str(tmp_path / "ck.bin")!r})
    lat.step(3)
    lat.markers()
    lat.swimmer_centres()
    lat.close()
""")
