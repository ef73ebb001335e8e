"""On one stream the first 512 steps after a change of the launches are launched
directly and later full chunks of 32 are replayed from a captured graph: runs that
cross the line, in calls of any size, give the bits of direct launches; so do runs
that cross it again after the launches changed (a time average begun, another launch
shape, a restored checkpoint), with the caller's own work between the replays."""
import numpy as np
import pytest

from paper_2202_12147_amd import lbmib, workloads as wl

pytestmark = pytest.mark.gpu


def _same(a, b):
    assert a.time == b.time
    assert np.array_equal(a.markers(), b.markers())
    assert np.array_equal(a.marker_forces(), b.marker_forces())
    assert np.array_equal(a.velocity(), b.velocity())
    assert np.array_equal(a.populations(), b.populations())


def _steps(lat, calls):
    for n in calls:
        lat.step(n)
        lat.bead_centres()


@pytest.mark.parametrize("storage", [lbmib.FP32_SHIFTED, lbmib.FP32_INPLACE])
def test_replayed_steps_equal_direct_ones(storage, tmp_path):
    import torch
    case = wl.small_case()
    case["swimmers"][0]["A"] = 5e-4
    a = lbmib.from_workload(case, storage=storage)
    b = lbmib.from_workload(case, storage=storage, use_graphs=False)
    print("first crossing", flush=True)
    _steps(a, [1, 511, 33, 64, 7, 32])  # 512 direct, then chunks beside odd rests
    _steps(b, [324, 324])
    _same(a, b)
    print("with an average", flush=True)
    for lat, calls in ((a, [300, 215, 97, 32, 1]), (b, [45, 600])):
        lat.average_begin(7)
        _steps(lat, calls)
    _same(a, b)
    (ua, na), (ub, nb) = a.average_velocity(), b.average_velocity()
    assert na == nb and np.array_equal(ua, ub)
    print("serial order", flush=True)
    for lat, calls in ((a, [512, 64, 5]), (b, [581])):
        lat.average_begin(0)
        lat.set_stream_collide_launch(256, False, -1)
        _steps(lat, calls)
    _same(a, b)
    print("restored", flush=True)
    path = str(tmp_path / "ck.bin")
    a.set_stream_collide_launch(512, False, 0)
    a.step(640)
    a.save(path)
    x = torch.ones(1 << 20, device="cuda")
    for _ in range(3):  # replays with other work between them
        a.load(path)
        a.step(96)
        x = x * 1.5 + torch.ones_like(x)
    torch.cuda.synchronize()
    b.set_stream_collide_launch(512, False, 0)
    b.step(736)
    _same(a, b)


def test_one_call_across_the_line():
    case = wl.small_case()
    a, b = lbmib.from_workload(case), lbmib.from_workload(case)
    a.step(700)
    _steps(b, [100] * 7)
    _same(a, b)


def test_plain_fluid_across_the_line():
    a, b = lbmib.Lattice((33, 18, 21), 0.8), lbmib.Lattice((33, 18, 21), 0.8, use_graphs=False)
    g = wl.random_deviation((33, 18, 21), 3, 1e-4)
    for lat in (a, b):
        lat.set_populations(g)
    _steps(a, [500, 80, 31, 64])
    _steps(b, [675])
    assert np.array_equal(a.populations(), b.populations())
    assert np.array_equal(a.velocity(), b.velocity())
