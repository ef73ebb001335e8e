"""FP32 handles at the edges of the rule between the fused step and the two-stream
schedule (36 beads or 256 surface patches in a box; 128 beads in a batch, 64 beyond 1
GiB of populations, 30 where a box holds more than 512 markers), and what the two-stream
schedule has for them alone: the persistent bulk launch that claims its blocks, and the
recompute of the adjoint.

Bars as everywhere for the coupled step: velocity rel-L2 1e-5 and element-wise
1e-5 of max |u| (FP32 sums), markers 1e-10 lattice units per step; the adjoint's
short horizons 2e-5 of each component."""
import math

import numpy as np
import pytest

from helpers import max_rel, oracle_from, rel_l2
from oracle import adjoint as oracle_adjoint
from paper_2202_12147_amd import lbmib, workloads as wl

pytestmark = pytest.mark.gpu

SHAPES = [(512, False, 0), (512, False, 1), (512, True, 2), (256, False, 4), (256, True, 1), (128, True, 3),
          (128, False, 8), (256, False, -1)]


def _box(count, level, width=3, rows=3):
    """`count` swimmers in a ragged box, `rows` along x and the rows 12 apart."""
    lines = -(-count // rows)
    sw = [wl.swimmer((16 + 33 * (i % rows), 2 + 12 * (i // rows), 3), 10.0, level=level, T=500.0, phi0=0.3 * i)
          for i in range(count)]
    return dict(name=f"{count} swimmers, level {level}", shape=(33 * rows, max(29, 12 * lines + 3), 29), tau=1.0,
                forcing=wl.GUO, width=width, swimmers=sw)


@pytest.mark.parametrize("count,level", [(4, 3), (5, 3), (2, 4), (12, 1), (13, 1), (22, 0)])
@pytest.mark.parametrize("storage", [lbmib.FP32_SHIFTED, lbmib.FP32_INPLACE])
def test_edges_match_oracle(count, level, storage):
    # 252 | 315 and 486 patches; 36 | 39 and 66 beads
    case = _box(count, level)
    print(case["name"], case["shape"], "storage", storage, flush=True)
    lat, o = lbmib.from_workload(case, storage=storage), oracle_from(case)
    lat.step(2)
    lat.step(4)
    o.step(6)
    u, ref = lat.velocity(), o.velocity()
    assert rel_l2(u, ref) < 1e-5 and max_rel(u, ref) < 1e-5
    assert np.abs(lat.markers() - o.markers()).max() < 1e-10 * 6


@pytest.mark.parametrize("storage,shape", [(lbmib.FP32_SHIFTED, (200, 197, 181)), (lbmib.FP32_INPLACE, (243, 241, 244))])
def test_populations_beyond_the_write_through_bound(storage, shape):
    # more than 1 GiB of populations (other loads and stores), each set below 4 GiB
    case = dict(wl.small_case(), shape=shape, swimmers=[wl.swimmer((6, 2, 90), 10.0, T=500.0)])
    print(shape, "storage", storage, flush=True)
    lat, o = lbmib.from_workload(case, storage=storage), oracle_from(case)
    lat.step(3)
    o.step(3)
    u, ref = lat.velocity(), o.velocity()
    assert rel_l2(u, ref) < 1e-5 and max_rel(u, ref) < 1e-5
    assert np.abs(lat.markers() - o.markers()).max() < 1e-10 * 3


def _same(a, b, what):
    assert np.array_equal(a.markers(), b.markers()), what
    assert np.array_equal(a.marker_forces(), b.marker_forces()), what
    assert np.array_equal(a.populations(), b.populations()), what


@pytest.mark.parametrize("storage", [lbmib.FP32_SHIFTED, lbmib.FP32_INPLACE])
def test_launch_shapes_of_a_two_stream_box(storage):
    case = _box(22, 0)
    ref = lbmib.from_workload(case, storage=storage)
    ref.step(41)
    for shape in SHAPES:
        for graphs in (True, False):
            print("shape", shape, "graphs", graphs, flush=True)
            lat = lbmib.from_workload(case, storage=storage, use_graphs=graphs)
            lat.set_stream_collide_launch(*shape)
            lat.step(9)
            lat.step(32)
            _same(lat, ref, (shape, graphs))


@pytest.mark.parametrize("storage", [lbmib.FP32_SHIFTED, lbmib.FP32_INPLACE, lbmib.FP32_PLAIN])
def test_averages_and_restarts_of_a_two_stream_box(storage, tmp_path):
    case = _box(22, 0)
    ref = lbmib.from_workload(case, storage=storage, use_graphs=False)
    ref.average_begin(3)
    ref.step(45)
    mean, samples = ref.average_velocity()
    path = str(tmp_path / "ck.bin")
    for shape in ((512, False, 0), (512, False, 1), (256, True, 2), (256, False, -1)):
        print("shape", shape, flush=True)
        lat = lbmib.from_workload(case, storage=storage)
        lat.set_stream_collide_launch(*shape)
        lat.average_begin(3)
        lat.step(13)
        lat.step(32)
        got, n = lat.average_velocity()
        assert n == samples and np.array_equal(got, mean), shape
        _same(lat, ref, shape)
        lat.save(path)
        lat.step(7)
        other = lbmib.from_workload(case, storage=storage)
        other.load(path)
        other.step(7)
        _same(lat, other, shape)


def test_launch_shapes_of_a_large_batch():
    ens = wl.ensemble(seed=7, nboxes=43)
    for i, b in enumerate(ens["boxes"]):
        b["shape"] = (33 + i % 7, 32 + i % 3, 40 - i % 5)
        mid = np.array([s // 2 for s in b["shape"]], float)
        sw = b["swimmers"][0]
        sw["centres"] = np.stack([mid - (10.0, 0, 0), mid, mid + (10.0, 0, 0)])
        sw["L0"] = np.array([10.0, 10.0])
    ref = lbmib.batch_from_ensemble(ens)
    ref.step(41)
    for shape in SHAPES:
        print("shape", shape, flush=True)
        lat = lbmib.batch_from_ensemble(ens)
        lat.set_stream_collide_launch(*shape)
        lat.step(9)
        lat.step(32)
        _same(lat, ref, shape)


@pytest.mark.parametrize("boxes,bitwise", [(5, True), (6, False)])
def test_batch_of_boxes_with_many_markers(boxes, bitwise):
    # two swimmers of 162-node beads per box: 972 markers; 30 | 36 beads.  On the
    # fused step a box gives the bits it gives alone
    cases = []
    for i in range(boxes):
        c = _box(2, 2, rows=1)
        cases.append(dict(c, shape=(34 + i, 30, 31), tau=1.0 - 0.02 * i))
    print("boxes", boxes, flush=True)
    batch = lbmib.batch_from_ensemble(dict(boxes=cases))
    batch.step(12)
    m = batch.markers().reshape(boxes, -1, 3)
    for i in (0, boxes - 1):
        one = lbmib.batch_from_ensemble(dict(boxes=cases[i:i + 1]))
        one.step(12)
        if bitwise:
            assert np.array_equal(batch.velocity(i), one.velocity(0))
            assert np.array_equal(m[i], one.markers())
        else:
            assert rel_l2(batch.velocity(i), one.velocity(0)) < 1e-5
            assert np.abs(m[i] - one.markers()).max() < 1e-10 * 12


@pytest.mark.parametrize("boxes,bitwise", [(21, True), (22, False)])
def test_batch_beyond_the_write_through_bound(boxes, bitwise):
    # more than 1 GiB of populations; 63 | 66 beads
    ens = wl.ensemble(seed=3, nboxes=boxes)
    for i, b in enumerate(ens["boxes"]):
        b["shape"] = (72 - i % 3, 71 + i % 2, 70)
        mid = np.array([s // 2 for s in b["shape"]], float)
        b["swimmers"][0]["centres"] = np.stack([mid - (10.0, 0, 0), mid, mid + (10.0, 0, 0)])
        b["swimmers"][0]["L0"] = np.array([10.0, 10.0])
    assert 2 * 19 * 4 * sum(int(np.prod(b["shape"])) for b in ens["boxes"]) > 1 << 30
    print("boxes", boxes, flush=True)
    batch = lbmib.batch_from_ensemble(ens)
    batch.step(6)
    m = batch.markers().reshape(boxes, -1, 3)
    for i in (0, boxes - 1):
        one = lbmib.batch_from_ensemble(dict(ens, boxes=ens["boxes"][i:i + 1]))
        one.step(6)
        if bitwise:
            assert np.array_equal(batch.velocity(i), one.velocity(0))
            assert np.array_equal(m[i], one.markers())
        else:
            assert rel_l2(batch.velocity(i), one.velocity(0)) < 1e-5
            assert np.abs(m[i] - one.markers()).max() < 1e-10 * 6


def test_adjoint_on_the_two_stream_schedule():
    case = wl.adjoint_case(reduced=True)
    case["swimmers"] = [wl.swimmer((12.0, 12.0, 12.0), 7.0, level=5, A=1e-3, T=2000.0, alpha=math.pi / 3)]
    print("level 5", flush=True)
    got = [lbmib.from_workload(case, use_graphs=g).adjoint(20, checkpoint=8) for g in (True, False)]
    assert got[0][0] == got[1][0] and np.array_equal(got[0][1], got[1][1])
    J, g = got[0]
    Jo, go = oracle_adjoint.displacement_gradient(case, 20, checkpoint_every=0)
    print(J, Jo, g, go, flush=True)
    assert abs(J - Jo) <= 2e-5 * abs(Jo)
    assert np.all(np.abs(g - go) <= 2e-5 * np.abs(go)), (g, go)
    # the segments' recompute repeats the forward run: one segment gives the same bits
    J1, g1 = lbmib.from_workload(case).adjoint(20, checkpoint=20)
    assert J1 == J and np.array_equal(g1, g)
