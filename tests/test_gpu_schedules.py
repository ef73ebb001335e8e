"""Batches on the two-stream schedule (more than 128 beads): the persistent bulk
launch, whose workgroups claim their blocks with FP32 storage, gives the bits of the
other launch shapes."""
import numpy as np
import pytest

from paper_2202_12147_amd import lbmib, workloads as wl

pytestmark = pytest.mark.gpu

SHAPES = [(512, False, 0), (512, False, 1), (512, True, 2), (256, False, 4), (256, True, 1), (128, True, 3),
          (128, False, 8), (256, False, -1)]


def _same(a, b, what):
    assert np.array_equal(a.markers(), b.markers()), what
    assert np.array_equal(a.marker_forces(), b.marker_forces()), what
    assert np.array_equal(a.populations(), b.populations()), what


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
