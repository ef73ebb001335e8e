"""GPU parity of the fused step's less travelled branches against the FP64
oracle: bead terms folded by a kernel of their own (a box of more than 64 beads,
a mesh of more surface patches than a spreading workgroup folds), beads beyond
the first 64 of a box, markers over several chunks, tiles covered by several
beads across ragged seams; and the two-stream schedule of large batches against
the fused step of their boxes.

Bars as everywhere for the coupled step: velocity rel-L2 1e-5 and element-wise
1e-5 of max |u| (FP32 sums), markers 1e-10 lattice units per step."""
import numpy as np
import pytest

from helpers import max_rel, oracle_from, rel_l2
from paper_2202_12147_amd import lbmib, workloads as wl

pytestmark = pytest.mark.gpu


def _check(case, steps):
    print("case", case["name"], case["shape"], flush=True)
    lat, o = lbmib.from_workload(case), oracle_from(case)
    lat.step(1)
    lat.step(steps - 1)
    o.step(steps)
    u, ref = lat.velocity(), o.velocity()
    assert rel_l2(u, ref) < 1e-5 and max_rel(u, ref) < 1e-5
    assert np.abs(lat.markers() - o.markers()).max() < 1e-10 * steps


def _many(count, level):
    """`count` swimmers in a ragged box, three along x and rows 12 apart."""
    rows = -(-count // 3)
    shape = (99, max(29, 12 * rows + 3), 29)
    sw = [wl.swimmer((16 + 33 * (i % 3), 2 + 12 * (i // 3), 3), 10.0, level=level, T=500.0, phi0=0.3 * i)
          for i in range(count)]
    return dict(name=f"{count} swimmers, level {level}", shape=shape, tau=1.0, forcing=wl.GUO, width=3, swimmers=sw)


@pytest.mark.parametrize("count,level", [(1, 0), (4, 2), (21, 1), (22, 1)])
def test_many_swimmers_in_one_box(count, level):
    # 22 swimmers have 66 beads: beads 64 and 65 are outside the cover masks
    _check(_many(count, level), 6)


@pytest.mark.parametrize("width", [2, 3, 4])
def test_fine_meshes(width):
    # level 4: 243 patches and 7686 markers (the last folded in the spreading
    # workgroups); level 5: 963 patches
    for level in ((4, 5) if width == 4 else (4,)):
        case = dict(name=f"level {level}, width {width}", shape=(61, 30, 37), tau=0.8, forcing=wl.SHAN_CHEN, width=width,
                    swimmers=[wl.swimmer((30, 1, 36), 16.0, radius=4.0, level=level, A=5e-4, T=2000.0)])
        _check(case, 4)


def test_large_batch_matches_fused_boxes():
    # 22 boxes (66 beads) share a bounded number of spreading workgroups
    ens = wl.ensemble(seed=11, nboxes=22)
    for b in ens["boxes"]:
        b["shape"] = tuple(max(33, s // 2 + 1) for s in b["shape"])
        sw = b["swimmers"][0]
        mid = np.array([s // 2 for s in b["shape"]], float)
        sp = 10.0
        sw["centres"] = np.stack([mid - (sp, 0, 0), mid, mid + (sp, 0, 0)])
        sw["L0"] = np.array([sp, sp])
    batch = lbmib.batch_from_ensemble(ens)
    batch.step(40)
    m = batch.markers().reshape(22, -1, 3)
    for i in (0, 13, 21):
        one = lbmib.batch_from_ensemble(dict(ens, boxes=ens["boxes"][i:i + 1]))
        one.step(40)
        assert rel_l2(batch.velocity(i), one.velocity(0)) < 1e-5
        assert np.abs(m[i] - one.markers()).max() < 1e-10 * 40
