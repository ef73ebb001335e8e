"""Bead terms folded by a kernel of their own (more than 256 surface patches in a
box): every workgroup of the launch that spreads and records the forces reads the
same terms, so a run repeats bit for bit, with graphs and without."""
import numpy as np
import pytest

from paper_2202_12147_amd import lbmib, workloads as wl

pytestmark = pytest.mark.gpu


def _run(steps, graphs):
    sw = [wl.swimmer((48, y, 16), 16.0, radius=4.0, level=4, A=5e-4, T=2000.0, phi0=0.4 * i)
          for i, y in enumerate((14, 42))]
    case = dict(name="two level-4 swimmers", shape=(96, 56, 32), tau=0.8, forcing=wl.GUO, width=4, swimmers=sw)
    lat = lbmib.from_workload(case, use_graphs=graphs)
    lat.step(steps)
    return lat.velocity(), lat.markers(), lat.marker_forces()


def test_folded_terms_repeat():
    print("two level-4 swimmers, 486 patches", flush=True)
    a = _run(9, True)
    for graphs in (True, False):
        for x, y in zip(a, _run(9, graphs)):
            assert np.array_equal(x, y)
