"""The marker adjoints (per-bead sums, force tangents) over the mesh sizes at
which their workgroups fill differently: 12 nodes and 20 triangles per bead
(less than one wavefront; an odd number of node groups per workgroup) and 642
nodes and 1280 triangles (more triangles than the per-bead workgroup has
lanes).  Bar as for the other short horizons: the FP32 rounding of the grid
adjoint over tens of steps, 2e-5 of each component."""
import math

import numpy as np
import pytest

from oracle import adjoint as oracle_adjoint
from paper_2202_12147_amd import lbmib, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("level", [0, 3])
def test_mesh_sizes_match_oracle(level):
    case = workloads.adjoint_case(reduced=True)
    case["swimmers"] = [workloads.swimmer((12.0, 12.0, 12.0), 7.0, level=level, A=1e-3, T=2000.0, alpha=math.pi / 3)]
    print("level", level, flush=True)
    J, g = lbmib.from_workload(case).adjoint(24, checkpoint=10)
    Jo, go = oracle_adjoint.displacement_gradient(case, 24, checkpoint_every=0)
    assert abs(J - Jo) <= 2e-5 * abs(Jo)
    assert np.all(np.abs(g - go) <= 2e-5 * np.abs(go)), (g, go)
