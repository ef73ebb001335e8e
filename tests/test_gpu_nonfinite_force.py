"""A force that is not finite (an actuation beyond the range of FP32) reaches the nodes
of its markers' stencils and no others, in one step of either schedule."""
import numpy as np
import pytest

from paper_2202_12147_amd import lbmib, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [2, 3, 4])
@pytest.mark.parametrize("storage", [lbmib.FP32_SHIFTED, lbmib.FP32_INPLACE, lbmib.FP16_SHIFTED])
def test_stays_within_the_stencils(storage, width):
    case = wl.small_case()
    sw = case["swimmers"][0]
    sw["A"] = sw["B"] = 1e42
    sw["phi0"] = 0.5
    case["width"] = width
    print("width", width, "storage", storage, flush=True)
    lat = lbmib.from_workload(case, storage=storage)
    m = lat.markers()  # where the forces of the step act
    lat.step(1)
    bad = ~np.isfinite(lat.velocity()).all(axis=0)  # [z, y, x]
    n = np.array(bad.shape[::-1])
    first = {2: np.floor(m), 3: np.floor(m + 0.5) - 1, 4: np.floor(m) - 1}[width].astype(int)
    reach = np.zeros(bad.shape, bool)
    k = np.arange(width)
    for f in first:
        x, y, z = ((f[a] + k) % n[a] for a in range(3))
        reach[np.ix_(z, y, x)] = True
    assert bad.any() and not (bad & ~reach).any()
