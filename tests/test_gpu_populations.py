"""The exchange of populations with the host: what is set comes back, rounded
once by the storage type, for boxes of more values than one exchange buffer
holds (2^23) and for batches whose boxes share a buffer."""
import numpy as np
import pytest

from paper_2202_12147_amd import lbmib, workloads as wl

pytestmark = pytest.mark.gpu

W = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12, np.float32)


def _stored(g, storage, scale):
    """g as the storage type holds it (FP64 of the rounded value)."""
    if storage == lbmib.FP16_SHIFTED:
        return (g.astype(np.float32) * np.float32(scale)).astype(np.float16).astype(np.float64) / scale
    if storage == lbmib.FP32_PLAIN:
        w = W.astype(np.float64).reshape(19, *[1] * (g.ndim - 1))
        return (w + g).astype(np.float32).astype(np.float64) - w
    return g.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("storage", [lbmib.FP32_SHIFTED, lbmib.FP16_SHIFTED, lbmib.FP32_PLAIN, lbmib.FP32_INPLACE])
@pytest.mark.parametrize("shape", [(16, 17, 19), (77, 79, 75)])
def test_round_trip(shape, storage):
    scale = 2.0 ** 20 if storage == lbmib.FP16_SHIFTED else 1.0
    g = 1e-3 * np.random.default_rng(5).standard_normal((19,) + shape[::-1])
    lat = lbmib.Lattice(shape, 0.9, storage=storage, fp16_scale=scale)
    lat.set_populations(g)
    assert np.array_equal(lat.populations(), _stored(g, storage, scale))


@pytest.mark.parametrize("storage", [lbmib.FP32_SHIFTED, lbmib.FP32_INPLACE])
def test_batch_boxes(storage):
    shapes = [(16, 18, 17), (81, 80, 79), (19, 16, 33)]
    boxes = [(s, 0.9, wl.GUO) for s in shapes]
    parts = [1e-3 * np.random.default_rng(i).standard_normal((19,) + s[::-1]) for i, s in enumerate(shapes)]
    b = lbmib.Batch(boxes, storage)
    g = np.concatenate([p.ravel() for p in parts])
    b._check(b.lib.lbm_set_populations(b.h, lbmib._ptr(g)))
    assert np.array_equal(b.populations(), g.astype(np.float32).astype(np.float64))
    for steps in (1, 2):  # both arrangements of the in-place set
        b.step(1)
        got = b.populations()
        at = 0
        for i, s in enumerate(shapes):
            one = lbmib.Lattice(s, 0.9, storage=storage)
            one.set_populations(parts[i])
            one.step(steps)
            n = parts[i].size
            assert np.array_equal(got[at:at + n], one.populations().ravel())
            at += n
