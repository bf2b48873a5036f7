"""GPU tests of the culled scans at the edges of their arithmetic and of their
runs and lists, against the direct scan and the scan of every tile."""
import numpy as np
import pytest

import ddsynth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

FP64, FP32, BF16, FP16, ANN, KMEANS = 0x1, 0x2, 0x4, 0x8, 0x10, 0x20
N0 = 1 << 18


@pytest.fixture(scope="module")
def L():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2012_00357_amd import _lib
    return _lib


@pytest.mark.parametrize("mode", ["fp64", "fp32", "bf16", "fp16"])
@pytest.mark.parametrize("flip", [False, True])
@pytest.mark.parametrize("far", [1e20, 1e42, 1e80, 1e160])
def test_states_beyond_single_precision(L, mode, flip, far):
    """A state whose coordinates exceed the FP32 range shares its group with states at
    the points of a last tile of 40 rows (the data lie on a line, so that one of its
    ends, by the sign of the axis, is that tile): its answer is the direct scan's."""
    import torch
    n = N0 + 40
    t = np.linspace(-1e-3, 1e-3, n)[:, None] * np.eye(6)[0]
    e = np.ascontiguousarray(t[::-1] if flip else t)
    s = np.zeros_like(e)
    ds = L.dd_dataset_create(to_dev(e), to_dev(s), np.eye(6), packs=FP64 | FP32 | BF16 | FP16)
    for end in (0, n - 1):
        y = np.repeat(ddsynth.states(e[end:end + 1], s[end:end + 1]), 16, 0)
        y[7] = 0.0
        y[7, 0] = far
        idx, dist = L.dd_project(ds, to_dev(y), mode=mode)
        ref, dref = L.dd_project(ds, to_dev(y), mode="direct")
        assert torch.equal(idx, ref)
        np.testing.assert_allclose(dist.cpu().numpy(), dref.cpu().numpy(), rtol=1e-14, atol=0)
    ds.close()
