"""GPU tests of the tree walks past the range in which their FP32 bounds hold (squares
beyond the largest float): the direct scan's answers, never an index that is none."""
import numpy as np
import pytest

import ddsynth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

FP64, ANN, KMEANS = 0x1, 0x10, 0x20


@pytest.fixture(scope="module")
def L():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2012_00357_amd import _lib
    return _lib


@pytest.mark.parametrize("mode", ["ann", "kmeans"])
@pytest.mark.parametrize("scale,far", [(1.0, 1e19), (1.0, 1e42), (1.0, 1e200), (1e19, 1e19), (1e25, 1e25)])
def test_walks_past_single_precision(L, C0, mode, scale, far):
    import torch
    n, m = 5000, 200
    e, s = ddsynth.data_points(n, 8100)
    qe, qs, base = ddsynth.queries(e, s, m, 8101)
    C = C0 / np.abs(C0).max()                 # strains and stresses of one size
    s, qs = s / np.abs(C0).max(), qs / np.abs(C0).max()
    e, s = e * 1e3 * scale, s * 1e3 * scale
    y = ddsynth.states(qe * 1e3 * scale, qs * 1e3 * scale)
    y[5:9] *= far / scale
    y[9, :] = far
    ds = L.dd_dataset_create(to_dev(e), to_dev(s), C, packs=FP64 | ANN | KMEANS)
    y = to_dev(y)
    ref, dref = L.dd_project(ds, y, mode="direct")
    warm = to_dev(base)
    for w in (None, warm):
        for call in (lambda: L.dd_project(ds, y, warm_start_idx=w, mode=mode, stats=True)[:2],
                     lambda: L.dd_project_noalloc(ds, y, warm_start_idx=w, mode=mode)):
            idx, dist = call()
            torch.cuda.synchronize()
            assert torch.equal(idx, ref)
            assert np.array_equal(dist.cpu().numpy(), dref.cpu().numpy(), equal_nan=True)
    # approximate searches: a data point for every state
    for kw in (dict(ann_budget=4), *([dict(ann_fd=0.4)] if mode == "kmeans" else [])):
        idx, _ = L.dd_project(ds, y, mode=mode, **kw)
        assert int(idx.min()) >= 0 and int(idx.max()) < n
    ds.close()
