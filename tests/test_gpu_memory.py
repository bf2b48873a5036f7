"""GPU test of the released memory that stays with the process for five seconds: it
goes by itself, also while the program has a stream capture open."""
import time

import pytest

import ddsynth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


def test_kept_memory_goes_during_a_capture(C0):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2012_00357_amd import _lib as L
    e, s = ddsynth.data_points(1_000_000, 61)
    e, s = to_dev(e), to_dev(s)
    x = torch.arange(1000.0, device="cuda")
    side = torch.cuda.Stream()
    L.dd_dataset_create(e, s, C0, packs=0x1 | 0x4).close()   # the runtime's own memory of the first kernels
    L._lib.dd_dataset_destroy(None)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    L.dd_dataset_create(e, s, C0, packs=0x1 | 0x4).close()
    kept = free0 - torch.cuda.mem_get_info()[0]
    assert kept > 100 << 20
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        y = x * 2.0
        time.sleep(6.5)
        y = y + 1.0
    assert free0 - torch.cuda.mem_get_info()[0] < kept // 4
    for k in range(3):
        x.add_(1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, x * 2.0 + 1.0)
