"""GPU tests of the released memory that stays with the process: used again with
right answers (several threads and streams, stale contents), bounded, and given up
by dd_dataset_destroy(NULL)."""
import threading

import numpy as np
import pytest

import ddsynth
import oracle
from gpu_util import compare_to_oracle, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2012_00357_amd import _lib
    return _lib


def test_released_memory_is_given_up(L, C0):
    import torch
    e, s = ddsynth.data_points(200_000, 61)
    e, s = to_dev(e), to_dev(s)
    L.dd_dataset_create(e, s, C0, packs=0x3F).close()   # the runtime's own memory of the first kernels
    L._lib.dd_dataset_destroy(None)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for _ in range(3):
        ds = L.dd_dataset_create(e, s, C0, packs=0x3F)
        held = free0 - torch.cuda.mem_get_info()[0]
        ds.close()
        assert free0 - torch.cuda.mem_get_info()[0] <= held + (8 << 20)   # nothing piles up
    L._lib.dd_dataset_destroy(None)
    assert free0 - torch.cuda.mem_get_info()[0] < held // 4


@pytest.mark.parametrize("sizes", [(40_000, 40_000, 43_000), (1_000, 70_000, 65_000)])
def test_reuse_by_threads(L, C0, sizes):
    import torch
    work = []
    for i, n in enumerate(sizes):
        e, s = ddsynth.data_points(n, 500 + i)
        qe, qs, _ = ddsynth.queries(e, s, 300, 600 + i)
        work.append((to_dev(e), to_dev(s), to_dev(ddsynth.states(qe, qs)), oracle.pd_raw(e, s, C0, qe, qs)))
    errors = []

    def run(k):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for r in range(4):
                    e, s, y, (oi, od, o2) = work[(k + r) % len(work)]
                    ds = L.dd_dataset_create(e, s, C0, packs=0x1 | 0x4 | 0x10 | 0x20, stream=stream)
                    for mode in ("fp64", "bf16", "ann", "kmeans"):
                        idx, dist = L.dd_project(ds, y, mode=mode, stream=stream)
                        stream.synchronize()
                        compare_to_oracle(idx.cpu().numpy(), dist.cpu().numpy(), oi, od, o2)
                    ds.close()
        except Exception as ex:   # reported below
            errors.append(repr(ex))

    torch.cuda.synchronize()
    threads = [threading.Thread(target=run, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
