"""GPU tests of exact tree-mode projections answered by a 16-bit scan: at the
sizes where the rule changes between walk and scan, the scan's answers equal the
walk's (a call that asks for statistics walks) bit for bit: both certify every
point within the smallest distance and rerank by the same FP64 direct form."""
import numpy as np
import pytest

import ddsynth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

FP64, BF16, FP16, ANN, KMEANS = 0x1, 0x4, 0x8, 0x10, 0x20


@pytest.fixture(scope="module")
def L():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2012_00357_amd import _lib
    return _lib


@pytest.mark.parametrize("N,packs,sizes", [
    (8191, ANN, (4096,)), (8192, ANN, (4095, 4096)), (9001, KMEANS | BF16, (4097,)),
    (32767, ANN, (512,)), (32768, ANN | KMEANS, (511, 512, 5000)), (65536, ANN, (511,)),
    (65537, ANN | KMEANS, (1, 8, 513)), (262145, ANN | BF16, (33, 20000)), (600000, KMEANS, (2, 4097))])
def test_scan_equals_walk(L, C0, N, packs, sizes):
    import torch
    e, s = ddsynth.data_points(N, 7000 + N % 997)
    e[N // 2:N // 2 + 40] = e[:40]      # equal points: the smaller index is the answer
    s[N // 2:N // 2 + 40] = s[:40]
    ds = L.dd_dataset_create(to_dev(e), to_dev(s), C0, packs=FP64 | packs)
    for m in sizes:
        qe, qs, base = ddsynth.queries(e, s, m, 7100 + m)
        y = ddsynth.states(qe, qs)
        far = max(1, m // 5)
        y[:far] *= 3.0                  # far from the data
        y[-min(m, 40):] = ddsynth.states(e[:min(m, 40)], s[:min(m, 40)])   # at data points
        if m > 1:
            y[1, 3] = np.nan
        warm = base.copy()
        warm[::7] = -1
        warm[::11] = N                  # not a data point: ignored
        for mode, pack in (("ann", ANN), ("kmeans", KMEANS)):
            if not packs & pack:
                continue
            for w in (None, to_dev(warm)):
                got, dist = L.dd_project(ds, to_dev(y), warm_start_idx=w, mode=mode)
                ref, dref, _ = L.dd_project(ds, to_dev(y), warm_start_idx=w, mode=mode, stats=True)
                assert torch.equal(got, ref), f"m {m} {mode}"
                assert np.array_equal(dist.cpu().numpy(), dref.cpu().numpy(), equal_nan=True)
    if not packs & (BF16 | FP16):       # the pack kept for this opens no mode
        with pytest.raises(L.DDError) as ex:
            L.dd_project(ds, to_dev(y), mode="fp16")
        assert ex.value.status == 8
    ds.close()


@pytest.mark.parametrize("m", [1, 9, 16383, 16384, 16391])
def test_large_walk_equals_fp64_scan(L, C0, m):
    """Beyond the scans' sizes the walk begins, without a warm start, with the seed
    bound: the FP64 scan's answers, bit for bit."""
    import torch
    N = (1 << 24) + 4097
    g = torch.Generator(device="cuda").manual_seed(77)
    C = torch.from_numpy(np.ascontiguousarray(C0)).cuda()
    e = 1e-3 * torch.randn(N, 6, dtype=torch.float64, device="cuda", generator=g)
    s = e @ C
    ds = L.dd_dataset_create(e, s, C0, packs=FP64 | ANN)
    pick = torch.randint(0, N, (m,), device="cuda", generator=g)
    y = torch.cat([e[pick], s[pick]], 1)
    y = (y * (1.0 + 0.2 * torch.randn(m, 12, dtype=torch.float64, device="cuda", generator=g))).contiguous()
    if m > 1:
        y[m // 2, 5] = float("nan")
    ref, dref = L.dd_project(ds, y, mode="fp64")
    for warm in (None, pick):
        got, dist = L.dd_project(ds, y, warm_start_idx=warm, mode="ann")
        assert torch.equal(got, ref)
        assert np.array_equal(dist.cpu().numpy(), dref.cpu().numpy(), equal_nan=True)
    ds.close()
