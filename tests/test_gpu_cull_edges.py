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


@pytest.mark.parametrize("mode", ["fp64", "fp32", "bf16", "fp16"])
def test_overflowing_lists_end_early(L, mode):
    """States far to one side of the data, whose distances the 16-bit formats cannot tell
    apart, overflow every list: the direct scan's answers, and the scan takes no longer
    than a few of ordinary states (a hundred and more where every point is appended)."""
    import torch
    n, m = 1 << 19, 2048
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn(n, 12, dtype=torch.float64, device="cuda", generator=g)
    X[:, 6:] = X[:, :6] + 0.01 * X[:, 6:]
    X[17], X[n - 5] = X[123], X[123]
    ds = L.dd_dataset_create(X[:, :6].contiguous(), X[:, 6:].contiguous(), np.eye(6), packs=FP64 | FP32 | BF16 | FP16)
    pick = torch.randint(0, n, (m,), device="cuda", generator=g)
    near = (X[pick] + 0.05 * torch.randn(m, 12, dtype=torch.float64, device="cuda", generator=g)).contiguous()
    side = 0.3 * torch.randn(m, 12, dtype=torch.float64, device="cuda", generator=g)
    side[:, :6] += 10.0
    side[:, 6:] -= 10.0
    ms = {}
    for name, y in (("near", near), ("side", side)):
        for _ in range(2):
            idx, dist, st = L.dd_project(ds, y, mode=mode, stats=True)
        ms[name] = st["scan_ms"]
        ref, dref = L.dd_project(ds, y, mode="direct")
        assert torch.equal(idx, ref) and torch.equal(dist, dref)
        if mode == "bf16" and name == "side":
            assert st["overflowed"] == m
    print(mode, ms)
    assert ms["side"] < 40 * ms["near"]
    ds.close()


@pytest.mark.parametrize("mode", ["fp64", "fp32", "bf16", "fp16"])
@pytest.mark.parametrize("splits", [1, 7, 64])
def test_splits_ask_for_every_tile(L, C0, mode, splits):
    """A caller who gives the splits gets the scan of every tile, with the same answers."""
    import torch
    n, m = N0 + 513, 700
    e, s = ddsynth.data_points(n, 7600)
    qe, qs, _ = ddsynth.queries(e, s, m, 7601)
    ds = L.dd_dataset_create(to_dev(e), to_dev(s), C0, packs=FP64 | FP32 | BF16 | FP16)
    y = to_dev(ddsynth.states(qe, qs))
    idx, dist, st = L.dd_project(ds, y, mode=mode, splits=splits, stats=True)
    ref, dref, sr = L.dd_project(ds, y, mode=mode, stats=True)
    assert torch.equal(idx, ref) and torch.equal(dist, dref)
    assert st["visited"] == n * m and sr["visited"] < 0.7 * n * 32 * ((m + 31) // 32)
    ds.close()


def _law(L, n, seed, C0):
    """n points near a linear law on the GPU, and states around m of them."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    C = torch.from_numpy(np.ascontiguousarray(C0)).cuda()
    e = torch.empty(n, 6, dtype=torch.float64, device="cuda")
    s = torch.empty_like(e)
    for a in range(0, n, 1 << 23):
        b = min(n, a + (1 << 23))
        e[a:b] = 1e-3 * torch.randn(b - a, 6, dtype=torch.float64, device="cuda", generator=g)
        s[a:b] = e[a:b] @ C

    def states(m):
        pick = torch.randint(0, n, (m,), device="cuda", generator=g)
        y = torch.cat([e[pick], s[pick]], 1)
        return (y * (1.0 + 0.05 * torch.randn(m, 12, dtype=torch.float64, device="cuda", generator=g))).contiguous(), pick
    return e, s, states


def _equal(a, b):
    import torch
    assert torch.equal(a[0], b[0])
    assert np.array_equal(a[1].cpu().numpy(), b[1].cpu().numpy(), equal_nan=True)


@pytest.mark.parametrize("mode", ["fp64", "fp32", "bf16", "fp16"])
def test_batch_beyond_a_mask(L, C0, mode):
    """A batch of more states than the masks hold at once (65536), the last run of them
    33: the answers of the scan of every tile, from a fraction of its pairs."""
    n, m = 1 << 18, 65536 + 33
    e, s, states = _law(L, n, 81, C0)
    ds = L.dd_dataset_create(e, s, C0, packs=FP64 | FP32 | BF16 | FP16)
    y, _ = states(m)
    y[5, 2] = y[m - 1, 7] = float("nan")
    idx, dist, st = L.dd_project(ds, y, mode=mode, stats=True)
    _equal((idx, dist), L.dd_project(ds, y, mode=mode, splits=8))
    assert 0 < st["visited"] < 0.5 * n * m
    ds.close()


def test_run_shorter_than_a_mask(L, C0):
    """So many tiles that the masks hold 120 of the batch's 124 words of states at once,
    an odd number of tiles, a last run of four words."""
    n, m = (1 << 26) + (1 << 22) + 77, 120 * 512 + 3 * 512 + 9
    e, s, states = _law(L, n, 82, C0)
    ds = L.dd_dataset_create(e, s, C0, packs=FP64)
    y, pick = states(m)
    del e, s
    idx, dist, st = L.dd_project(ds, y, mode="fp64", stats=True)
    full = L.dd_project(ds, y, warm_start_idx=pick, mode="fp64", splits=8)
    _equal((idx, dist), full)
    assert 0 < st["visited"] < 0.1 * n * m
    ds.close()


@pytest.mark.parametrize("m", [1, 300, 16390])
def test_large_kmeans_walk_equals_fp64_scan(L, C0, m):
    """The k-means walk beyond the scans' sizes, begun with the seed bound or a warm start."""
    n = (1 << 24) + 4097
    e, s, states = _law(L, n, 83, C0)
    ds = L.dd_dataset_create(e, s, C0, packs=FP64 | KMEANS)
    y, pick = states(m)
    if m > 1:
        y[m // 2, 5] = float("nan")
    ref = L.dd_project(ds, y, mode="fp64")
    for warm in (None, pick):
        _equal(L.dd_project(ds, y, warm_start_idx=warm, mode="kmeans"), ref)
    ds.close()
