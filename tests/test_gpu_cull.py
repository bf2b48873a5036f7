"""GPU tests of the culled scans (the tiles beyond every query's bound left out)
at the sizes where they start (2^18 data points) and at the edges of their
tiles, query groups and mask words, against the CPU oracle.  Distances are held
to the parity tests' bar: the oracle evaluates the raw metric, the library the
whitened direct form, both exact up to FP64 rounding (about 1e-15 relative, so
1e-12)."""
import sys

import numpy as np
import pytest

import ddsynth
import oracle
from gpu_util import compare_to_oracle, to_dev

pytestmark = pytest.mark.gpu

SCANS = ["fp64", "fp32", "bf16", "fp16"]
PACKS = 0x1 | 0x2 | 0x4 | 0x8
N0 = 1 << 18


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def L():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2012_00357_amd import _lib
    return _lib


@pytest.fixture(scope="module")
def data(L, C0):
    """Data sets of whole and partial last tiles and chunks, shared by the tests."""
    out = {}
    for n, tile in ((N0, 2048), (N0 + 1, 2048), (N0 + 255, 128), (N0 + 64 * 256 + 257, 512)):
        e, s = ddsynth.data_points(n, 7000 + n % 977)
        out[n] = (e, s, L.dd_dataset_create(to_dev(e), to_dev(s), C0, packs=PACKS, tile=tile))
    return out


@pytest.mark.parametrize("mode", SCANS)
@pytest.mark.parametrize("m", [1, 15, 17, 33, 64, 65, 513, 1030])
def test_edges_of_groups_and_tiles(L, C0, data, mode, m):
    """Batches at the edges of a query group (16 or 32), a wavefront (64) and a
    mask word (512 or 1024 queries); fewer pairs than all are evaluated."""
    for n, (e, s, ds) in data.items():
        if m > 100 and n != N0 + 1:
            continue
        _say("cull", mode, n, m)
        qe, qs, base = ddsynth.queries(e, s, m, 7100 + m)
        oi, od, o2 = oracle.pd_raw(e, s, C0, qe, qs)
        states = to_dev(ddsynth.states(qe, qs))
        idx, dist, st = L.dd_project(ds, states, mode=mode, stats=True)
        compare_to_oracle(idx.cpu().numpy(), dist.cpu().numpy(), oi, od, o2)
        assert 0 < st["visited"] < n * ((m + 31) // 32 * 32)


@pytest.mark.parametrize("mode", SCANS)
def test_unusual_queries(L, C0, data, mode):
    """Queries on data points of the first and the last (partial) tile, non-finite
    ones, ones far outside the data (1e4 and 1e9 times its extent, past the reach
    of the 16-bit formats and of FP32 squares), and 200 equal ones (all in one
    cell of the grouping): as the oracle; a warm start far off or out of range
    changes nothing."""
    import torch
    n = N0 + 64 * 256 + 257
    e, s, ds = data[n]
    rng = np.random.default_rng(3)
    picks = np.concatenate([np.arange(3), np.arange(n - 3, n), rng.integers(0, n, 20)])
    qe, qs, _ = ddsynth.queries(e, s, 40, 7301)
    one = np.repeat(qe[:1], 200, 0), np.repeat(qs[:1], 200, 0)
    q_e = np.concatenate([e[picks], qe, qe[:6] * 1e4, qe[:4] * 1e9, qe[:1] * 1e25, one[0]])
    q_s = np.concatenate([s[picks], qs, qs[:6] * 1e4, qs[:4] * 1e9, qs[:1] * 1e25, one[1]])
    oi, od, o2 = oracle.pd_raw(e, s, C0, q_e, q_s)
    states = ddsynth.states(q_e, q_s)
    bad = np.array([[np.nan] + [0.0] * 11, [0.0] * 11 + [np.inf]])
    _say("unusual", mode)
    q = to_dev(np.concatenate([bad[:1], states, bad[1:]]))
    idx, dist, st = L.dd_project(ds, q, mode=mode, stats=True)
    i, d = idx.cpu().numpy(), dist.cpu().numpy()
    assert i[0] == -1 and i[-1] == -1 and np.isnan(d[0]) and np.isnan(d[-1])
    compare_to_oracle(i[1:-1], d[1:-1], oi, od, o2)
    assert np.all(d[1:1 + len(picks)] == 0.0)
    # (a warm start of 2^18 points needs a large batch to be culled: the batch repeated)
    reps = (1 << 32) // n // len(i) + 1 if mode in ("bf16", "fp16") else 3
    big = q.repeat(reps, 1).contiguous()
    warm = to_dev(rng.integers(-5, n + 5, big.shape[0]).astype(np.int64))
    iw, dw, sw = L.dd_project(ds, big, warm_start_idx=warm, mode=mode, stats=True)
    assert sw["visited"] < n * big.shape[0]
    assert torch.equal(iw, idx.repeat(reps))
    np.testing.assert_allclose(dw.cpu().numpy(), np.tile(d, reps), rtol=1e-14, atol=0)


@pytest.mark.parametrize("mode", SCANS)
def test_duplicates_and_a_line(L, C0, mode):
    """More copies of a point than a candidate list holds (the fallback answers,
    lowest index first), and data that differ in one strain component only."""
    n = N0 + 100
    e, s = ddsynth.data_points(n, 7401)
    dup = np.arange(5000, 5100)
    e[dup], s[dup] = e[77], s[77]
    ds = L.dd_dataset_create(to_dev(e), to_dev(s), C0, packs=PACKS)
    picks = np.array([77, 5050, 0, n - 1])
    idx, dist = L.dd_project(ds, to_dev(ddsynth.states(e[picks], s[picks])), mode=mode)
    assert idx.cpu().tolist() == [77, 77, 0, n - 1] and np.all(dist.cpu().numpy() == 0.0)
    ds.close()
    e = np.repeat(e[:1], n, 0) + np.linspace(-1e-3, 1e-3, n)[:, None] * np.eye(6)[0]
    s = np.repeat(s[:1], n, 0)
    qe, qs, _ = ddsynth.queries(e, s, 60, 7402)
    oi, od, o2 = oracle.pd_raw(e, s, C0, qe, qs)
    ds = L.dd_dataset_create(to_dev(e), to_dev(s), C0, packs=PACKS)
    idx, dist = L.dd_project(ds, to_dev(ddsynth.states(qe, qs)), mode=mode)
    compare_to_oracle(idx.cpu().numpy(), dist.cpu().numpy(), oi, od, o2)
    ds.close()
