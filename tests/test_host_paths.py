"""CPU tests of the library's host code on a HIP runtime without a device (fake_hip.c):
memory order and limits, scratch sizes, alignment, the server's accounting."""
import os
import textwrap

import pytest

from host_paths import LIB, run_scenario

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libdd.so not built")


def scenario(tmp_path, text):
    return run_scenario(tmp_path, textwrap.dedent(text))


def test_mask_rows_are_aligned(tmp_path):
    """The 16-byte reads of mask rows: odd numbers of tiles, runs of an odd number of
    mask words, last runs of a multiple of four words."""
    out = scenario(tmp_path, """
        rc, ds = create(dd, 400001 * 256, FP64)
        assert rc == 0, dd.dd_last_error()
        hip.fake_watch(b"plan_kernel", 2, (ctypes.c_int * 2)(8, 4))
        assert project(dd, ds, 83 * 512 + 4 * 512, "fp64") == 0, dd.dd_last_error()
        n = hip.fake_launches(b"plan_kernel")
        rows = [(hip.fake_arg(b"plan_kernel", i, 0), hip.fake_arg(b"plan_kernel", i, 1)) for i in range(n)]
        print(rows)
        assert n == 4 and {w for _, w in rows} != {rows[0][1]}      # two runs of different widths
        assert all(p % 16 == 0 for p, w in rows if w % 4 == 0)
        """)
    assert out


@pytest.mark.parametrize("packs", ["FP64 | ANN | BF16", "FP64 | FP32", "FP64 | KMEANS | FP16"])
def test_idle_memory_fails_no_allocation(tmp_path, packs):
    """What the library holds without using it (idle temporaries of a creation, blocks of
    destroyed objects) is given up before an allocation fails, of any size: what can be
    created in some memory can be created in more, and after a destroyed data set too."""
    scenario(tmp_path, f"""
        n, ok = 1 << 18, []
        base = hip.fake_live()
        for mb in range(20, 140, 1):
            hip.fake_limit(base + (mb << 20))
            rc, ds = create(dd, n, {packs})
            assert rc in (0, 3)
            ok.append(rc == 0)
            if rc == 0:
                dd.dd_dataset_destroy(ds)
            dd.dd_dataset_destroy(None)
        print(ok)
        assert not ok[0] and all(ok[ok.index(True):]), "created in less memory than this"
        hip.fake_limit(base + (400 << 20))
        rc, ds = create(dd, n, {packs})
        dd.dd_dataset_destroy(ds)
        assert hip.fake_live() > base                 # kept blocks
        hip.fake_limit(hip.fake_live())               # and not a byte beside them
        rc, ds = create(dd, 100, FP64)                # small buffers only
        assert rc == 0, dd.dd_last_error()
        rc = project(dd, ds, 5000, "fp64")            # stream-ordered scratch
        assert rc == 0, dd.dd_last_error()
        """)


@pytest.mark.parametrize("packs", ["ANN", "KMEANS", "ANN | KMEANS"])
def test_unrequested_pack_takes_what_is_left(tmp_path, packs):
    """The 16-bit pack that a tree's exact searches use fails no creation: what can be
    created in some memory can be created in more.  Where it finds no room it leaves
    nothing behind, and the searches walk."""
    scenario(tmp_path, f"""
        n, sizes = 1 << 20, []
        base = hip.fake_live()
        for mb in range(90, 400, 3):
            hip.fake_limit(base + (mb << 20))
            rc, ds = create(dd, n, FP64 | {packs})
            assert rc in (0, 3)
            sizes.append(held(dd, ds) if rc == 0 else 0)
            if rc == 0:
                dd.dd_project(ds, vp(4096), 600, None, ctypes.byref(ProjectOpts(MODE["{packs.split()[0].lower()}"])), vp(4096), None, None)
                dd.dd_dataset_destroy(ds)
            dd.dd_dataset_destroy(None)
        least = next(i for i, s in enumerate(sizes) if s)
        print(sizes)
        assert least > 0 and all(sizes[least:]), "created in less memory than this"
        without, whole = sizes[least], sizes[-1]
        assert whole - without >= 32 * n            # no part of the pack stays without the rest
        assert set(sizes) == {{0, without, whole}}
        """)


def test_kept_memory_goes_without_a_call(tmp_path):
    """Released blocks leave the process after their five seconds although the program does
    not call the library again, and the process ends normally with some kept (also where
    a child process of it ended first)."""
    scenario(tmp_path, """
        import os
        base = hip.fake_live()
        rc, ds = create(dd, 1 << 18, FP64 | BF16)
        dd.dd_dataset_destroy(ds)
        kept = hip.fake_live() - base
        assert kept > 20 << 20
        t = time.time()
        while hip.fake_live() > base and time.time() - t < 8.0:
            time.sleep(0.05)
        assert hip.fake_live() == base and 4.0 < time.time() - t < 7.0
        rc, ds = create(dd, 1 << 18, FP64 | BF16)
        dd.dd_dataset_destroy(ds)
        assert hip.fake_live() > base
        child = os.fork()
        if child == 0:
            sys.exit(0)          # runs the exit handlers, without the thread
        assert os.waitpid(child, 0)[1] == 0
        """)


def test_server_memory_is_not_kept(tmp_path):
    """What a server allocates goes back to the driver when it releases it: its budget
    bounds what it holds, and nothing of it stays behind."""
    scenario(tmp_path, """
        rc, ds = create(dd, 1 << 18, FP64 | BF16)
        dd.dd_dataset_destroy(None)
        base = hip.fake_live()
        budget = 400 << 20
        hip.fake_peak()
        rc, srv = server(dd, ds, budget, "bf16", 4096)
        assert rc == 0, dd.dd_last_error()
        for n in (6, 8, 7):                    # operators of 10 to 38 MB, formed and kept by the data set
            assert dd.dd_server_wait(srv, submit(dd, srv, n, n, n), None, 60.0) in (0, 5)
        assert hip.fake_peak() - base <= budget
        operators = 8 * sum(((3 * (n + 1) ** 3 + 63) // 64 * 64) ** 2 for n in (6, 8, 7))
        reserve = stats(dd, srv).reserve_bytes
        slack = 1 << 20                        # buffers below 256 bytes, rounded up
        assert hip.fake_live() - base <= reserve + operators + slack, (hip.fake_live() - base, reserve, operators)
        dd.dd_server_destroy(srv)
        assert hip.fake_live() - base <= operators + slack
        dd.dd_dataset_destroy(ds)
        dd.dd_dataset_destroy(None)
        """)


def test_kept_blocks_are_counted_as_they_are(tmp_path):
    """A data set in blocks that another one left is as large as in its own."""
    scenario(tmp_path, """
        sizes = []
        for first in (0, 290_000, 262_144):
            if first:
                rc, ds = create(dd, first, FP64 | BF16)
                dd.dd_dataset_destroy(ds)
            rc, ds = create(dd, 1 << 18, FP64 | BF16)
            before = hip.fake_live()
            dd.dd_dataset_destroy(None)        # what is left is the data set's
            sizes.append((held(dd, ds), hip.fake_live()))
            dd.dd_dataset_destroy(ds)
            dd.dd_dataset_destroy(None)
        assert len(set(sizes)) == 1, sizes
        """)


@pytest.mark.parametrize("mode,points,tile", [
    ("bf16", 1 << 24, 0), ("bf16", 1 << 26, 0), ("bf16", 1 << 27, 0), ("fp16", 1 << 24, 512), ("bf16", 1 << 22, 128),
    ("bf16", 1 << 26, 128), ("fp32", 1 << 24, 0), ("fp64", 1 << 24, 0), ("fp64", 1 << 27, 0), ("bf16", 1_000_000, 0)])
def test_server_batches_cull(tmp_path, mode, points, tile):
    """The batches of a server, whole ones too, leave out tiles in the scratch it holds,
    and that holds the fallback of every query of a batch."""
    pack = {"bf16": "BF16", "fp16": "FP16", "fp32": "FP32", "fp64": "FP64"}[mode]
    scenario(tmp_path, f"""
        rc, ds = create(dd, {points}, FP64 | {pack}, {tile})
        assert rc == 0, dd.dd_last_error()
        for top in (65536, 40000, 5000):
            need = scratch_need(dd, ds, "{mode}", top)
            for m in (top, top - 1, top // 2 + 1, 4096):
                for left in (0, 1, 700, m):
                    hip.fake_watch(b"none", 0, None)
                    hip.fake_word(b"merge_rerank", min(left, m))
                    rc = project_reserved(hip, dd, ds, "{mode}", m, need)
                    assert rc == 0, (top, m, left, dd.dd_last_error())
                    assert hip.fake_launches(b"cull_kernel") > 0, (top, m, left)
        """)


@pytest.mark.parametrize("mode", ["bf16", "fp32", "fp64", "ann"])
def test_any_block_holds_a_call_or_is_refused_before(tmp_path, mode):
    """Whatever the block, a culled batch that begins in it also ends in it, with every
    query left to the fallback."""
    scenario(tmp_path, f"""
        rc, ds = create(dd, 1 << 22, FP64 | FP32 | BF16 | ANN, 128)
        m = 20000
        need = scratch_need(dd, ds, "{mode}", m)
        culled = 0
        for k in range(400):
            room = need // 4 + k * (need // 200)
            for left in (0, 700, m):
                hip.fake_watch(b"none", 0, None)
                hip.fake_word(b"merge_rerank" if "{mode}" != "ann" else b"walk", left)
                rc = project_reserved(hip, dd, ds, "{mode}", m, room)
                n = hip.fake_launches(b"cull_kernel")
                culled += n > 0
                assert rc == 0 or (n == 0 and room < need), (room, need, left, dd.dd_last_error())
        assert culled > 100, culled
        """)


@pytest.mark.parametrize("box", [(30, 30, 5), (9, 9, 9), (24, 24, 24)])
def test_server_charges_what_it_holds(tmp_path, box):
    """The charged peak covers what forming an operator takes; a body free to move beyond
    the inverse's sizes (16384 unknowns) is solved by CG and charged no operator."""
    large = 3 * (box[0] + 1) * (box[1] + 1) * (box[2] + 1) > 16384
    scenario(tmp_path, f"""
        for clamp in (True, False):
            rc, ds = create(dd, 1 << 14, FP64 | BF16)
            dd.dd_dataset_destroy(None)
            hip.fake_watch(b"none", 0, None)
            base = hip.fake_live()
            hip.fake_peak()
            rc, srv = server(dd, ds, 8 << 30, "bf16", 1024)
            assert dd.dd_server_wait(srv, submit(dd, srv, *{box}, clamp=clamp), None, 60.0) in (0, 5)
            s, peak, formed = stats(dd, srv), hip.fake_peak() - base, hip.fake_launches(b"gj_first_kernel")
            print(clamp, s.reserve_bytes, s.peak_bytes, peak, formed)
            assert (formed > 0) == (clamp or not {large})
            fetch = 96 * 8 * {box[0] * box[1] * box[2]}       # strains and stresses on their way to the host
            assert peak <= s.peak_bytes + fetch + 4096
            assert formed or s.peak_bytes - s.reserve_bytes < 100 << 20     # solver buffers alone
            dd.dd_server_destroy(srv)
            dd.dd_dataset_destroy(ds)
        """)


def test_which_scans_are_culled(tmp_path):
    """Both sides of the lines that the rule draws, warm and cold, per format."""
    scenario(tmp_path, """
        def culled(ds, m, mode, warm, **kw):
            hip.fake_watch(b"none", 0, None)
            assert project(dd, ds, m, mode, vp(4096) if warm else None, **kw) == 0, dd.dd_last_error()
            return hip.fake_launches(b"cull_kernel") > 0
        want = {            # points: (queries, 16 bits warm, 16 bits cold, FP64 warm, FP64 cold)
            1 << 16: [(2048, 0, 0, 0, 0), (2049, 0, 0, 1, 1), (65536, 0, 0, 1, 1)],
            (1 << 18) - 1: [(8, 0, 0, 0, 0), (20000, 0, 0, 1, 1)],
            1 << 18: [(8, 0, 1, 0, 1), (16383, 0, 1, 1, 1), (16384, 1, 1, 1, 1)],
            1 << 19: [(8, 0, 1, 1, 1), (8191, 0, 1, 1, 1), (8192, 1, 1, 1, 1)],
            5 * (1 << 17): [(768, 1, 1, 1, 1), (769, 0, 1, 1, 1), (2048, 0, 1, 1, 1), (2049, 1, 1, 1, 1)],
            (1 << 20) + 1: [(768, 1, 1, 1, 1), (1024, 0, 1, 1, 1), (1025, 1, 1, 1, 1), (2048, 1, 1, 1, 1)],
            1 << 21: [(1, 1, 1, 1, 1), (1024, 1, 1, 1, 1)]}
        for n, rows in want.items():
            rc, ds = create(dd, n, FP64 | FP32 | BF16 | FP16)
            assert rc == 0
            for m, w16, c16, w64, c64 in rows:
                for mode, w, c in (("bf16", w16, c16), ("fp16", w16, c16), ("fp32", w64, c64), ("fp64", w64, c64)):
                    assert culled(ds, m, mode, True) == w, (n, m, mode, "warm")
                    assert culled(ds, m, mode, False) == c, (n, m, mode, "cold")
                    assert culled(ds, m, mode, True, passes=2) == c, (n, m, mode, "stale warm start")
                    assert not culled(ds, m, mode, False, splits=8)
            dd.dd_dataset_destroy(ds)
        """)
