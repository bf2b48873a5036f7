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
