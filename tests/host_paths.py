"""libdd.so on the device-less runtime of fake_hip.c, for the host-path tests (run as a
child process per scenario: a process has one HIP runtime)."""
import ctypes
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2012_00357_amd", "libdd.so")
vp, i64, i32, u64 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_uint64
FP64, FP32, BF16, FP16, ANN, KMEANS = 0x1, 0x2, 0x4, 0x8, 0x10, 0x20
MODE = dict(fp64=0, fp32=1, bf16=2, ann=3, direct=4, fp16=5, kmeans=6)
C6 = (ctypes.c_double * 36)(*[1.0 if i % 7 == 0 else 0.0 for i in range(36)])


class DatasetOpts(ctypes.Structure):
    _fields_ = [("packs", ctypes.c_uint32), ("tile", i32), ("flags", ctypes.c_uint32)]


class ProjectOpts(ctypes.Structure):
    _fields_ = [("mode", i32), ("splits", i32), ("ann_budget", i32), ("passes", i32), ("stats", vp),
                ("ann_radius_discount", ctypes.c_double)]


class Mesh(ctypes.Structure):
    _fields_ = [("nx", i32), ("ny", i32), ("nz", i32), ("lx", ctypes.c_double), ("ly", ctypes.c_double),
                ("lz", ctypes.c_double)]


class ServerOpts(ctypes.Structure):
    _fields_ = [(n, i32) for n in ("mode", "max_active", "max_batch", "max_queue", "ann_budget", "reserved")]


class Request(ctypes.Structure):
    _fields_ = [("mesh", Mesh), ("mask", vp), ("force", vp), ("init", vp), ("max_iter", i32), ("reserved", i32),
                ("deadline_s", ctypes.c_double)]


class Statistics(ctypes.Structure):
    _fields_ = [(n, i64) for n in ("submitted", "completed", "failed", "rejected", "cancelled", "active", "queued",
                                   "batches", "queries", "peak_active", "peak_bytes", "budget_bytes")] + [
        (n, ctypes.c_double) for n in ("a", "b", "c", "d", "e", "f", "g", "h")] + [("reserve_bytes", i64)]


def load():
    hip = ctypes.CDLL(os.environ["FAKE_HIP"], mode=ctypes.RTLD_GLOBAL)
    dd = ctypes.CDLL(LIB)
    for f in ("fake_live", "fake_peak"):
        getattr(hip, f).restype = ctypes.c_size_t
    for f in ("fake_refused", "fake_launches"):
        getattr(hip, f).restype = ctypes.c_long
    hip.fake_arg.restype = u64
    hip.fake_limit.argtypes = [ctypes.c_size_t]
    dd.dd_last_error.restype = ctypes.c_char_p
    dd.dd_dataset_destroy.argtypes = [vp]
    dd.dd_dataset_info.argtypes = [vp, vp, vp]
    dd.dd_project.argtypes = [vp, vp, i64, vp, vp, vp, vp, vp]
    dd.dd_server_create.argtypes = [vp, ctypes.c_size_t, vp, vp]
    dd.dd_server_submit.argtypes = [vp, vp, vp]
    dd.dd_server_wait.argtypes = [vp, u64, vp, ctypes.c_double]
    dd.dd_server_stats.argtypes = [vp, vp]
    dd.dd_server_destroy.argtypes = [vp]
    return hip, dd


def create(dd, n, packs, tile=0):
    """(status, handle) of a data set of n points; the addresses of its points are not read."""
    out = vp()
    opts = DatasetOpts(packs, tile, 0)
    rc = dd.dd_dataset_create(vp(4096), vp(4096), i64(n), C6, ctypes.byref(opts), None, ctypes.byref(out))
    return rc, out


def held(dd, ds):
    b = i64()
    assert dd.dd_dataset_info(ds, None, ctypes.byref(b)) == 0
    return b.value


def project(dd, ds, m, mode, warm=None, splits=0, passes=0):
    opts = ProjectOpts(MODE[mode], splits, 0, passes, None, 0.0)
    return dd.dd_project(ds, vp(4096), m, warm, ctypes.byref(opts), vp(4096), None, None)


def server(dd, ds, budget, mode, max_batch):
    out = vp()
    o = ServerOpts(MODE[mode], 0, max_batch, 0, 0, 0)
    rc = dd.dd_server_create(ds, budget, ctypes.byref(o), ctypes.byref(out))
    return rc, out


def stats(dd, srv):
    s = Statistics()
    assert dd.dd_server_stats(srv, ctypes.byref(s)) == 0
    return s


def submit(dd, srv, nx, ny, nz, clamp=True, max_iter=1):
    """A solve on a box, its face x = 0 clamped or not; returns its ticket."""
    nodes = (nx + 1) * (ny + 1) * (nz + 1)
    mask = (ctypes.c_uint8 * (3 * nodes))()
    if clamp:
        for k in range(0, nodes, nx + 1):
            mask[3 * k] = mask[3 * k + 1] = mask[3 * k + 2] = 1
    force = (ctypes.c_double * (3 * nodes))()
    init = (i64 * (8 * nx * ny * nz))()
    r = Request(Mesh(nx, ny, nz, float(nx), float(ny), float(nz)), ctypes.addressof(mask),
                ctypes.addressof(force), ctypes.addressof(init), max_iter, 0, 0.0)
    t = u64()
    rc = dd.dd_server_submit(srv, ctypes.byref(r), ctypes.byref(t))
    assert rc == 0, dd.dd_last_error()
    return t.value


def run_scenario(tmp_path, source):
    """Runs `source` (Python, with this module's names) in a child process on the fake runtime."""
    so = os.path.join(str(tmp_path), "libfakehip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.c"), "-lpthread"],
                   check=True, timeout=60)
    code = f"import sys, time, ctypes\nsys.path.insert(0, {HERE!r})\nfrom host_paths import *\nhip, dd = load()\n" + source
    r = subprocess.run([sys.executable, "-c", code], env={**os.environ, "FAKE_HIP": so}, capture_output=True,
                       text=True, timeout=110)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


class Arena(ctypes.Structure):     # ScratchArena of csrc/dd_internal.h
    _fields_ = [("block", vp), ("bytes", ctypes.c_size_t), ("done", vp), ("pinned", vp)]


def scratch_need(dd, ds, mode, m_max):
    f = dd._ZN2dd20project_scratch_needERKNS_7DatasetEil
    f.argtypes, f.restype = [vp, ctypes.c_int, i64], ctypes.c_size_t
    return f(ds, MODE[mode], m_max)


def project_reserved(hip, dd, ds, mode, m, room, warm=vp(4096)):
    """A projection in a block of `room` bytes, as a server's batches run it."""
    block = vp()
    assert hip.hipMalloc(ctypes.byref(block), ctypes.c_size_t(room)) == 0
    f = dd._ZN2dd16project_reservedERKNS_7DatasetEPKdblPKlPK15dd_project_optsPlPdPNS_12ScratchArenaEP12ihipStream_t
    f.argtypes = [vp, vp, ctypes.c_bool, i64, vp, vp, vp, vp, vp, vp]
    pinned = (ctypes.c_uint32 * 64)()
    arena = Arena(block, room, None, ctypes.cast(pinned, vp))
    opts = ProjectOpts(MODE[mode], 0, 0, 0, None, 0.0)
    rc = f(ds, vp(4096), True, m, warm, ctypes.byref(opts), vp(4096), vp(4096), ctypes.byref(arena), None)
    hip.hipFree(block)
    return rc
