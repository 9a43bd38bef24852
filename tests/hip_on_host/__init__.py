"""The library's sources compiled for the CPU (hip/hip_runtime.h here stands in
for HIP's), for tests of indexing and of arrival orders without a GPU."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
_lib = None


def _build(out):
    from paper_1205_1171_amd.build import SOURCES
    csrc = os.path.join(out, "pkg", "csrc")
    os.makedirs(csrc)
    os.symlink(os.path.join(ROOT, "include"), os.path.join(out, "include"))
    src = os.path.join(ROOT, "paper_1205_1171_amd", "csrc")
    for name in os.listdir(src):
        if name.endswith((".hip", ".hpp", ".cpp")):
            with open(os.path.join(src, name)) as fh:
                text = fh.read()
            with open(os.path.join(csrc, name), "w") as fh:  # dynamic LDS: one array for all
                fh.write(text.replace("extern __shared__", "extern"))
    so = os.path.join(out, "libhull3d_host.so")
    flags = ["g++", "-std=c++17", "-O2", "-g1", "-fPIC", "-ffp-contract=off", "-w", "-fno-strict-aliasing",
             "-I", HERE]
    objs, jobs = [], []
    for s in [os.path.join(csrc, n) for n in SOURCES] + [os.path.join(HERE, "emu.cpp")]:
        obj = os.path.join(out, os.path.basename(s) + ".o")
        objs.append(obj)
        jobs.append(subprocess.Popen([*flags, "-I", csrc, "-x", "c++", "-c", s, "-o", obj]))
    assert all([j.wait() == 0 for j in jobs])
    subprocess.check_call(["g++", "-shared", "-Wl,-Bsymbolic", "-o", so, *objs])
    return so


def lib():
    """The library, built once per process."""
    global _lib
    if _lib is None:
        tmp = tempfile.TemporaryDirectory()
        _lib = ctypes.CDLL(_build(tmp.name))
        _lib.tmp = tmp
    return _lib


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def _workspace(size, fill):
    ws = np.full(size + 256, fill, np.uint8)
    at = -ws.ctypes.data % 256
    return ws[at:at + size]


def filter_rc(p):
    """Status of extent_and_filter."""
    L = lib()
    n = len(p)
    size = ctypes.c_size_t()
    assert L.hull_workspace_bytes(ctypes.c_int64(n), 0, ctypes.byref(size)) == 0
    ws = _workspace(size.value, 0xA5)
    L.emu_order(0)
    return L.emu_filter(_p(p), ctypes.c_int64(n), _p(ws), size)


def hull(p, entry="hull_full", order=0, fill=0xA5):
    """Faces of int32 (int64: wide) points by an entry point of single hulls."""
    L = lib()
    wide = p.dtype == np.int64
    n = len(p)
    size = ctypes.c_size_t()
    assert L.hull_workspace_bytes(ctypes.c_int64(n), 1 if wide else 0, ctypes.byref(size)) == 0
    ws = _workspace(size.value, fill)
    faces = np.full((max(2 * n, 1), 3), -9, np.int32)
    info = np.full(2, -9, np.int64)
    L.emu_order(int(order))
    rc = getattr(L, entry + ("_wide" if wide else ""))(
        _p(p), ctypes.c_int64(n), _p(faces), ctypes.c_int64(2 * n), _p(info), _p(ws), size, None)
    assert rc == 0 and info[0] == 0, (rc, info)
    return faces[:info[1]]


def hull_batched(parts, order=0, fill=0xA5, schedule=None):
    """Faces and face offsets of a batch of int32 clouds."""
    L = lib()
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.int64)
    x = np.ascontiguousarray(np.concatenate(parts), dtype=np.int32)
    n, H = int(off[-1]), len(parts)
    size = ctypes.c_size_t()
    assert L.hull_workspace_bytes_batched(ctypes.c_int64(n), ctypes.c_int64(H), ctypes.byref(size)) == 0
    ws = _workspace(size.value, fill)
    faces = np.full((2 * n, 3), -9, np.int32)
    face_off = np.full(H + 1, -9, np.int64)
    info = np.full(2, -9, np.int64)
    L.emu_order(int(order))
    rc = L.hull_full_batched(_p(x), _p(off), _p(off), ctypes.c_int64(H), _p(faces), ctypes.c_int64(2 * n),
                             _p(face_off), _p(info), _p(ws), size,
                             ctypes.byref(schedule) if schedule is not None else None, None)
    assert rc == 0 and info[0] == 0, (rc, info)
    return faces[:info[1]], face_off


def face_adjacency(faces, face_off=None, pt_off=None, order=0):
    """(status, adjacency rows, edges without a twin) of face rows."""
    L = lib()
    F = len(faces)
    size = ctypes.c_size_t()
    assert L.hull_adjacency_workspace_bytes(ctypes.c_int64(F), ctypes.byref(size)) == 0
    ws = _workspace(size.value, 0xA5)
    adj = np.full((max(F, 1), 3), -9, np.int32)
    info = np.full(2, -9, np.int64)
    L.emu_order(int(order))
    H = 1 if face_off is None else len(face_off) - 1
    assert L.hull_face_adjacency(
        _p(faces), ctypes.c_int64(F), _p(face_off) if face_off is not None else None,
        _p(pt_off) if pt_off is not None else None, ctypes.c_int64(H), _p(adj), _p(info), _p(ws), size, None) == 0
    return int(info[0]), adj[:F], int(info[1])
