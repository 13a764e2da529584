"""The library's plans of its launches, for tests that have to know which kernel a call takes
(test helper). ``helpers/plan.cpp`` (built here into ``helpers/libplan.so``, linked to
librngx.so) asks the library's own functions; no device is needed."""
from __future__ import annotations

import ctypes
import os
import subprocess

from paper_1609_01257_amd import build as _pkg
from paper_1609_01257_amd import rngx

_HERE = os.path.dirname(os.path.abspath(__file__))
_SRC = os.path.join(_HERE, "helpers", "plan.cpp")
_LIB = os.path.join(_HERE, "helpers", "libplan.so")
_FIELDS = ("block", "chunks", "nontemporal", "pace_gbs", "aligned16", "scheduled", "shift", "segs",
           "seg_rows")


def build(force: bool = True) -> str:
    sources = [_SRC, os.path.join(_pkg.CSRC, "internal.h")]
    if force or not os.path.exists(_LIB) or \
            max(map(os.path.getmtime, sources)) > os.path.getmtime(_LIB):
        tmp = _LIB + ".tmp%d" % os.getpid()
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-fPIC", "-shared",
                        "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I",
                        os.path.join(_pkg.ROOT, "include"), "-I", _pkg.CSRC, "-o", tmp, _SRC,
                        "-L", _pkg.PKG, "-l:librngx.so",
                        "-Wl,-rpath,$ORIGIN/../../paper_1609_01257_amd"], check=True)
        os.replace(tmp, _LIB)
    return _LIB


_lib = None


def lib():
    global _lib
    if _lib is None:
        build(force=False)
        _lib = ctypes.CDLL(_LIB)
    return _lib


def query(n, iters, u32=False, star=False, out=0, launch=None, in_place=False):
    """The plan of a plain launch as a dict; launch: (block, chunks, nontemporal, pace_gbs), by
    default the library's own; in_place: the states stay in their buffer, as after a capture."""
    v = (ctypes.c_uint32 * len(_FIELDS))()
    lib().plan_query(ctypes.byref(rngx.Launch(*(launch or (512, 2, 1, 7000)))),
                     ctypes.c_int(u32), ctypes.c_int(star), ctypes.c_uint32(n),
                     ctypes.c_uint32(iters), ctypes.c_uint64(out), ctypes.c_int(in_place), v)
    return dict(zip(_FIELDS, v))


def served(values):
    """The configuration a served batch of this many (padded) values runs."""
    c = rngx.BatchCfg()
    lib().serve_order_query(ctypes.c_uint64(values), ctypes.byref(c))
    return {name: getattr(c, name) for name, _ in c._fields_}


def batch(values, anchors=True):
    """The configuration an API batch of this many values runs under the default one."""
    c = rngx.BatchCfg()
    lib().batch_order_query(ctypes.c_uint64(values), ctypes.c_int(anchors), ctypes.byref(c))
    return {name: getattr(c, name) for name, _ in c._fields_}


def run_batch_without_anchors(reqs, out):
    """One batch on the null stream as a large one runs without memory for anchors."""
    rc = lib().batch_without_anchors(ctypes.c_void_p(reqs.ctypes.data), ctypes.c_uint32(len(reqs)),
                                     ctypes.c_void_p(out.data_ptr()), ctypes.c_uint64(out.numel()))
    assert rc == rngx.RNGX_OK, rngx.last_error()


def anchor_room(need):
    """Anchors that a slot allocates where it needs this many (one for 8,192 values)."""
    lib().anchor_room_query.restype = ctypes.c_uint64
    return lib().anchor_room_query(ctypes.c_uint64(need))


def stage_tail_faults(chunk, line, columns):
    """Reads of a staged row's last words that miss their word or leave the stage."""
    return lib().stage_tail_faults(ctypes.c_uint32(chunk), ctypes.c_uint32(line),
                                   ctypes.c_uint32(columns))


def table_chunks(m):
    """16-byte pieces in which the table of a batch of m requests is uploaded."""
    lib().table_chunks_query.restype = ctypes.c_uint64
    return lib().table_chunks_query(ctypes.c_uint64(m))
