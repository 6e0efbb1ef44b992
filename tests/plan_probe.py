"""The library's host side built over recording launchers (tests/c/plan_probe.cpp):
what a call would launch, on the CPU, for a given number of compute units."""
import ctypes
import functools
import os
import subprocess
import tempfile
from types import SimpleNamespace

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = [os.path.join(ROOT, "tests", "c", "plan_probe.cpp"),
           os.path.join(ROOT, "paper_2606_25041_amd", "csrc", "ws_api.cpp")]


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "plan_probe.so")
        subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", *SOURCES, "-o", so], check=True)
        lib = ctypes.CDLL(so)
    lib.ws_workspace_bytes.restype = ctypes.c_size_t
    return lib


def _ints(x):
    return np.ascontiguousarray(x, np.int32)


def step(batch, hq, hkv, d, new_len, lens, new_lens=None, f32=False, cus=256):
    """Status of a step and its plan: ragged (every stream has its own split
    count), splits per stream, work items and work-groups launched."""
    lib = _lib()
    lib.probe_cus(cus)
    lens, ns, work, ragged = _ints(lens), np.zeros(batch, np.int32), (ctypes.c_int64 * 2)(), ctypes.c_int(0)
    nl = None if new_lens is None else _ints(new_lens)
    rc = lib.probe_step(batch, hq, hkv, d, new_len, ctypes.c_void_p(lens.ctypes.data),
                        None if nl is None else ctypes.c_void_p(nl.ctypes.data), int(f32), ctypes.byref(ragged),
                        ctypes.c_void_p(ns.ctypes.data), work)
    return SimpleNamespace(status=rc, ragged=bool(ragged.value), splits=ns.tolist(), items=work[0], launched=work[1])


def prefill(batch, hq, hkv, d, seq, block=32, cus=256):
    """Status of a contiguous prefill in equal blocks and its plan: key groups per work-group,
    dealt classes (units per XCD and their log2 per group, 0 units: plain
    order), items per group, work items and work-groups launched."""
    lib = _lib()
    lib.probe_cus(cus)
    out, work = (ctypes.c_int * 4)(), (ctypes.c_int64 * 2)()
    rc = lib.probe_prefill(batch, hq, hkv, d, seq, block, out, work)
    return SimpleNamespace(status=rc, key_groups=out[0], units=out[1], deal_log2=out[2], per_group=out[3],
                           items=work[0], launched=work[1])


def workspace_bytes(op, batch, hq, hkv, max_q, max_k, cus):
    lib = _lib()
    lib.probe_cus(cus)
    return lib.ws_workspace_bytes(op, batch, hq, hkv, max_q, max_k)
