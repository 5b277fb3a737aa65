"""Which kernel the library runs for a call, without a GPU: the C ABI's host
side compiled by the host compiler with the launchers replaced
(host_plan.cpp). Nothing is computed; the pointers are never followed."""

from __future__ import annotations

import ctypes
import functools
import os
import subprocess
import tempfile
from typing import NamedTuple

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(ROOT, "paper_2609_34538_amd")
FAKE = 1 << 20
KERNELS = ["none", "valu", "split", "balanced", "chunk"]
PATHS = {"auto": 0, "valu": 1, "mfma": 2, "balanced": 3}


class _Cache(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in
                ("dtype", "num_depths", "num_layers", "num_kv_heads", "head_dim", "num_pages",
                 "num_k_planes", "num_v_planes")] + [
        ("k_plane", ctypes.c_int32 * 65), ("v_plane", ctypes.c_int32 * 65),
        ("k_pool", ctypes.c_void_p), ("v_pool", ctypes.c_void_p)]


class _Batch(ctypes.Structure):
    _fields_ = [("batch", ctypes.c_int32), ("max_pages_per_seq", ctypes.c_int32),
                ("prefix_len", ctypes.c_void_p), ("block_table", ctypes.c_void_p),
                ("dev_error", ctypes.c_void_p)]


class _Options(ctypes.Structure):
    _fields_ = [("path", ctypes.c_int32), ("pages_per_split", ctypes.c_int32)]


class Plan(NamedTuple):
    status: int
    kernel: str
    merge: bool
    pages_per_split: int
    nsplit: int       # splits or chunks of a unit
    chunk_tiles: int
    workspace: int    # bytes the call was given


def compile_host(src: str, out: str, include=os.path.join(PKG, "csrc")) -> ctypes.CDLL:
    cmd = ["g++", "-shared", "-fPIC", "-O1", "-std=c++17", "-x", "c++", "-D__HIP_PLATFORM_AMD__",
           "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-I" + include, src,
           "-Wl,-Bsymbolic", "-o", out]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    return ctypes.CDLL(out)


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        lib = compile_host(os.path.join(HERE, "host_plan.cpp"), os.path.join(d, "host_plan.so"))
    lib.das_attn_workspace_bytes_ex.restype = ctypes.c_size_t
    return lib


def plan(dtype: str, batch: int, hkv: int, group: int, dh: int, pages: int, w: int,
         path: str = "auto", pps: int = 0, workspace=None, noalloc: bool = False) -> Plan:
    """The plan of a call with `pages` columns of block table. workspace: its
    bytes, by default what the library asks for."""
    lib = _lib()
    c = _Cache(0 if dtype == "f32" else 1, 4, 1, hkv, dh, 1 << 20, 1, 1)
    for r in range(65):
        c.k_plane[r] = c.v_plane[r] = 0
    c.k_pool = c.v_pool = FAKE
    b = _Batch(batch, pages, FAKE, FAKE, None)
    o = _Options(PATHS[path], pps)
    hq = hkv * group
    if workspace is None:
        workspace = lib.das_attn_workspace_bytes_ex(ctypes.byref(c), ctypes.byref(b), hq, w,
                                                    ctypes.byref(o))
    ptrs = [ctypes.c_void_p(FAKE)] * 4 + [None]  # q, keys, values, out; no lse
    head = (ctypes.byref(c), ctypes.byref(b), 0, 1, 4, hq, w, *ptrs)
    if noalloc:
        st = lib.das_attn_policy_noalloc(*head, ctypes.byref(o), None)
    else:
        st = lib.das_attn_policy(*head, ctypes.c_void_p(FAKE), ctypes.c_size_t(workspace),
                                 ctypes.byref(o), None)
    got = (ctypes.c_int32 * 6)()
    lib.last_plan(got)
    return Plan(st, KERNELS[got[0]], bool(got[1]), got[2], got[3], got[4], workspace)
