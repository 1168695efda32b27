"""Which launches a product takes: the library's own rules
(paper_2609_09095_amd/csrc/dispatch.hpp), compiled with g++ on first use, so
that a test of one kernel can assert that its shape still reaches it."""
from __future__ import annotations

import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_09095_amd", "csrc")
_HOST = os.path.join(ROOT, "tests", "host")
_SRC = os.path.join(_HOST, "dispatch_rules.cpp")
_HDR = os.path.join(CSRC, "dispatch.hpp")
_LIB = os.path.join(_HOST, "libdispatch.so")
_lib = None


def rules():
    global _lib
    if _lib is None:
        newest = max(os.path.getmtime(_SRC), os.path.getmtime(_HDR))
        if not os.path.exists(_LIB) or os.path.getmtime(_LIB) < newest:
            tmp = _LIB + ".tmp%d" % os.getpid()
            subprocess.check_call(["g++", "-O2", "-std=c++20", "-shared", "-fPIC", f"-I{CSRC}", "-o", tmp, _SRC])
            os.replace(tmp, _LIB)
        L = ctypes.CDLL(_LIB)
        i64 = ctypes.c_int64
        for name, args, res in (("rule_one_kernel", 5, ctypes.c_int), ("rule_fused_a", 2, ctypes.c_int),
                                ("rule_fused_moduli", 1, ctypes.c_int), ("rule_reconstruct_strips", 2, ctypes.c_int),
                                ("rule_xcd_ranges", 3, ctypes.c_int),
                                ("rule_both_at_once", 5, ctypes.c_int), ("rule_scan_both_slabs", 2, i64),
                                ("rule_scan_both_blocks", 3, i64)):
            f = getattr(L, name)
            f.argtypes = [i64] * args
            f.restype = res
        _lib = L
    return _lib


def route(m, n, k, lda=None, ldb=None):
    """"one" (one launch), "fused" (storage mode F for A) or "staged": what
    the fixed-t ozaki25_dgemm* entry points run."""
    L = rules()
    if L.rule_one_kernel(m, n, k, k if lda is None else lda, n if ldb is None else ldb):
        return "one"
    return "fused" if L.rule_fused_a(m, n) else "staged"
