"""The library's internal GEMM planner and launcher (csrc/kernels.h) for tests
that need no device memory: the argument structures and the two C++ symbols."""
import ctypes as ct
import re
import subprocess

import paper_2608_17995_amd as avits

RESID_GATE = 2  # EpiMode


class Problem(ct.Structure):
    _fields_ = [("A", ct.c_void_p), ("lda", ct.c_int64), ("W", ct.c_void_p), ("bias", ct.c_void_p), ("M", ct.c_int64),
                ("out0", ct.c_void_p), ("ld0", ct.c_int64), ("out1", ct.c_void_p), ("ld1", ct.c_int64),
                ("out2", ct.c_void_p), ("ld2", ct.c_int64), ("resid", ct.c_void_p), ("ldr", ct.c_int64),
                ("gate", ct.c_void_p), ("scat", ct.c_void_p), ("scat_idx", ct.c_void_p), ("scat_row0", ct.c_int64),
                ("scat_ld", ct.c_int64), ("scat_n", ct.c_int64), ("row0", ct.c_int64)]


class ModRows(ct.Structure):
    _fields_ = [("B", ct.c_int32), ("stride", ct.c_int64), ("end", ct.c_int64 * 32)]


class Args(ct.Structure):
    _fields_ = [("p", Problem * 2), ("nprob", ct.c_int), ("N", ct.c_int64), ("K", ct.c_int64), ("n_split", ct.c_int64),
                ("n_split2", ct.c_int64), ("mode0", ct.c_int), ("mode1", ct.c_int), ("mode2", ct.c_int), ("mod", ModRows)]


class Plan(ct.Structure):
    _fields_ = [("bn", ct.c_int), ("splits", ct.c_int), ("stages", ct.c_int), ("tiles", ct.c_int64), ("tail", ct.c_int64),
                ("tail_splits", ct.c_int)]


def _symbol(name):
    out = subprocess.run(["nm", "-D", "--defined-only", avits.lib_path()], capture_output=True, text=True).stdout
    return getattr(ct.CDLL(avits.lib_path()), re.search(rf"\bT (_ZN5avits\d+{name}\w*)", out).group(1))


def launch(args, dtype, partial, partial_bytes):
    f = _symbol("launch_gemm")
    f.argtypes = [ct.c_void_p, ct.c_int, ct.c_void_p, ct.c_char_p, ct.c_void_p, ct.c_size_t, ct.c_void_p]
    return f(ct.addressof(args), dtype, None, b"gemm", partial, partial_bytes, None)


def plan(args, dtype, partial_bytes):
    f = _symbol("plan_gemm")
    f.argtypes = [ct.c_void_p, ct.c_int, ct.c_size_t, ct.c_char_p, ct.c_bool]
    f.restype = Plan
    return f(ct.addressof(args), dtype, partial_bytes, b"gemm", False)
