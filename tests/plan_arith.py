"""The kernels' split arithmetic (cf_plan_arith.h) compiled for the host and called through ctypes."""
import collections
import ctypes
import os
import subprocess

_HERE = os.path.dirname(os.path.abspath(__file__))
_SRC = os.path.join(_HERE, "native", "plan_arith_host.cpp")
_LIB = os.path.join(_HERE, "native", "libplan_arith_host.so")
_DEPENDS = [_SRC] + [os.path.join(_HERE, "..", "paper_2508_18850_amd", "csrc", f) for f in ("cf_plan_arith.h",)]
_lib = None


def load():
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB) or any(os.path.getmtime(_LIB) < os.path.getmtime(f) for f in _DEPENDS):
            part = "%s.%d" % (_LIB, os.getpid())
            subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-Wall", "-shared", "-fPIC", "-o", part, _SRC], check=True)
            os.replace(part, _LIB)
        _lib = ctypes.CDLL(_LIB)
    return _lib


Dealt = collections.namedtuple("Dealt", "items size splits ranges")      # ranges: per row a list of (t0, t1)


def ragged_gain(head_dim):
    return load().pa_ragged_gain(head_dim)


def deal(lens, team_size, tokens_per_split, gain, pairmap=1, ulps=0):
    n = len(lens)
    size, splits, flat = ctypes.c_int(), (ctypes.c_int * 16)(), (ctypes.c_int * (2 * 16 * 64))()
    items = load().pa_deal(n, (ctypes.c_int * n)(*lens), team_size, tokens_per_split, gain, pairmap, ulps, ctypes.byref(size), splits, flat)
    ranges, at = [], 0
    for b in range(n if items else 0):
        ranges.append([(flat[2 * k], flat[2 * k + 1]) for k in range(at, at + splits[b])])
        at += splits[b]
    return Dealt(items, size.value, list(splits)[:n] if items else [], ranges)
