"""The choices of csrc/plan.h (pure host code) as plain functions, compiled with the host compiler."""

import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_14220_amd", "csrc")

_SHIM = """
#include "plan.h"
extern "C" int response_blocks(int term, int64_t T, int64_t n_seq, int64_t cus) {
  return tim::response_blocks((tim::ResponseTerm)term, T, n_seq, cus);
}
extern "C" int stream_shape(int64_t rows, int d, int n_ht, int cus) {
  const tim::StreamShape s = tim::stream_shape(rows, d, n_ht, cus);
  return 10 * s.row_blocks + s.group;
}
extern "C" int norm_fused(int64_t T, int d) { return tim::norm_fused(T, d); }
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "shim.cpp"), os.path.join(d, "plan.so")
        with open(src, "w") as f:
            f.write(_SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", so, src],
                       check=True)
        lib = ctypes.CDLL(so)
    lib.response_blocks.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3
    lib.stream_shape.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 3
    lib.norm_fused.argtypes = [ctypes.c_int64, ctypes.c_int]
    return lib


K1, K3, PPO = 0, 1, 2  # ResponseTerm


def response_blocks(term, T, n_seq, cus=256):
    return _lib().response_blocks(term, T, n_seq, cus)


def stream_shape(rows, d, V, cus=256):
    """(row blocks, group) of the wave-per-half kernel for a decode batch, or None for the two-wave tiles."""
    c = _lib().stream_shape(rows, d, -(-V // 128), cus)
    return divmod(c, 10) if c else None


def norm_fused(T, d):
    return bool(_lib().norm_fused(T, d))
