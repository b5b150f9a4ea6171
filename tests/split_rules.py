"""The rules by which split products take their form (csrc/split_rules.h), compiled for the host (not a test module itself)."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2303_13775_amd", "csrc")
FEW, NARROW, WIDE = 1, 2, 4
N_CU = 256              # compute units of an MI355X

_SOURCE = r"""
#include <cstdint>
#define __host__
#define __device__
#include "split_rules.h"
extern "C" int forms(long long ub, int N, int K, int heads, int pieces, int n_cu) { return split_forms(ub, N, K, heads, pieces, n_cu); }
extern "C" int form(int f, long long rows, int N, int K, int heads, int pieces, int n_cu) { return split_form(f, rows, N, K, heads, pieces, n_cu); }
extern "C" int grad_block(long long ub, int M, int N) { return split_grad_block(ub, M, N); }
extern "C" int grad_chunks(long long ub, int M, int N, int heads, int n_cu) { return split_grad_chunks(ub, M, N, heads, n_cu); }
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, lib = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
        with open(src, "w") as f:
            f.write(_SOURCE)
        subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
        L = ctypes.CDLL(lib)
    L.forms.argtypes = [ctypes.c_longlong] + [ctypes.c_int] * 5
    L.form.argtypes = [ctypes.c_int, ctypes.c_longlong] + [ctypes.c_int] * 5
    L.grad_block.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    L.grad_chunks.argtypes = [ctypes.c_longlong] + [ctypes.c_int] * 4
    return L


def form(cap, rows, K, N, heads=1, pieces=None):
    """Form of a rows x K x N product of a level bounded by `cap` rows (pieces: rows of whole 16-byte pieces)."""
    pieces = K % 4 == 0 if pieces is None else pieces
    return _lib().form(_lib().forms(cap, N, K, heads, pieces, N_CU), rows, N, K, heads, pieces, N_CU)


def grad_block(cap, M, N):
    """Block of the weight gradients M x N of a level bounded by `cap` rows."""
    return _lib().grad_block(cap, M, N)


def grad_chunks(cap, M, N, heads=1):
    """Chunks of rows of the weight gradients M x N of a level bounded by `cap` rows."""
    return _lib().grad_chunks(cap, M, N, heads, N_CU)
