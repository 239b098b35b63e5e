"""The library's own tile rule and tile walk of the linear layers (csrc/linear_walk.h), compiled for the CPU."""
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2604_15408_amd.build import CSRC

HERE = os.path.dirname(os.path.abspath(__file__))


@functools.lru_cache(None)
def lib() -> ctypes.CDLL:
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "linear_walk_check.so")
        subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Wextra", "-Werror",
                        f"-I{CSRC}", "-o", so, os.path.join(HERE, "linear_walk_check.cpp")], check=True)
        return ctypes.CDLL(so)


# tiles of 32 nj features x 32 mt rows, per_cu work-groups on a CU
SHAPES = [(8, 8, 1), (8, 7, 1), (8, 6, 1), (8, 5, 1), (8, 4, 1), (6, 4, 1), (6, 2, 1), (4, 4, 1), (4, 3, 1), (2, 1, 1),
          (6, 4, 2), (6, 3, 2), (4, 4, 2), (4, 2, 2), (2, 4, 2), (2, 2, 2)]


@functools.lru_cache(None)
def stages():
    """{(nj, mt, per_cu): LDS stages} as the library has them, in its order."""
    out = (ctypes.c_int * 4)()
    res = {}
    for i in range(lib().linear_shape_count()):
        lib().linear_shape(i, out)
        res[tuple(out[:3])] = out[3]
    return res


def table():
    """The shapes that the rule chooses from, in its order."""
    out = (ctypes.c_int * 3)()
    res = []
    for i in range(lib().linear_table_size()):
        lib().linear_table_shape(i, out)
        res.append(tuple(out))
    return res


def pick(rows_hint, rows, N, K, act):
    """((nj, mt, per_cu), tiles) of a call over `rows` rows with this row estimate."""
    out = (ctypes.c_int * 4)()
    lib().linear_pick(rows_hint, rows, N, K, {"none": 0, "gelu": 1}[act], out)
    return tuple(out[:3]), out[3]


@functools.lru_cache(None)
def call_for(shape, act, K):
    """(rows_hint, N) with the fewest outputs for which the rule picks this shape, or None."""
    nj, mt, _ = shape
    best = None
    for n_tiles in range(1, 65):
        N = 32 * nj * n_tiles
        if N > 8192:
            break
        for m_tiles in range(1, 513):
            for hint in (32 * mt * m_tiles - 31, 32 * mt * m_tiles):
                if (best is None or hint * N < best[0] * best[1]) and hint * N <= 1 << 25 and pick(hint, hint, N, K, act)[0] == shape:
                    best = (hint, N)
    return best


def call_beyond_the_ring(shape, act):
    """(rows_hint, N, K): the same with at least two steps more than the LDS ring has stages."""
    for K in (64 * (stages()[shape] + 2), 768, 1536, 3072):
        found = call_for(shape, act, K)
        if found:
            return (*found, K)
    raise AssertionError(f"no call takes {shape}")
