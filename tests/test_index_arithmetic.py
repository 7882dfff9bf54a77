"""The index arithmetic that kernels share with this host build (csrc/q8_index.h): every piece of work is dealt out
exactly once, and every address that follows from it lies inside the array it reads."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    out = os.path.join(ROOT, "tests", "support", "_build")
    os.makedirs(out, exist_ok=True)
    so = os.path.join(out, "q8_index_host.so")
    subprocess.run(["gcc", "-O2", "-std=c11", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_1804_05038_amd", "csrc"),
                    os.path.join(ROOT, "tests", "support", "q8_index_host.c"), "-o", so], check=True)
    return ctypes.CDLL(so)


def _ints(n):
    return (ctypes.c_int * n)()


@pytest.mark.parametrize("first", [0, 1, 90, 100000])
@pytest.mark.parametrize("lens", [[30, 30, 30], [1], [7, 0, 0, 5, 0], [0, 0], [60] * 200, [1] * 3, [1024] * 1000])
@pytest.mark.parametrize("blocks", [1, 2, 97, 384, 768])
def test_position_runs_cover_the_sentences_of_a_group_once(lib, first, lens, blocks):
    """Offsets that begin at any value: the runs are back to back from the first position to the last, none longer
    than the others by more than one, and each begins inside one of the sentences."""
    off = np.concatenate([[first], first + np.cumsum(lens)]).astype(np.int32)
    pos, end = _ints(blocks), _ints(blocks)
    lib.q8x_position_runs(off.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), len(lens), blocks, pos, end)
    pos, end = np.array(pos[:]), np.array(end[:])
    assert pos[0] == off[0] and end[-1] == off[-1] and (pos[1:] == end[:-1]).all()
    assert (end >= pos).all() and np.ptp(end - pos) <= 1
    for p in pos[pos < end]:
        assert ((off[:-1] <= p) & (p < off[1:])).sum() == 1
