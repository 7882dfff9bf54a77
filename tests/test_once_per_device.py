"""The helper that a launcher asks a device for a kernel's LDS with (csrc/q8_once.h): once per device, again after a
failure, and nothing that one device granted counts for another."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_once_per_device():
    out = os.path.join(ROOT, "tests", "support", "_build")
    os.makedirs(out, exist_ok=True)
    so = os.path.join(out, "q8_once_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_1804_05038_amd", "csrc"),
                    os.path.join(ROOT, "tests", "support", "q8_once_host.cpp"), "-o", so], check=True)
    #        device, works, expected to run, expected to be done
    steps = [(0, 1, 1, 1), (0, 1, 0, 1), (1, 1, 1, 1), (1, 0, 0, 1), (7, 0, 1, 0), (7, 1, 1, 1), (7, 0, 0, 1), (0, 0, 0, 1), (63, 1, 1, 1), (63, 1, 0, 1),
             (64, 1, 1, 1), (64, 1, 1, 1), (-1, 1, 1, 1), (-1, 0, 1, 0)]
    n = len(steps)
    arr = lambda k: (ctypes.c_int * n)(*[s[k] for s in steps])
    ran, ok = (ctypes.c_int * n)(), (ctypes.c_int * n)()
    ctypes.CDLL(so).q8o_run(arr(0), arr(1), n, ran, ok)
    assert list(ran) == [s[2] for s in steps] and list(ok) == [s[3] for s in steps]


def test_no_launcher_keeps_a_flag_of_its_own_for_the_process():
    """Dynamic LDS is asked for through the helper, or on every launch (f32_lds, whose sizes vary)."""
    csrc = os.path.join(ROOT, "paper_1804_05038_amd", "csrc")
    for name in os.listdir(csrc):
        if name.endswith((".hip", ".cpp", ".h")):
            text = open(os.path.join(csrc, name)).read()
            asks = text.count("hipFuncSetAttribute(")
            assert asks == {"q8_internal.h": 1, "q8_fp32.hip": 1}.get(name, 0), name
