"""The naps between the polls of a bounded wait (host code, compiled here with the host compiler): the limit is a number of
polls, so a wait that naps for less gives up sooner."""
import ctypes
import shutil
import subprocess

import pytest

from paper_2406_14066_amd import build as B


@pytest.fixture(scope="module")
def total_nap(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("bounded_wait")
    src, lib = d / "wait.cpp", d / "libwait.so"
    src.write_text('#include "bounded_wait.h"\n'
                   'extern "C" long total_nap(int polls, int few, int small) { long t = 0; for (int i = 0; i < polls; ++i) t += nap_length(i, few, small); return t; }\n')
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", B.CSRC, "-o", str(lib), str(src)], check=True)
    f = ctypes.CDLL(str(lib)).total_nap
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_long
    return f


@pytest.mark.parametrize("few", [0, 1])
@pytest.mark.parametrize("small", [0, 1])
def test_every_wait_gives_up_after_about_the_same_time(total_nap, few, small):
    limit = 1 << 20                                     # the default
    assert total_nap(limit, few, small) >= 0.99 * 32 * limit
    # ... and what the data usually takes is polled at short intervals where few blocks wait or the launch is small
    assert total_nap(8, few, small) <= (64 if few or small else 256)
