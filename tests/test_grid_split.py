"""The mix of attention and rejection rows of a launch (host code, compiled here with the host compiler):
attention rows at a regular distance of 2, 4, 6 or 8 rows would always fall on the same compute units
of an XCD, and a step then takes up to half as long again."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2406_14066_amd import build as B


@pytest.fixture(scope="module")
def attention_rows_mixed(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("grid_split")
    src = d / "grid_split.cpp"
    src.write_text('#include "grid_split.h"\nextern "C" int rows_mixed(int a, int r, double s) { return attention_rows_mixed(a, r, s); }\n')
    lib = d / "libgrid_split.so"
    subprocess.run([cxx, "-O1", "-shared", "-fPIC", "-I", B.CSRC, "-o", str(lib), str(src)], check=True)
    f = ctypes.CDLL(str(lib)).rows_mixed
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_double], ctypes.c_int
    return f


def period(rows_mixed, rows_reject):
    return (rows_mixed + rows_reject) / rows_mixed


# (B, Hkv, rejection items: statistics, race, final) of steps whose period was 4.0 to 4.1
@pytest.mark.parametrize("B,Hkv,items", [(96, 8, 864 + 288 + 12), (120, 8, 1080 + 360 + 15), (88, 8, 792 + 264 + 11), (112, 8, 1008 + 336 + 14)])
def test_steps_that_were_in_step_with_the_compute_units(attention_rows_mixed, B, Hkv, items):
    rows_attn, rows_reject = B * Hkv // 8, (items + 7) // 8
    assert 3.9 < period(rows_attn // 2, rows_reject) < 4.1      # half of the attention rows, as they are
    rows = attention_rows_mixed(rows_attn, rows_reject, 0.5)
    assert 3.6 < period(rows, rows_reject) <= 3.7


@pytest.mark.parametrize("span", [0.5, 0.3, 0.9])
def test_attention_rows_spread_over_the_compute_units(attention_rows_mixed, span):
    for rows_attn in (1, 2, 3, 7, 16, 33, 64, 96, 128, 200, 256, 511, 1024):
        for rows_reject in list(range(1, 400, 3)) + [512, 777, 1024, 4096]:
            rows = attention_rows_mixed(rows_attn, rows_reject, span)
            plain = min(max(int(rows_attn * span), 1), rows_attn)
            assert 1 <= rows <= rows_attn
            p0, p1 = period(plain, rows_reject), period(rows, rows_reject)
            if not 3.69 < p0 < 3.81 and all(abs(p0 - e) > 0.0501 * e for e in (2, 4, 6, 8)):
                assert rows == plain
            if rows < 24 or p1 > 8.6:
                continue
            # the positions of the attention rows, as the kernel computes them, over the places of a group of 4
            row = np.arange(rows + rows_reject, dtype=np.int64)
            at = row[(row + 1) * rows // (rows + rows_reject) > row * rows // (rows + rows_reject)]
            assert len(at) == rows
            share = np.bincount(at % 4, minlength=4).max() / rows
            assert share <= 0.5, (rows_attn, rows_reject, rows, p1, share)
