"""Build-time check of the KV append's loads (hipcc cross-compiles without a GPU): what the kernel is made
for is a short chain of loads, and the compiler moves them, which no parity test notices."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_14066_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="hipcc not installed")
def test_rows_are_whole_vectors_and_16_bit_rows_come_first(tmp_path):
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    asm = tmp_path / "attn_generic.s"
    subprocess.run([HIPCC] + flags + ["-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, "-S", "--cuda-device-only", "-o", str(asm),
                                      os.path.join(B.CSRC, "attn_generic.hip")], check=True, capture_output=True)
    kernels = {}
    for m in re.finditer(r"^_ZN\S*kv_append_kernelI([ft])(?:Lb(\d)E)?E\S*:\s(.*?)^\.Lfunc_end", asm.read_text(), re.S | re.M):
        kernels[m.group(1), m.group(2)] = re.findall(r"^\t(global_(?:load|store)\w*)", m.group(3), re.M)
    assert set(kernels) == {("f", "0"), ("t", "0"), ("t", "1")}, sorted(kernels)     # (element, tiled)
    for (element, tiled), ops in kernels.items():
        loads = [o for o in ops if "load" in o]
        vectors, shorts = loads.count("global_load_dwordx4"), loads.count("global_load_ushort")
        assert (vectors, shorts) == {("f", "0"): (4, 0), ("t", "0"): (2, 0), ("t", "1"): (1, 8)}[element, tiled], (element, tiled, ops)
        if element == "t":     # the rows, then the lengths they do not depend on
            assert set(loads[: vectors + shorts]) <= {"global_load_dwordx4", "global_load_ushort"}, (tiled, loads)
