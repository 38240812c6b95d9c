"""Build-time check of the fp32 step kernels (hipcc cross-compiles without a GPU): no private memory, and two
blocks per compute unit except for the widest variant."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_14066_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="hipcc not installed")
def test_f32_step_kernels_use_no_private_memory(tmp_path):
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [HIPCC] + flags + ["-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, "-Rpass-analysis=kernel-resource-usage",
                             "-S", "--cuda-device-only", "-o", str(tmp_path / "f32.s"), os.path.join(B.CSRC, "step_f32.hip")]
    out = subprocess.run(cmd, check=True, capture_output=True, text=True).stderr
    kernels, name = {}, None
    for line in out.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            v = re.search(r"f32_step_kernelILi(\d)ELi(\d)ELi(\d+)E", m.group(1))
            name = tuple(int(x) for x in v.groups()) if v else None
        m = re.search(r"remark:\s+(ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]): (\d+)", line)
        if m and name is not None:
            kernels.setdefault(name, {})[m.group(1).split(" ")[0]] = int(m.group(2))
    assert len(kernels) == 10, sorted(kernels)   # (row tiles, wave groups, head dim)
    for key, r in kernels.items():
        assert r["ScratchSize"] == 0, (key, r)
        assert r["Occupancy"] >= (1 if key == (3, 4, 128) else 2), (key, r)
