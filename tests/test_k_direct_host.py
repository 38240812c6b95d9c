"""The attention kernels with K straight into operand order: what they are built from (hipcc cross-compiles
without a GPU)."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2406_14066_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="hipcc not installed")
def test_they_use_no_private_memory_and_keep_two_blocks_per_unit(tmp_path):
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]

    def compile_part(part):
        cmd = [HIPCC] + flags + ["-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, "-DSPEC_STEP_PART=%d" % part,
                                 "-Rpass-analysis=kernel-resource-usage", "-S", "--cuda-device-only", "-o", str(tmp_path / ("p%d.s" % part)),
                                 os.path.join(B.CSRC, B.STEP_KERNEL)]
        return subprocess.run(cmd, check=True, capture_output=True, text=True).stderr

    with ThreadPoolExecutor(max_workers=3) as pool:
        outs = list(pool.map(compile_part, (1, 2, 3)))
    kernels, name = {}, None
    for line in "\n".join(outs).splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            v = re.search(r"attn_k_direct_kernelILi(\d)ELi(\d)E", m.group(1))
            name = tuple(int(x) for x in v.groups()) if v else None
        m = re.search(r"remark:\s+(ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]): (\d+)", line)
        if m and name is not None:
            kernels.setdefault(name, {})[m.group(1).split(" ")[0]] = int(m.group(2))
    assert set(kernels) == {(2, 1), (3, 1), (2, 2), (3, 2)}, sorted(kernels)   # (row tiles, wave groups)
    for key, r in kernels.items():
        assert r["ScratchSize"] == 0 and r["Occupancy"] >= 2, (key, r)
