"""Build-time check of the split requests' merge (hipcc cross-compiles without a GPU): with one row tile
or a head dim of 64 the three loads of a chunk's partial results are issued together.  With a
condition per lane on each, the compiler puts a branch around every load, and launches of split
requests take up to 6% longer, which no parity test notices."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2406_14066_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="hipcc not installed")
def test_a_chunk_of_the_merge_is_loaded_under_one_branch(tmp_path):
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]

    def compile_part(part):
        asm = tmp_path / ("step_part%d.s" % part)
        subprocess.run([HIPCC] + flags + ["-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, "-DSPEC_STEP_PART=%d" % part, "-S",
                                          "--cuda-device-only", "-o", str(asm), os.path.join(B.CSRC, B.STEP_KERNEL)],
                       check=True, capture_output=True)
        return asm

    with ThreadPoolExecutor(max_workers=3) as pool:
        parts = list(pool.map(compile_part, range(3)))
    runs = {}   # kernel -> lengths of the uninterrupted runs of the merge's loads
    for asm in parts:
        name, run = None, 0
        for line in open(asm):
            m = re.match(r"^\S*spec_step_kernelILi(\d)ELi1ELb1ELb0ELi(\d)E\S*:\s", line)   # one wave group, attention alone
            if m:
                name = tuple(int(x) for x in m.groups())
                runs[name], run = [], 0
            elif name is not None and re.search(r"^\s+global_load_dwordx2 .* sc1\s", line):   # (the partials are read past the XCD's cache)
                run += 1
            elif name is not None and (re.match(r"^\.LBB|^\s+s_cbranch|^\s+s_branch", line) or "-- End function" in line):
                if run:
                    runs[name].append(run)
                run = 0
                if "-- End function" in line:
                    name = None
    assert len(runs) == 15, sorted(runs)   # (row tiles, variant); variants 3 and 4 have a head dim of 64
    for name, lengths in runs.items():
        assert sum(lengths) == 24 * (2 if name[0] >= 2 else 1), (name, lengths)   # 8 chunks of 1 or 2 rows
        if name[0] == 1 or name[1] in (3, 4):
            assert all(n % 3 == 0 for n in lengths), (name, lengths)
