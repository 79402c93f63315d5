"""Static check of the compiled combine of a split second GEMM (no GPU needed): every number of slabs keeps all its
partial sums in registers (8 per slab and lane, requested together), and up to six slabs leave room for eight
wavefronts per SIMD -- 64 of its 512 registers each -- which the loads in flight at larger batches depend on."""
import os
import re
import subprocess

import pytest

from paper_2605_19945_amd import build as moe_build


@pytest.fixture(scope="module")
def usage():
    cmd = [moe_build._hipcc(), *moe_build.FLAGS, "-c", "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
           os.path.join(moe_build.CSRC, "moe_permute.hip"), "-o", os.devnull]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"remark:\s+(Function Name|VGPRs|ScratchSize \[bytes/lane\]): (\S+)", line)
        if m and m.group(1) == "Function Name":
            name = m.group(2)
            out[name] = {}
        elif m:
            out[name][m.group(1).split()[0]] = int(m.group(2))
    return out


@pytest.mark.parametrize("slabs", range(2, 9))
def test_combine_split_registers(usage, slabs):
    found = [v for n, v in usage.items() if f"combine_split_kernelILi{slabs}E" in n]
    assert len(found) == 1, f"no kernel for {slabs} slabs"
    assert found[0]["ScratchSize"] == 0
    assert found[0]["VGPRs"] >= 8 * slabs
    assert slabs > 6 or found[0]["VGPRs"] <= 64
