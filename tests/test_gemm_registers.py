"""Registers of the compiled grouped GEMM kernels that inline asm relies on (no GPU needed): M0 is written in front of
every token load and nowhere else, so that nothing the compiler keeps there is lost."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_19945_amd import build as moe_build

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
@pytest.mark.parametrize("unit", ["moe_gemm_swiglu", "moe_gemm_partial_stream", "moe_gemm_pairsum"])
def test_m0_is_used_by_the_token_loads_only(unit, tmp_path):
    out = tmp_path / "unit.s"
    r = subprocess.run([HIPCC, *moe_build.FLAGS, "-S", "--cuda-device-only", "-o", str(out),
                        os.path.join(moe_build.CSRC, unit + ".hip")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    in_asm, written, loads, other = False, 0, 0, []
    for n, line in enumerate(out.read_text().splitlines()):
        s = line.split(";")[0].strip() if not line.strip().startswith(";;#ASM") else line.strip()
        if s.startswith(";;#ASM"):
            in_asm = s.startswith(";;#ASMSTART")
        elif in_asm:
            written += s.startswith("s_mov_b32 m0,")
            loads += s.startswith("global_load_lds_dwordx4")
        elif re.search(r"\bm0\b", s) or "load_lds" in s:
            other.append(f"line {n + 1}: {s}")
    assert written == loads > 0 and not other, other[:5]
