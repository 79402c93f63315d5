"""Registers of the compiled grouped GEMM kernels that inline asm relies on (no GPU needed): M0 is written in front of
every token load and nowhere else, so that nothing the compiler keeps there is lost (it takes no clobber of M0)."""
import re

import pytest

from paper_2605_19945_amd import build as moe_build

UNITS = [u[:-len(".hip")] for u in moe_build.SOURCES if u.startswith("moe_gemm_")]


def test_every_unit_is_looked_at():
    assert len(UNITS) == 7


@pytest.mark.parametrize("unit", UNITS)
def test_m0_is_used_by_the_token_loads_only(unit, gemm_unit_asm):
    in_asm, written, loads, other = False, 0, 0, []
    for n, line in enumerate(gemm_unit_asm[unit]):
        s = line.split(";")[0].strip() if not line.strip().startswith(";;#ASM") else line.strip()
        if s.startswith(";;#ASM"):
            in_asm = s.startswith(";;#ASMSTART")
        elif in_asm:
            written += s.startswith("s_mov_b32 m0,")
            loads += s.startswith("global_load_lds_dwordx4")
        elif re.search(r"\bm0\b", s) or "load_lds" in s:
            other.append(f"line {n + 1}: {s}")
    assert written == loads > 0 and not other, other[:5]
