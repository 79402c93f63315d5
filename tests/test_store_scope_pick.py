"""Device scope of the expert GEMMs' output stores at both sides of every line of the rule (host function of the library,
no GPU needed)."""
import ctypes as C

import pytest

LOW, MAIN, DECODE = 0, 1, 5
NONE, GEMM1, BOTH = 0, 1, 3


@pytest.mark.parametrize("cls,rows,d,scopes", [
    # other classes, and loads whose row tiles share their weight panels
    (LOW, 8, 4096, NONE), (LOW, 128, 4096, NONE), (DECODE, 16, 4096, NONE), (2, 60, 4096, NONE), (MAIN, 288.1, 7168, NONE),
    # both up to 180 rows, then the first GEMM alone
    (MAIN, 25, 4096, BOTH), (MAIN, 180, 4096, BOTH), (MAIN, 180.1, 4096, GEMM1), (MAIN, 288, 4096, GEMM1),
    # no more than an eighth of d
    (MAIN, 288, 2304, GEMM1), (MAIN, 288, 2240, NONE), (MAIN, 256, 2048, GEMM1), (MAIN, 257, 2048, NONE),
    (MAIN, 72, 576, BOTH), (MAIN, 73, 576, NONE), (MAIN, 32, 256, BOTH), (MAIN, 33, 256, NONE),
])
def test_scopes_at_the_lines(cls, rows, d, scopes):
    import paper_2605_19945_amd as moe
    pick = moe.load_library().gemm_pick_scopes
    pick.restype, pick.argtypes = C.c_int, [C.c_int, C.c_double, C.c_int]
    assert pick(cls, rows, d) == scopes
