"""Device scope of the expert GEMMs' output stores at both sides of every line of the rule (host function of the library,
no GPU needed)."""
import ctypes as C

import pytest

LOW, MAIN, DECODE = 0, 1, 5
NONE, GEMM1, BOTH = 0, 1, 3


@pytest.mark.parametrize("cls,rows,E_local,d,f,scopes", [
    # other classes, and loads whose row tiles share their weight panels
    (LOW, 8, 32, 4096, 4096, NONE), (LOW, 128, 32, 4096, 4096, NONE), (DECODE, 16, 32, 4096, 4096, NONE),
    (2, 60, 32, 4096, 4096, NONE), (MAIN, 288.1, 32, 7168, 2048, NONE),
    # a round of second-GEMM work items: both up to 180 rows, then the first GEMM alone; no full round: the first alone
    (MAIN, 25, 16, 4096, 4096, BOTH), (MAIN, 180, 16, 4096, 4096, BOTH), (MAIN, 180.1, 16, 4096, 4096, GEMM1),
    (MAIN, 288, 16, 4096, 4096, GEMM1), (MAIN, 25, 15, 4096, 4096, GEMM1), (MAIN, 25, 15, 4160, 4096, GEMM1),
    (MAIN, 25, 15, 4352, 4096, GEMM1), (MAIN, 25, 15, 4416, 4096, BOTH),
    # weights of 256 MiB (44.7 million elements in each of the three)
    (MAIN, 64, 128, 832, 448, BOTH), (MAIN, 64, 128, 768, 448, NONE),
    # 400 work items of the first GEMM
    (MAIN, 64, 128, 1024, 384, NONE), (MAIN, 25, 16, 4096, 3200, BOTH), (MAIN, 25, 16, 4096, 3072, NONE),
    (MAIN, 25, 8, 4096, 6400, GEMM1), (MAIN, 96, 1, 8192, 51200, GEMM1), (MAIN, 96, 1, 8192, 51072, NONE), (MAIN, 96, 2048, 65536, 65536, BOTH),
    # mean load of no more than an eighth of d
    (MAIN, 288, 16, 2304, 4096, GEMM1), (MAIN, 288, 16, 2240, 4096, NONE), (MAIN, 256, 16, 2048, 4096, GEMM1),
    (MAIN, 257, 16, 2048, 4096, NONE), (MAIN, 72, 128, 576, 2048, BOTH), (MAIN, 73, 128, 576, 2048, NONE),
])
def test_scopes_at_the_lines(cls, rows, E_local, d, f, scopes):
    import paper_2605_19945_amd as moe
    pick = moe.load_library().gemm_pick_scopes
    pick.restype, pick.argtypes = C.c_int, [C.c_int, C.c_double, C.c_int, C.c_int, C.c_int]
    assert pick(cls, rows, E_local, d, f) == scopes
