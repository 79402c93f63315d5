"""Tile class of the expert GEMMs at both sides of every line of the rule (host function of the library, no GPU needed)."""
import ctypes as C

import pytest

LOW, MAIN, DECODE = 0, 1, 5


@pytest.mark.parametrize("assigned,E,E_local,d,f,cls", [
    # the mean load alone: below 12 rows per expert, up to 24, above
    (11.9 * 8, 8, 8, 4096, 14336, LOW), (96, 8, 8, 4096, 14336, DECODE), (192, 8, 8, 4096, 14336, DECODE),
    (193, 8, 8, 4096, 14336, MAIN), (16, 8, 8, 4096, 14336, LOW),
    # both GEMMs fill their rounds: 32 experts x 16 weight-row tiles; fewer experts, narrower d, narrower f do not
    (32 * 16, 32, 32, 4096, 2048, LOW), (32 * 16 + 1, 32, 32, 4096, 2048, MAIN), (32 * 12, 32, 32, 3841 // 64 * 64 + 64, 2048, LOW),
    (256 * 16, 256, 25, 4096, 2048, DECODE), (32 * 16, 32, 32, 2816, 2048, DECODE), (32 * 16, 32, 32, 4096, 512, DECODE),
    (32 * 16 + 1, 32, 32, 4096, 512, DECODE), (64 * 20, 64, 64, 2048, 512, DECODE),
    # one and a half rounds, the last one half empty; 1.75 rounds; 2.25 rounds; 2.5 rounds, both ways round
    (48 * 13, 48, 48, 4160, 1024, DECODE), (64 * 14, 64, 64, 3712, 896, LOW), (48 * 20, 48, 48, 3008, 1536, DECODE),
    (64 * 20, 64, 64, 2560, 2048, MAIN), (64 * 20, 64, 64, 4096, 1280, MAIN), (64 * 20, 64, 64, 4096, 1152, DECODE),
    # few items in the first GEMM: loaded experts x 16 weight-row tiles against 140
    (4, 256, 32, 7168, 2048, DECODE), (70, 256, 32, 7168, 2048, DECODE), (100, 256, 32, 7168, 2048, LOW),
    (8, 128, 128, 2048, 768, DECODE), (32, 128, 128, 2048, 768, LOW), (1, 1, 1, 64, 64, DECODE),
    (4, 1, 1, 64, 64, DECODE), (5, 1, 1, 64, 64, LOW), (8, 2, 2, 128, 256, DECODE), (9, 2, 2, 128, 256, LOW),
])
def test_class_at_the_lines(assigned, E, E_local, d, f, cls):
    import paper_2605_19945_amd as moe
    pick = moe.load_library().gemm_pick_class_for
    pick.restype, pick.argtypes = C.c_int, [C.c_double] + [C.c_int] * 4
    assert pick(assigned, E, E_local, d, f) == cls
