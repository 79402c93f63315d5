"""The order of a work list (csrc/moe_schedule.h, compiled for the host): for every number of heavy and light tiles up to 300,
and around the numbers at which the heavy ones are dealt in longer chunks, each tile stands in exactly one entry, no queue
holds more than an eighth of them rounded up, and nothing stands behind the entries that every launch has; in whole lists
of random loads every 32-row block of every expert meets every weight-row tile once."""
import os

import numpy as np
import pytest

import sched_host

PROGRAM = r"""
#include "moe_schedule.h"
#include <cstdio>
#include <utility>
#include <vector>
int main() {
    std::vector<std::pair<int, int>> lists;  // tiles, light ones among them
    for (int total = 0; total <= 300; ++total)
        for (int n_light = 0; n_light <= total; ++n_light) lists.push_back({total, n_light});
    for (int heavy : {503, 511, 512, 513, 639, 1024, 2031, 2047, 2048, 2049, 2303, 2304, 6144, 20011})
        for (int n_light : {0, 1, 7, 8, 9, 100, heavy / 2 - 1, heavy / 2, heavy / 2 + 1, 3 * heavy}) lists.push_back({heavy + n_light, n_light});
    for (auto [total, n_light] : lists)
        for (bool alike : {false, true}) {
            std::vector<int> heavy(total - n_light), light(n_light);
            int queue[8] = {0};
            for (int b = 0; b < total + 64; ++b) {
                bool is_light;
                const int g = sched_entry(total, n_light, b, &is_light, alike);
                if (g < 0) continue;
                std::vector<int>& tiles = is_light ? light : heavy;
                if (g >= (int)tiles.size() || b >= total + 8 || tiles[g]++ || ++queue[b % 8] > (total + 7) / 8) {
                    printf("total %d light %d entry %d -> %d\n", total, n_light, b, g);
                    return 1;
                }
            }
            for (int x = 0, n = 0; x < 8; ++x)
                if ((n += queue[x], x == 7 && n != total)) {
                    printf("total %d light %d: %d tiles listed\n", total, n_light, n);
                    return 1;
                }
        }
    return 0;
}
"""


needs_hipcc = pytest.mark.skipif(not os.path.exists(sched_host.HIPCC), reason="no hipcc")


@needs_hipcc
def test_every_tile_stands_in_one_entry(tmp_path):
    sched_host.run(sched_host.compile_host(PROGRAM, str(tmp_path)), "")


@pytest.fixture(scope="module")
def lists(tmp_path_factory):
    return sched_host.compile_host(sched_host.PROGRAM, str(tmp_path_factory.mktemp("lists")))


def _loads(kind, E, rng):
    if kind == "zipf":
        return [int(20000 / (e + 1)) for e in rng.permutation(E)]
    if kind == "sparse":
        return [int(n) for n in rng.integers(0, 2, E) * rng.integers(1, 700, E)]
    if kind == "one_block":
        return [int(n) for n in rng.integers(0, 33, E)]
    return [int(n) for n in rng.integers(0, 1200, E)]


@needs_hipcc
@pytest.mark.parametrize("kind", ["zipf", "sparse", "one_block", "even"])
@pytest.mark.parametrize("E,nt,bm", [(1, 1, 288), (3, 112, 288), (8, 16, 128), (31, 5, 64), (64, 24, 288), (256, 7, 288)])
def test_every_block_of_rows_meets_every_weight_row_tile_once(lists, kind, E, nt, bm):
    rows = _loads(kind, E, np.random.default_rng(E * nt + len(kind)))
    cap, entries = sched_host.work_list(lists, rows, nt, bm)
    off = np.concatenate([[0], np.cumsum(rows)])
    seen = set()
    for e, row0, n, n0, _ in entries:
        assert 0 < n <= 32 * cap and (row0 - off[e]) % 32 == 0 and off[e] <= row0 and row0 + n <= off[e + 1]
        assert n % 32 == 0 or row0 + n == off[e + 1]
        for r in range(row0, row0 + n, 32):
            assert (r, n0) not in seen
            seen.add((r, n0))
    assert len(seen) == nt * sum((n + 31) // 32 for n in rows) and {n0 for _, n0 in seen} <= {256 * i for i in range(nt)}


@needs_hipcc
def test_the_tall_loads_of_the_gpu_tests_keep_their_tiles(lists):
    from test_gpu_group_loads import TALL_ROWS, TALL_WIDTHS
    for nt in {(2 * f + 255) // 256 for _, f in TALL_WIDTHS} | {(d + 255) // 256 for d, _ in TALL_WIDTHS}:
        _, entries = sched_host.work_list(lists, TALL_ROWS, nt)
        assert {(rows + 31) // 32 for _, _, rows, _, _ in entries} == {5, 6, 7, 8, 9}, nt


@needs_hipcc
def test_the_last_expert_of_the_epilogue_tests_keeps_its_tile(lists):
    import ctypes as C
    import paper_2605_19945_amd as moe
    from test_gpu_epilogue_edges import D, E, LAST, WHOLE_LOADS
    pick = moe.load_library().gemm_pick_scopes
    pick.restype, pick.argtypes = C.c_int, [C.c_int, C.c_double, C.c_int, C.c_int, C.c_int]
    for (cls, stores), (F, rows, heights) in WHOLE_LOADS.items():
        bm, bn = {0: (128, 256), 1: (288, 256), 5: (64, 128)}[cls]
        for n in {32 * h - less for h in heights for less in LAST}:
            assert pick(cls, (sum(rows) + n) / E, E, D, F) == (3 if stores == "device scope" else 0)
            for nt in (2 * F // bn, D // bn):
                _, entries = sched_host.work_list(lists, rows + [n], nt, bm)
                assert [t[2] for t in entries if t[0] == E - 1] == [n] * nt, (cls, stores, n, nt)
                blocks = {(t[2] + 31) // 32 for t in entries}
                assert blocks >= set(heights), (cls, stores, n, nt)
