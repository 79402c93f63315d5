"""The order of a work list (csrc/moe_schedule.h, compiled for the host): for every number of heavy and light tiles up to 300,
and around the numbers at which the heavy ones are dealt in longer chunks, each tile stands in exactly one entry, no queue
holds more than an eighth of them rounded up, and nothing stands behind the entries that every launch has."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

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


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_every_tile_stands_in_one_entry(tmp_path):
    src, exe = tmp_path / "entries.hip", tmp_path / "entries"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_2605_19945_amd", "csrc")
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-I", csrc, "-o", str(exe), str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
