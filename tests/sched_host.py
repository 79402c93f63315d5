"""The work-list code of csrc/moe_schedule.h compiled for the host: whole lists from the rows of every expert."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

# In: experts, weight-row tiles, tallest tile in blocks, reduction splits, entries of the list, rows of every expert.
# Out: the cap, then expert, first row, rows, first packed weight row and XCD of every entry that holds a tile.
PROGRAM = r"""
#include "moe_schedule.h"
#include <cstdio>
#include <vector>
int main() {
    int E, nt, hmax, nsplit, grid;
    if (scanf("%d %d %d %d %d", &E, &nt, &hmax, &nsplit, &grid) != 5) return 1;
    std::vector<int> off(E + 1), tot(SCHED_CAPS + 1);
    std::vector<int> pre[2] = {std::vector<int>(E + 1), std::vector<int>(E + 1)};
    bool alike = true;
    for (int e = 0; e < E; ++e) {
        int n;
        if (scanf("%d", &n) != 1) return 1;
        off[e + 1] = off[e] + n;
        const int nblk = (n + 31) / 32;
        alike &= nblk <= 1;
        tot[0] += nblk;
        for (int c = 0; c < SCHED_CAPS; ++c)
            if (hmax - c >= sched_min_cap_blocks(32 * hmax)) tot[c + 1] += (nblk + hmax - c - 1) / (hmax - c);
    }
    const int cap = sched_cap(tot.data(), hmax, nt, nsplit, grid);
    for (int e = 0; e < E; ++e) {
        const int nblk = (off[e + 1] - off[e] + 31) / 32, mte = (nblk + cap - 1) / cap;
        const bool heavy = alike || sched_heavy(nblk, mte);
        pre[0][e + 1] = pre[0][e] + (heavy ? mte : 0);
        pre[1][e + 1] = pre[1][e] + (heavy ? 0 : mte);
    }
    printf("%d\n", cap);
    const int n_light = pre[1][E] * nt, total = pre[0][E] * nt + n_light;
    for (int b = 0; b < grid; ++b) {
        bool light;
        const int g = sched_entry(total, n_light, b, &light, alike);
        if (g < 0) continue;
        const TileDesc t = sched_tile(g, pre[light ? 1 : 0].data(), off.data(), E, nt, 256);
        printf("%d %d %d %d %d\n", t.expert, t.row0, t.rows, t.n0, b % 8);
    }
    return 0;
}
"""


def compile_host(program, where):
    """Path of `program` compiled against the work-list header, in the directory `where`."""
    src, exe = os.path.join(where, "sched.hip"), os.path.join(where, "sched")
    with open(src, "w") as fh:
        fh.write(program)
    csrc = os.path.join(ROOT, "paper_2605_19945_amd", "csrc")
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-I", csrc, "-o", exe, src],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


def run(exe, text):
    r = subprocess.run([exe], input=text, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    return r.stdout


def work_list(exe, rows, nt, bm=288, nsplit=1, n_rows_cap=None):
    """(cap, [(expert, first row, rows, first packed weight row, XCD), ...]) for the list a plan of `bm`-row tiles has."""
    n = sum(rows) if n_rows_cap is None else n_rows_cap
    tall = n // bm + min(n, len(rows)) + 1   # the host's bound on the row tiles, and a quarter more
    grid = (tall + tall // 4) * nt + 64
    lines = run(exe, f"{len(rows)} {nt} {bm // 32} {nsplit} {grid} " + " ".join(map(str, rows))).splitlines()
    return int(lines[0]), [tuple(map(int, x.split())) for x in lines[1:]]
