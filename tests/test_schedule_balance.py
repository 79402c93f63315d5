"""Work of the eight XCDs in a work list (csrc/moe_schedule.h, compiled for the host) of row tiles of unequal height: nothing
is stolen between their queues, so the tall tiles must not gather in one of them."""
import os

import pytest

import sched_host

PROGRAM = r"""
#include "moe_schedule.h"
#include <cstdio>
#include <vector>
int main() {  // in: number of tiles, their heights in list order; out: sum of height + 1 of each XCD
    int n;
    if (scanf("%d", &n) != 1) return 1;
    std::vector<int> h(n);
    for (int& v : h)
        if (scanf("%d", &v) != 1) return 1;
    long sum[8] = {0};
    for (int b = 0; b < n + 64; ++b) {
        bool light;
        const int g = sched_entry(n, 0, b, &light);
        if (g >= n || (g >= 0 && light)) return 1;
        if (g >= 0) sum[b % 8] += h[g] + 1;
    }
    for (long s : sum) printf("%ld ", s);
    return 0;
}
"""

# experts' (row tiles, height of each in 32-row blocks) along the list, weight-row tiles
CASES = {
    "four_tall_four_low": ([(1, 9)] * 4 + [(1, 5)] * 4, 112),
    "first_half_tall": ([(1, 9)] * 32 + [(1, 5)] * 32, 24),
    "rising": ([(1, 5 + i // 13) for i in range(64)], 24),
    "falling_row_tiles": ([(12, 9), (6, 9), (4, 9), (3, 9), (3, 8), (2, 8), (2, 7), (2, 6), (2, 5), (1, 5), (1, 4)], 32),
    "short_list": ([(1, 9)] * 16 + [(1, 4)] * 16, 9),
}


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(sched_host.HIPCC):
        pytest.skip("no hipcc")
    return sched_host.compile_host(PROGRAM, str(tmp_path_factory.mktemp("balance")))


@pytest.mark.parametrize("case", sorted(CASES))
def test_unequal_heights_are_spread_over_the_xcds(program, case):
    experts, nt = CASES[case]
    heights = [h for tiles, h in experts for _ in range(tiles * nt)]
    out = sched_host.run(program, f"{len(heights)} " + " ".join(map(str, heights)))
    work = [int(v) for v in out.split()]
    assert sum(work) == sum(h + 1 for h in heights)
    # Heights that only rise or only fall: in a pair of laps an XCD has chunks x and 15 - x, so two XCDs differ by no more
    # than one chunk times the drop in those laps; the drops of all laps and of the stretch behind them add up to the whole
    # drop, and the stretch may be one tile longer.
    chunk = 32 if len(heights) >= 2048 else 16 if len(heights) >= 512 else 8
    assert max(work) - min(work) <= chunk * (max(heights) - min(heights)) + max(heights) + 1, work
